// Sketches of float rows: a row's elements rounded to 8 bits under a scale of its own, with a bound of
// what the rounding took away.  A search reads the sketch of a vertex first (128 bytes where the
// row has 320 to 496, 256 where it has 640 to 1,008) and the row itself only if the vertex may still be nearer than the
// beam's last entry.  A vertex is dropped only where its distance, as the search would compute it, is
// certainly beyond that entry, so nothing that a search returns depends on the sketches.
//
// Layout: lane `sub` of a group of eight holds dwords j = 0 .. 4 SK - 1, dword j the four elements of the
// row's 16-byte piece sub + 8 j (the pieces that the lane holds of the query, too), four dwords per 16
// bytes at (8 s + sub) * 16.  The last dword of lane 7 belongs to no piece: it holds the scale (high
// half, the upper half of a float) and the bound (low half, likewise).
//
// With x the row, s its scale, v the rounded row (whole numbers of at most 127), e >= |x - s v|; q the
// query, t v' its rounding to whole numbers of at most 32,512; A = <v, v'>, exact in 32 bits
// (127 * 32,512 * 252):
//   inner product: <q, x> <= t s A + |q| (e + |q - t v'| / |q| * |s v|), and |q - t v'| <= 2.5e-4 |q|
//     whatever q (half a step per element, at most 252 elements, the largest of which is 32,512 steps).
//     The bound that is stored is e + 4e-4 |x|: the rest of the 1.5e-4 is for the rounding of the fp32 sums on
//     both sides (at most 64 * 2^-24 of |q| |x| each).
//   squared L2: |q - x| >= |q - s v| - e, and |q - s v|^2 = |q|^2 + s^2 <v, v> - 2 t s A up to
//     2 |q - t v'| |s v| <= r (|q|^2 + |s v|^2), r = |q - t v'| / |q| (measured once per query); the rounding of these
//     few fp32 operations is within 2^-16 of |q|^2 + |s v|^2, and that of the distance the search
//     itself would compute within 2^-18 of it.
// Rows and queries that these bounds don't cover (largest element outside 1e-12 .. 1e12, infinities, NaN)
// are marked so that every comparison fails and nothing is dropped.
#pragma once
#include "ann_device.hpp"

namespace annmi {

constexpr float SKETCH_LEAST = 1e-12f, SKETCH_MOST = 1e12f;
// Rows with a sketch of 128 SK bytes have at least so many pieces (sketch_bytes: 20 to 31, 40 to 63), so that every lane
// of a group has pieces in each 16-byte part that it holds.
template <int SK>
constexpr u32 SKETCH_PIECES = SK == 1 ? 20 : 40;
static_assert(SKETCH_PIECES<1> >= (u32)LPC && SKETCH_PIECES<2> >= 32u + (u32)LPC);

struct SketchTable {
  const char* base;  // 128 * SK bytes per vertex
};

__device__ __forceinline__ float group_max(float v) {
  v = __builtin_fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true)));
  v = __builtin_fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, true)));
  v = __builtin_fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xF, 0xF, true)));
  return v;
}
// every lane of a group of eight gets the word of the group's last lane (row_newbcast of lanes 7 and 15)
__device__ __forceinline__ u32 group_last(u32 v) {
  const int lo = __builtin_amdgcn_update_dpp(0, (int)v, 0x157, 0xF, 0x3, false);
  return (u32)__builtin_amdgcn_update_dpp(lo, (int)v, 0x15F, 0xF, 0xC, false);
}

// the query as two planes of 8 bits, v' = 256 hi + lo, in LDS: 16 bytes per plane, piece and lane of a group
struct SketchQuery {
  const uint4* mine;  // this lane's first: piece s of the high plane at [2 s * 8], of the low one at [(2 s + 1) * 8]
  float t;   // NaN: nothing may be dropped
  float a;   // inner product: |q|; squared L2: (1 - r) |q|^2
  float r1;  // squared L2: 1 - r
};

template <int KIND, int NCH, int SK>
__device__ __forceinline__ SketchQuery sketch_query(const QueryRegs<KIND, 16, NCH>& Q, uint4* lds, int lane) {
  SketchQuery S;
  u32* words = reinterpret_cast<u32*>(lds);
  const int sub = lane & (LPC - 1);
  S.mine = lds + sub;
  float most = 0.0f, sum = 0.0f;
#pragma unroll
  for (int u = 0; u < NCH; ++u)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float x = __uint_as_float(Q.q[u].w[i]);
      most = __builtin_fmaxf(most, __builtin_fabsf(x));
      sum = __builtin_fmaf(x, x, sum);
    }
  most = group_max(most);
  sum = group_sum(sum);
  const float t = most * (1.0f / 32512.0f);
  const float inv = 32512.0f / most;
  float err = 0.0f;
#pragma unroll
  for (int j = 0; j < 4 * SK; ++j) {
    u32 h = 0, l = 0;
    if (j < NCH) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float x = __uint_as_float(Q.q[j < NCH ? j : 0].w[i]);
        float v = __builtin_rintf(x * inv);
        v = __builtin_fminf(__builtin_fmaxf(v, -32512.0f), 32512.0f);
        const float e = __builtin_fmaf(-t, v, x);
        err = __builtin_fmaf(e, e, err);
        const int n = (int)v, hi = (n + 128) >> 8, lo = n - hi * 256;
        h |= ((u32)hi & 0xFFu) << (8 * i);
        l |= ((u32)lo & 0xFFu) << (8 * i);
      }
    }
    if (lane < LPC) {
      words[(((j >> 2) * 2 + 0) * LPC + sub) * 4 + (j & 3)] = h;
      words[(((j >> 2) * 2 + 1) * LPC + sub) * 4 + (j & 3)] = l;
    }
  }
  __syncthreads();
  err = group_sum(err);
  // (a NaN among the elements passes by the maximum, but not by the sum)
  const bool ok = most >= SKETCH_LEAST && most <= SKETCH_MOST && sum < __builtin_inff();
  S.t = ok ? t : __builtin_nanf("");
  if constexpr (KIND == K_F32_IP) {
    S.a = __builtin_sqrtf(sum) * 1.00001f;
    S.r1 = 0.0f;
  } else {
    S.r1 = 1.0f - (__builtin_sqrtf(err / sum) * 1.001f + 1.6e-5f);
    S.a = S.r1 * sum;
  }
  return S;
}

// What the beam's last entry sets for a launch of candidates: certainly beyond it is what compares so.
struct SketchBound {
  float w, w2;
};
template <int KIND>
__device__ __forceinline__ SketchBound sketch_bound(u64 worst) {
  const float d = float_from_dkey(key_dkey(worst));
  if constexpr (KIND == K_F32_IP) return SketchBound{-d, 0.0f};
  const float w = d * 1.00001f;
  return SketchBound{w, __builtin_sqrtf(w) * 2.00001f};
}

// Passes t0 .. t0 + PBX - 1 over the candidates cid[0 .. cnt), eight per pass as in eval_passes; `drop`
// becomes true in the lanes whose candidate (cand_of_lane) is certainly beyond the bound.
template <int KIND, int SK, int PBX>
__device__ __forceinline__ void sketch_passes(const SketchTable& K, const SketchQuery& S, const SketchBound& B,
                                              const u32* cid, u32 cnt, u32 t0, u32 last_off, int sub, u32 grp, bool& drop) {
  uint4 x[PBX][SK];
#pragma unroll
  for (int tt = 0; tt < PBX; ++tt) {
    const u32 c = 8u * (t0 + tt) + grp;
    const char* row = K.base + (u64)cid[c < cnt ? c : 0u] * (128u * SK);
#pragma unroll
    for (int s = 0; s < SK; ++s)
      x[tt][s] = *reinterpret_cast<const uint4*>(row + (s + 1 < SK ? (u32)(s * 128 + sub * 16) : last_off));
  }
  i32 ah[PBX], al[PBX], vv[PBX];
#pragma unroll
  for (int tt = 0; tt < PBX; ++tt) ah[tt] = al[tt] = vv[tt] = 0;
#pragma unroll
  for (int s = 0; s < SK; ++s) {
    const uint4 h = S.mine[2 * s * LPC], l = S.mine[(2 * s + 1) * LPC];
#pragma unroll
    for (int tt = 0; tt < PBX; ++tt) {
      const uint4 w = x[tt][s];
      ah[tt] = __builtin_amdgcn_sdot4((i32)h.x, (i32)w.x, ah[tt], false);
      al[tt] = __builtin_amdgcn_sdot4((i32)l.x, (i32)w.x, al[tt], false);
      ah[tt] = __builtin_amdgcn_sdot4((i32)h.y, (i32)w.y, ah[tt], false);
      al[tt] = __builtin_amdgcn_sdot4((i32)l.y, (i32)w.y, al[tt], false);
      ah[tt] = __builtin_amdgcn_sdot4((i32)h.z, (i32)w.z, ah[tt], false);
      al[tt] = __builtin_amdgcn_sdot4((i32)l.z, (i32)w.z, al[tt], false);
      ah[tt] = __builtin_amdgcn_sdot4((i32)h.w, (i32)w.w, ah[tt], false);
      al[tt] = __builtin_amdgcn_sdot4((i32)l.w, (i32)w.w, al[tt], false);
      if constexpr (KIND == K_F32_L2) {
        i32 v = __builtin_amdgcn_sdot4((i32)w.x, (i32)w.x, 0, false);
        v = __builtin_amdgcn_sdot4((i32)w.y, (i32)w.y, v, false);
        v = __builtin_amdgcn_sdot4((i32)w.z, (i32)w.z, v, false);
        const i32 last = s + 1 == SK && sub == LPC - 1 ? 0 : (i32)w.w;  // (scale and bound do not count)
        vv[tt] += __builtin_amdgcn_sdot4(last, last, v, false);
      }
    }
  }
#pragma unroll
  for (int tt = 0; tt < PBX; ++tt) {
    const u32 meta = group_last(x[tt][SK - 1].w);
    const float dot = (float)group_sum(ah[tt] * 256 + al[tt]) * S.t * __uint_as_float(meta & 0xFFFF0000u);
    const float e = __uint_as_float(meta << 16);
    bool beyond;
    if constexpr (KIND == K_F32_IP) {
      beyond = __builtin_fmaf(e, S.a, dot) < B.w;
    } else {
      const float s = __uint_as_float(meta & 0xFFFF0000u);
      const float xx = (float)group_sum(vv[tt]) * s * s;
      beyond = __builtin_fmaf(xx, S.r1, S.a) - 2.0f * dot > __builtin_fmaf(e, e + B.w2, B.w);
    }
    if ((u32)sub == t0 + tt) drop = beyond;
  }
}

// Which of the candidates cid[0 .. cnt), cnt <= 64, are certainly beyond the bound (by cand_of_lane).
template <int KIND, int SK>
__device__ __forceinline__ bool sketch_drops(const SketchTable& K, const SketchQuery& S, u64 worst, const u32* cid,
                                             u32 cnt, u32 last_off, int lane) {
  const int sub = lane & (LPC - 1);
  const u32 grp = (u32)lane >> 3;
  const SketchBound B = sketch_bound<KIND>(worst);
  const u32 npass = (cnt + 7u) >> 3;
  constexpr u32 PB = 4;
  bool drop = false;
  u32 t0 = 0;
  for (; npass - t0 >= PB; t0 += PB) sketch_passes<KIND, SK, PB>(K, S, B, cid, cnt, t0, last_off, sub, grp, drop);
  if (PB > 2u && npass - t0 >= 2u) {
    sketch_passes<KIND, SK, 2>(K, S, B, cid, cnt, t0, last_off, sub, grp, drop);
    t0 += 2u;
  }
  if (npass != t0) sketch_passes<KIND, SK, 1>(K, S, B, cid, cnt, t0, last_off, sub, grp, drop);
  return drop;
}

// eval_up_to_64 for rows that have sketches (same pieces per lane, same sums in the same order), with cnt >= 1:
// a lane's pieces lie at constant distances, and only those behind the first SKETCH_WHOLE can be missing (rows have
// 20 to 31 pieces at four per lane, 40 to 48, 49 to 56 and 57 to 63 at six, seven and eight).
template <int NCH>
constexpr int SKETCH_WHOLE = NCH == 4 ? 2 : NCH == 6 ? 5 : NCH - 1;

template <int KIND, int NCH, int PBX, class Query>
__device__ __forceinline__ void row_passes(const VecTable& T, const Query& Q, const u32* cid, u32 cnt, u32 t0, int sub,
                                           u32 grp, u32& result) {
  Piece<16> x[PBX][NCH];
#pragma unroll
  for (int tt = 0; tt < PBX; ++tt) {
    const u32 c = 8u * (t0 + tt) + grp;
    const char* row = T.base + ((u64)cid[c < cnt ? c : 0u] * T.row_bytes + (u32)sub * 16u);
#pragma unroll
    for (int u = 0; u < NCH; ++u)
      x[tt][u] = u < SKETCH_WHOLE<NCH> || (u32)sub + LPC * u < T.npieces ? load_piece<16>(row + u * 128) : zero_piece<16>();
  }
#pragma unroll
  for (int tt = 0; tt < PBX; ++tt) {
    const u32 dk = distance_key<KIND, 16, NCH>(Q, x[tt]);
    if ((u32)sub == t0 + tt) result = dk;
  }
}
template <int KIND, int NCH, class Query>
__device__ __forceinline__ u32 eval_rows(const VecTable& T, const Query& Q, const u32* cid, u32 cnt, int lane) {
  constexpr int PB = PassBatch<16, NCH>::value;
  const int sub = lane & (LPC - 1);
  const u32 grp = (u32)lane >> 3;
  const u32 npass = (cnt + 7u) >> 3;
  u32 result = 0, t0 = 0;
  for (; npass - t0 >= (u32)PB; t0 += PB) row_passes<KIND, NCH, PB>(T, Q, cid, cnt, t0, sub, grp, result);
  if constexpr (PB >= 4) {
    if (npass - t0 >= 2u) {
      row_passes<KIND, NCH, 2>(T, Q, cid, cnt, t0, sub, grp, result);
      t0 += 2u;
    }
  }
  if constexpr (PB >= 2) {
    if (npass != t0) row_passes<KIND, NCH, 1>(T, Q, cid, cnt, t0, sub, grp, result);
  }
  return result;
}

}  // namespace annmi
