// The alpha-prune scan of Sec. 4.1 as a wavefront-wide device routine, shared by step 1 and
// step 2 of BatchInsert.
//
// prune(p, C, R) walks C in order of (distance to p, id); a candidate is selected unless a point
// selected before it removes it (alpha * d(p*, c) <= d(p, c)); the walk ends with R selections.
// The wave follows that walk eight candidates at a time: each group of 8 lanes holds one of the
// next eight candidates in registers and measures it against every point selected so far (the
// same selected vector is broadcast from LDS to all groups) and against the other seven; the
// eight verdicts are then settled in order on bit masks.  Candidates behind the R-th selection
// are never looked at.  The vectors of the selected points (at most R) are kept in LDS when they
// fit, with their squared norms, so the only global traffic is one load per candidate, issued a
// block ahead.
#pragma once

#include <utility>

#include "ann_device.hpp"
#include "wave_sort.hpp"

namespace annmi {

// In-place ascending bitonic sort of n2 keys (a power of two >= 2) by one wave, every step a trip
// through LDS: for the sizes the register version below does not cover.
__device__ __forceinline__ void bitonic_sort_keys_lds(u64* a, u32 n2, int lane) {
  for (u32 k = 2; k <= n2; k <<= 1) {
    for (u32 j = k >> 1; j > 0; j >>= 1) {
      for (u32 t = lane; t < (n2 >> 1); t += 64) {
        const u32 i = 2u * t - (t & (j - 1u));
        const u32 l = i + j;
        const bool up = (i & k) == 0u;
        const u64 x = a[i], y = a[l];
        if ((x > y) == up) {
          a[i] = y;
          a[l] = x;
        }
      }
      __syncthreads();
    }
  }
}

// The same sort with the keys in registers (wave_sort.hpp), no barrier, no LDS round trip.
template <int KPL>
__device__ __forceinline__ void bitonic_sort_regs(u64* a, int lane) {
  u64 v[KPL];
#pragma unroll
  for (int q = 0; q < KPL; ++q) v[q] = a[64 * q + lane];
  BitonicStage<KPL, 2, false>::run(v);
#pragma unroll
  for (int q = 0; q < KPL; ++q) a[64 * q + lane] = v[q];
}

// In-place ascending sort of n2 keys in LDS (a power of two >= 64) by one wave; the keys must be
// visible to the wave when it is called and are visible to it on return.
__device__ __forceinline__ void bitonic_sort_keys(u64* a, u32 n2, int lane) {
  switch (n2) {
    case 64: bitonic_sort_regs<1>(a, lane); break;
    case 128: bitonic_sort_regs<2>(a, lane); break;
    case 256: bitonic_sort_regs<4>(a, lane); break;
    case 512: bitonic_sort_regs<8>(a, lane); break;
    default: bitonic_sort_keys_lds(a, n2, lane); return;
  }
  __syncthreads();
}

// LDS copy of the selected points' vectors
struct SelStage {
  unsigned char* vec;  // R rows of `stride` bytes, or null: read the vectors from device memory
  u32* xx;             // <x,x> of each selected point (integer kinds)
  u32 stride;
};

// Does a selected point remove candidate c?  Qc holds c's vector, dkey_pc = d(p, c).
template <int KIND, int VEC, int NCH>
__device__ __forceinline__ bool removed_by_selected(const VecTable& T, const SelStage& st,
                                                    const QueryRegs<KIND, VEC, NCH>& Qc, u32 dkey_pc,
                                                    const u32* out, u32 nout, const AlphaParam& al, int lane,
                                                    u32& pair_evals) {
  pair_evals += nout;
  if (st.vec != nullptr) {
    const int sub = lane & (LPC - 1);
    const u32 grp = (u32)lane >> 3;
    bool dom = false;
    const u32 npass = (nout + 7u) >> 3;
    for (u32 t = 0; t < npass; ++t) {
      const u32 idx = 8u * t + grp;
      const bool ok = idx < nout;
      const unsigned char* src = st.vec + (ok ? idx : 0u) * st.stride;
      Piece<VEC> x[NCH];
#pragma unroll
      for (int u = 0; u < NCH; ++u) {
        const u32 pc = sub + LPC * u;
        x[u] = pc < T.npieces ? load_piece<VEC>(reinterpret_cast<const char*>(src) + pc * VEC) : zero_piece<VEC>();
      }
      u32 dk;
      if constexpr (KindTraits<KIND>::is_int) {
        i32 qx = 0;
#pragma unroll
        for (int u = 0; u < NCH; ++u)
#pragma unroll
          for (int i = 0; i < VEC / 4; ++i) {
            if constexpr (KIND == K_U8)
              qx = (i32)__builtin_amdgcn_udot4(Qc.q[u].w[i], x[u].w[i], (u32)qx, false);
            else
              qx = __builtin_amdgcn_sdot4((i32)Qc.q[u].w[i], (i32)x[u].w[i], qx, false);
          }
        dk = dkey_from_int(Qc.qq + (i32)st.xx[ok ? idx : 0u] - 2 * group_sum(qx));
      } else {
        dk = distance_key<KIND, VEC, NCH>(Qc, x);
      }
      dom = dom || (ok && alpha_dominates<KIND>(al, dk, dkey_pc));
    }
    return ballot(dom) != 0;
  }
  for (u32 base = 0; base < nout; base += 64) {
    const u32 cnt = nout - base < 64u ? nout - base : 64u;
    const u32* ob = out + base;
    const u32 dk = eval_up_to_64<KIND, VEC, NCH>(T, Qc, [ob](u32 i) { return ob[i]; }, cnt, lane);
    const bool dom = cand_of_lane(lane) < cnt && alpha_dominates<KIND>(al, dk, dkey_pc);
    if (ballot(dom) != 0) return true;
  }
  return false;
}

template <int KIND, int VEC, int NCH>
__device__ __forceinline__ void stage_selected(const VecTable& T, const SelStage& st,
                                               const QueryRegs<KIND, VEC, NCH>& Qc, u32 slot, int lane) {
  if (st.vec == nullptr) return;
  if (lane < LPC) {
#pragma unroll
    for (int u = 0; u < NCH; ++u) {
      const u32 pc = lane + LPC * u;
      if (pc < T.npieces) {
        unsigned char* dst = st.vec + slot * st.stride + pc * VEC;
#pragma unroll
        for (int i = 0; i < VEC / 4; ++i) reinterpret_cast<u32*>(dst)[i] = Qc.q[u].w[i];
      }
    }
    if (lane == 0) st.xx[slot] = (u32)Qc.qq;
  }
}

// floor(d * 2^16 / a16) for 0 <= d < 2^31, 0 < a16 < 2^31, clamped to INT32_MAX: the largest D with
// alpha * D <= d
__device__ __forceinline__ i32 alpha_threshold(i32 d, i64 a16) {
  const u64 x = (u64)(u32)d << 16;
  u64 t = (u64)__builtin_floor((double)x / (double)a16);
  if (t * (u64)a16 > x)
    --t;
  else if ((t + 1) * (u64)a16 <= x)
    ++t;
  return t > 0x7FFFFFFFull ? 0x7FFFFFFF : (i32)t;
}

// is the distance between the group's candidate (in Qc) and the row pieces x at most thr?  xx = <x,x>
template <int KIND, int VEC, int NCH>
__device__ __forceinline__ bool removes_pieces(i32 thr, const QueryRegs<KIND, VEC, NCH>& Qc, const Piece<VEC> (&x)[NCH],
                                               i32 xx) {
  i32 qx = 0;
#pragma unroll
  for (int u = 0; u < NCH; ++u)
#pragma unroll
    for (int i = 0; i < VEC / 4; ++i) {
      if constexpr (KIND == K_U8)
        qx = (i32)__builtin_amdgcn_udot4(Qc.q[u].w[i], x[u].w[i], (u32)qx, false);
      else
        qx = __builtin_amdgcn_sdot4((i32)Qc.q[u].w[i], (i32)x[u].w[i], qx, false);
    }
  return Qc.qq + xx - 2 * group_sum(qx) <= thr;
}

// cand[0..m): keys (distance to p | id), ids distinct, p absent, SORTED ascending.
// Selected ids go to out[0..return) in selection order.  Byte rows of 257 to 512 bytes come here, and rows of up to
// 128 bytes that are no multiple of 32 where R is above 128 (mfma_prune_ok: copies of the selected rows beyond
// 24 KB of LDS); the walks on the matrix cores further down take the others.  blk: LDS for 8 rows of st.stride bytes
// plus 8 norms (used even when the selected vectors themselves are not staged).
template <int KIND, int VEC, int NCH>
__device__ __forceinline__ u32 prune_sorted(const VecTable& T, const SelStage& st, unsigned char* blk,
                                            const u64* cand, u32 m, u32 R, const AlphaParam& al, u32* out,
                                            int lane, u32& pair_evals) {
  const int sub = lane & (LPC - 1);
  const u32 grp = (u32)lane >> 3;
  u32* blkxx = reinterpret_cast<u32*>(blk + 8u * st.stride);
  u32 nout = 0;
  if (m == 0) return 0;
  const u64 k0 = grp < m ? cand[grp] : KEY_INF;
  u64 nkey = k0;
  QueryRegs<KIND, VEC, NCH> nxt =
      load_query_raw<KIND, VEC, NCH>(T.base + (u64)(grp < m ? key_id(k0) : 0u) * T.row_bytes, T.npieces, lane);
  for (u32 i0 = 0; i0 < m && nout < R; i0 += 8) {
    QueryRegs<KIND, VEC, NCH> cur = nxt;
    const u64 key = nkey;
    const bool valid = i0 + grp < m;
    query_finish<KIND, VEC, NCH>(cur);
    const i32 thr = alpha_threshold(valid ? int_from_dkey(key_dkey(key)) : 0, al.a16);
    const u32 nb = m - i0 < 8u ? m - i0 : 8u;

    // park the block's vectors in LDS for the tests among the eight
#pragma unroll
    for (int u = 0; u < NCH; ++u) {
      const u32 pc = sub + LPC * u;
      if (pc < T.npieces) {
        unsigned char* dst = blk + grp * st.stride + pc * VEC;
#pragma unroll
        for (int i = 0; i < VEC / 4; ++i) reinterpret_cast<u32*>(dst)[i] = cur.q[u].w[i];
      }
    }
    if (sub == 0) blkxx[grp] = (u32)cur.qq;

    // against everything selected before this block
    bool dom = false;
    if (st.vec != nullptr) {
      auto test = [&](u32 t) -> bool {
        const unsigned char* src = st.vec + t * st.stride;
        Piece<VEC> x[NCH];
#pragma unroll
        for (int u = 0; u < NCH; ++u) {
          const u32 pc = sub + LPC * u;
          x[u] = pc < T.npieces ? load_piece<VEC>(reinterpret_cast<const char*>(src) + pc * VEC) : zero_piece<VEC>();
        }
        return removes_pieces<KIND, VEC, NCH>(thr, cur, x, (i32)st.xx[t]);
      };
      // four selected points per trip, written out by hand (loops around cross-lane operations
      // are not unrolled for us), so that their LDS reads overlap
      u32 t = 0;
      for (; t + 4 <= nout; t += 4) {
        const bool r0 = test(t), r1 = test(t + 1), r2 = test(t + 2), r3 = test(t + 3);
        dom = dom | r0 | r1 | r2 | r3;
      }
      for (; t < nout; ++t) {
        const bool r = test(t);
        dom = dom | r;
      }
    } else {
      // the rows lie in device memory: several are requested before the first is tested.  One at a
      // time, each waited for its own trip through the cache.
      constexpr u32 AHEAD = NCH <= 2 ? 4 : 2;
      for (u32 t = 0; t < nout; t += AHEAD) {
        Piece<VEC> x[AHEAD][NCH];
#pragma unroll
        for (u32 q = 0; q < AHEAD; ++q) {  // (past the end: the last row again, which changes no verdict)
          const char* src = T.base + (u64)out[t + q < nout ? t + q : nout - 1u] * T.row_bytes;
#pragma unroll
          for (int u = 0; u < NCH; ++u) {
            const u32 pc = sub + LPC * u;
            x[q][u] = pc < T.npieces ? load_piece<VEC>(src + (u64)pc * VEC) : zero_piece<VEC>();
          }
        }
#pragma unroll
        for (u32 q = 0; q < AHEAD; ++q) {
          i32 xx = 0;
#pragma unroll
          for (int u = 0; u < NCH; ++u)
#pragma unroll
            for (int i = 0; i < VEC / 4; ++i) {
              if constexpr (KIND == K_U8)
                xx = (i32)__builtin_amdgcn_udot4(x[q][u].w[i], x[q][u].w[i], (u32)xx, false);
              else
                xx = __builtin_amdgcn_sdot4((i32)x[q][u].w[i], (i32)x[q][u].w[i], xx, false);
            }
          xx = group_sum(xx);
          const bool r = removes_pieces<KIND, VEC, NCH>(thr, cur, x[q], xx);
          dom = dom | r;
        }
      }
    }
    {  // the next block's vectors travel while this block is settled.  Not earlier: rows read from device
      // memory need the registers, and the tests against staged rows hide nothing that settling does not
      const u32 ci = i0 + 8u + grp;
      nkey = ci < m ? cand[ci] : KEY_INF;
      nxt = load_query_raw<KIND, VEC, NCH>(T.base + (u64)(ci < m ? key_id(nkey) : 0u) * T.row_bytes, T.npieces, lane);
    }
    pair_evals += nout * nb;
    const u64 dead_before = ballot(dom && valid);
    __syncthreads();

    // among the eight: bit 8g of by[t] says "candidate t of the block removes candidate g"
    u64 by[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      by[t] = 0;
      if ((u32)t < nb) {  // uniform
        const unsigned char* src = blk + t * st.stride;
        Piece<VEC> x[NCH];
#pragma unroll
        for (int u = 0; u < NCH; ++u) {
          const u32 pc = sub + LPC * u;
          x[u] = pc < T.npieces ? load_piece<VEC>(reinterpret_cast<const char*>(src) + pc * VEC) : zero_piece<VEC>();
        }
        const bool r = removes_pieces<KIND, VEC, NCH>(thr, cur, x, (i32)blkxx[t]);
        by[t] = ballot(r && valid && (u32)t < grp);
      }
    }
    pair_evals += nb * (nb - 1) / 2;

    // settle the eight in order
    u32 selmask = 0, nsel = 0;
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      if ((u32)g < nb && nout + nsel < R) {
        bool removed = (dead_before >> (8 * g)) & 1ull;
#pragma unroll
        for (int t = 0; t < g; ++t) removed = removed || (((selmask >> t) & 1u) && ((by[t] >> (8 * g)) & 1ull));
        if (!removed) {
          selmask |= 1u << g;
          ++nsel;
        }
      }
    }
    // commit the selected ones: ids, vectors and norms, in order
    if (valid && ((selmask >> grp) & 1u)) {
      const u32 slot = nout + (u32)__builtin_popcount(selmask & ((1u << grp) - 1u));
      if (sub == 0) out[slot] = key_id(key);
      if (st.vec != nullptr) {
#pragma unroll
        for (int u = 0; u < NCH; ++u) {
          const u32 pc = sub + LPC * u;
          if (pc < T.npieces) {
            unsigned char* dst = st.vec + slot * st.stride + pc * VEC;
#pragma unroll
            for (int i = 0; i < VEC / 4; ++i) reinterpret_cast<u32*>(dst)[i] = cur.q[u].w[i];
          }
        }
        if (sub == 0) st.xx[slot] = (u32)cur.qq;
      }
    }
    nout += nsel;
    __syncthreads();
  }
  return nout;
}

// ---------------------------------------------------------------------------------------------
// The same walk for u8/i8 rows of at most 256 bytes, 32 candidates at a time, with the pair
// distances taken on the matrix cores.
//
// For a block of 32 candidates two small matrix products decide everything: (selected so far) x
// (block) tells which candidates are removed by an earlier selection, and (block) x (block) which
// candidate would remove which later one.  Both are Gram-type products of int8 vectors (u8 data
// is shifted by -128; distances do not change), exact in int32, computed with
// v_mfma_i32_32x32x32_i8 from LDS copies of the vectors: D(i,j) = |x_i|^2 + |x_j|^2 - 2<x_i,x_j>,
// and "i removes j" is D(i,j) <= floor(d(p,j) * 2^16 / a16).  The 32 verdicts are then settled in
// order on bit masks.  Rows of 129 to 256 bytes (300,000 uint8 points of 200, R = 64, L = 128): build 64.4 ->
// 36.7 ms against the walk above; of 500,000 such points, step 1's prune 31.5 -> 7.6 ms, the re-prunes 41.2 -> 19.7.
// ---------------------------------------------------------------------------------------------
typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef int v16i_t __attribute__((ext_vector_type(16)));

// bytes between staged rows (128 or 256, and 16 that spread the LDS banks)
__host__ __device__ constexpr u32 mm_stride(u32 row_bytes) { return row_bytes <= 128u ? 144u : 272u; }
constexpr u32 MM_BLOCK = 32;  // candidates per block

template <int KIND, int VEC, int NCH>
struct MfmaPruneOk {
  static constexpr bool value = KindTraits<KIND>::is_int && (8 * NCH * VEC <= 256);
  static constexpr bool always = value && NCH == 2;  // at every R: the walk above is not compiled
};

// LDS areas of the matrix-core walk (all 16-byte aligned)
struct MfmaLds {
  unsigned char* sel;  // roundup(R, 32) rows of mm_stride bytes: vectors of the selected points,
                       // or null: the matrix operand is loaded straight from the vectors in device
                       // memory (more waves per CU): rows of whole multiples of 32 bytes, and all rows
                       // above 128 bytes, whose copies would leave room for six waves
  u32* selnorm;        // roundup(R, 32): their squared norms (shifted vectors)
  unsigned char* blk;  // 32 rows: the current block of candidates
  u32* cnorm;          // 32
  i32* cthr;           // 32: removal thresholds of the block's candidates
  u32* cid;            // 32
};
__host__ __device__ constexpr u32 mfma_rows(u32 R) { return (R + 31u) & ~31u; }
__host__ __device__ constexpr bool mfma_sel_in_lds(u32 row_bytes) { return row_bytes <= 128u && (row_bytes % 32u) != 0u; }
__host__ __device__ constexpr u32 mfma_lds_bytes(u32 R, u32 row_bytes) {
  return (mfma_sel_in_lds(row_bytes) ? mfma_rows(R) * mm_stride(row_bytes) : 0u) + mfma_rows(R) * 4u +
         MM_BLOCK * mm_stride(row_bytes) + 3u * MM_BLOCK * 4u;
}
constexpr u32 MFMA_LDS_MAX = 24576;  // beyond, the walk leaves room for too few waves
static_assert(mfma_lds_bytes(512, 256) <= MFMA_LDS_MAX, "rows above 128 bytes have no other walk (MfmaPruneOk::always)");
__device__ __forceinline__ MfmaLds mfma_lds_carve(unsigned char* base, u32 R, u32 row_bytes) {
  MfmaLds M;
  const bool in_lds = mfma_sel_in_lds(row_bytes);
  M.sel = in_lds ? base : nullptr;
  M.blk = base + (in_lds ? mfma_rows(R) * mm_stride(row_bytes) : 0u);
  M.selnorm = reinterpret_cast<u32*>(M.blk + MM_BLOCK * mm_stride(row_bytes));
  M.cnorm = M.selnorm + mfma_rows(R);
  M.cthr = reinterpret_cast<i32*>(M.cnorm + MM_BLOCK);
  M.cid = reinterpret_cast<u32*>(M.cthr + MM_BLOCK);
  return M;
}

template <int R_>
__device__ __forceinline__ void mm_block_rows(const v16i_t& acc, const uint4 (&n4)[4], i32 ncol, i32 tcol, u32& by) {
  // accumulator register R_ of lane l is entry (row 8*(R_/4) + 4*(l/32) + R_%4, column l%32)
  constexpr int mlo = 8 * (R_ / 4) + (R_ % 4);
  const u32 nrow = (R_ % 4) == 0 ? n4[R_ / 4].x : (R_ % 4) == 1 ? n4[R_ / 4].y : (R_ % 4) == 2 ? n4[R_ / 4].z : n4[R_ / 4].w;
  const i32 D = (i32)nrow + ncol - 2 * acc[R_];
  const u64 bm = ballot(D <= tcol);
  by = writelane_pair<mlo, mlo + 4>(by, bm);
}
template <int... Rs>
__device__ __forceinline__ void mm_block_rows_all(const v16i_t& acc, const uint4 (&n4)[4], i32 ncol, i32 tcol, u32& by,
                                                  std::integer_sequence<int, Rs...>) {
  (mm_block_rows<Rs>(acc, n4, ncol, tcol, by), ...);
}

template <int KIND, int VEC, int NCH>
__device__ __forceinline__ u32 prune_sorted_mfma(const VecTable& T, const MfmaLds& M, const u64* cand, u32 m, u32 R,
                                                 i64 a16, u32* out, int lane, u32& pair_evals) {
  const int sub = lane & (LPC - 1);
  const u32 grp = (u32)lane >> 3;
  const u32 half = (u32)lane >> 5;
  const u32 col = (u32)lane & 31u;
  const u32 flip = KIND == K_U8 ? 0x80808080u : 0u;
  constexpr u32 KS = 4u * NCH, MM_STRIDE = mm_stride(128u * NCH);
  const u32 ksteps = (T.row_bytes + 31u) / 32u;  // <= KS
  u32 nout = 0;
  if (m == 0) return 0;

  Piece<VEC> nx[4][NCH];  // the next block's vectors, 4 passes of 8 candidates
  auto issue = [&](u32 i0) {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const u32 c = i0 + 8u * p + grp;
      const bool ok = c < m;
      const u32 id = ok ? key_id(cand[c]) : 0u;
      const char* src = T.base + (u64)id * T.row_bytes;
#pragma unroll
      for (int u = 0; u < NCH; ++u) {
        const u32 pc = sub + LPC * u;
        nx[p][u] = (ok && pc < T.npieces) ? load_piece<VEC>(src + (u64)pc * VEC) : zero_piece<VEC>();
      }
    }
  };
  issue(0);

  for (u32 i0 = 0; i0 < m && nout < R; i0 += MM_BLOCK) {
    const u32 nb = m - i0 < MM_BLOCK ? m - i0 : MM_BLOCK;
    // park the block in LDS (as int8), take the norms
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const u32 c = 8u * p + grp;
      const bool ok = c < nb;
      i32 nn = 0;
#pragma unroll
      for (int u = 0; u < NCH; ++u) {
        const u32 pc = sub + LPC * u;
#pragma unroll
        for (int i = 0; i < VEC / 4; ++i) {
          const u32 wv = (ok && pc < T.npieces) ? (nx[p][u].w[i] ^ flip) : 0u;
          nn = __builtin_amdgcn_sdot4((i32)wv, (i32)wv, nn, false);
          *reinterpret_cast<u32*>(M.blk + c * MM_STRIDE + pc * VEC + 4 * i) = wv;
        }
      }
      nn = group_sum(nn);
      if (sub == 0) M.cnorm[c] = (u32)nn;
    }
    if (lane < (int)MM_BLOCK) {
      const bool ok = (u32)lane < nb;
      const u64 key = ok ? cand[i0 + lane] : KEY_INF;
      M.cthr[lane] = ok ? alpha_threshold(int_from_dkey(key_dkey(key)), a16) : -1;
      M.cid[lane] = key_id(key);
    }
    if (i0 + MM_BLOCK < m) issue(i0 + MM_BLOCK);  // travels while this block is settled
    __syncthreads();

    // column operand: candidate `col`, this lane's 16 bytes of every k-step
    v4i_t bv[KS];
#pragma unroll
    for (u32 ks = 0; ks < KS; ++ks) {
      const v4i_t v =
          *reinterpret_cast<const v4i_t*>(M.blk + col * MM_STRIDE + 32u * (ks < ksteps ? ks : ksteps - 1u) + 16u * half);
      bv[ks] = ks < ksteps ? v : v4i_t{0, 0, 0, 0};
    }
    const i32 ncol = (i32)M.cnorm[col];
    const i32 tcol = M.cthr[col];

    // removed by a point selected before this block?  The row operand of each 32-point slice is
    // requested in one go, and the next slice's before this one's products are taken, so that a
    // block costs one trip to memory rather than one per instruction.
    bool rem = false;
    const u32 kclamp = ksteps - 1u;
    const u32 aflip = M.sel != nullptr ? 0u : flip;
    auto load_slice = [&](u32 s0, v4i_t (&av)[KS]) {
      if (M.sel != nullptr) {
#pragma unroll
        for (u32 ks = 0; ks < KS; ++ks)
          av[ks] = *reinterpret_cast<const v4i_t*>(M.sel + (s0 + col) * MM_STRIDE + 32u * (ks < kclamp ? ks : kclamp) +
                                                   16u * half);
      } else {
        const u32 sid = s0 + col < nout ? out[s0 + col] : out[0];
        const char* src = T.base + (u64)sid * T.row_bytes + 16u * half;
#pragma unroll
        for (u32 ks = 0; ks < KS; ++ks) {
          // (a row's odd last piece: its other half meets zeros in the block)
          const u32 at = 32u * (ks < kclamp ? ks : kclamp);
          av[ks] = *reinterpret_cast<const v4i_t*>(NCH == 1 || at + 16u * half < T.row_bytes ? src + at : src);
        }
      }
    };
    // (rows above 128 bytes: the registers of a second slice would cost a wave per SIMD)
    constexpr bool AHEAD = NCH == 1;
    v4i_t av[KS];
    if (AHEAD && nout > 0) load_slice(0, av);
    for (u32 s0 = 0; s0 < nout; s0 += 32) {
      if (!AHEAD) load_slice(s0, av);
      v4i_t cur[KS];
#pragma unroll
      for (u32 ks = 0; ks < KS; ++ks)
        cur[ks] = ks < ksteps ? (av[ks] ^ (int)aflip) : v4i_t{0, 0, 0, 0};  // device memory holds u8
      if (AHEAD && s0 + 32 < nout) load_slice(s0 + 32, av);
      v16i_t acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
      for (u32 ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(cur[ks], bv[ks], acc, 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const u32 sb = s0 + 8u * q + 4u * half;
        const uint4 n4 = *reinterpret_cast<const uint4*>(M.selnorm + sb);
        rem = rem | (sb + 0 < nout && (i32)n4.x + ncol - 2 * acc[4 * q + 0] <= tcol);
        rem = rem | (sb + 1 < nout && (i32)n4.y + ncol - 2 * acc[4 * q + 1] <= tcol);
        rem = rem | (sb + 2 < nout && (i32)n4.z + ncol - 2 * acc[4 * q + 2] <= tcol);
        rem = rem | (sb + 3 < nout && (i32)n4.w + ncol - 2 * acc[4 * q + 3] <= tcol);
      }
    }
    const u64 rm = ballot(rem);
    const u32 removed_old = (u32)rm | (u32)(rm >> 32);

    // which candidate of the block would remove which: lane t ends up with the mask of row t
    u32 by = 0;
    {
      v16i_t acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
      for (u32 ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(bv[ks], bv[ks], acc, 0, 0, 0);
      uint4 n4[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) n4[q] = *reinterpret_cast<const uint4*>(M.cnorm + 8u * q + 4u * half);
      mm_block_rows_all(acc, n4, ncol, tcol, by, std::make_integer_sequence<int, 16>{});
    }
    pair_evals += nb * nout + nb * (nb - 1) / 2;

    // settle the block in order
    u32 alive = (nb >= 32u ? ~0u : ((1u << nb) - 1u)) & ~removed_old;
    u32 selmask = 0, nsel = 0;
    while (alive != 0 && nout + nsel < R) {
      const int t = __builtin_ctz(alive);
      selmask |= 1u << t;
      ++nsel;
      alive &= ~readlane_u32(by, t);
      alive &= ~(1u << t);
    }
    // commit: ids, norms and vectors of the selected candidates, in order
    if (lane < (int)MM_BLOCK && ((selmask >> lane) & 1u)) {
      const u32 slot = nout + (u32)__builtin_popcount(selmask & ((1u << lane) - 1u));
      out[slot] = M.cid[lane];
      M.selnorm[slot] = M.cnorm[lane];
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const u32 t = 8u * p + grp;
      if (M.sel != nullptr && ((selmask >> t) & 1u)) {
        const u32 slot = nout + (u32)__builtin_popcount(selmask & ((1u << t) - 1u));
        *reinterpret_cast<uint4*>(M.sel + slot * MM_STRIDE + 16u * sub) =
            *reinterpret_cast<const uint4*>(M.blk + t * MM_STRIDE + 16u * sub);
      }
    }
    nout += nsel;
    __syncthreads();
  }
  return nout;
}

// ---------------------------------------------------------------------------------------------
// The same walk for float rows, 16 candidates at a time, with the inner products taken on the matrix
// cores (v_mfma_f32_16x16x1_4b_f32: four independent 16 x 16 outer products, one fp32 fma per entry).
//
// A block of 16 candidates lies in registers as the matrix operand: lane (blk, r) = (lane / 16, lane %
// 16) holds the 16-byte pieces 8 u + 4 h + blk of candidate r (h = 0, 1; u < NCH).  Piece p is summed by
// lane p % 8 of a group in distance_key, so one instruction takes the same element of four of those
// eight partial sums, and an entry's eight sums, added up in the order of group_sum, are bit for bit the
// inner product that distance_key computes.
//
//  - Inner product: the verdicts are those of the vector path.
//  - Squared L2: distance_key sums (a - b)^2, which is no matrix product.  With a' = a - p the products
//    give S = |a'|^2 + |b'|^2 - 2 <a', b'>, and |S - D| <= E for the D that distance_key computes (see
//    GRAM_ERR): S + E and S - E decide nearly every pair, and the rest is measured by distance_key's own
//    sum.  Both give the vector path's verdicts.  Moving the origin to p makes E small against the
//    distances of p's neighbourhood wherever the data lies.
//
// What bounds it: the matrix cores (NCH * 8 instructions of 32 cycles for 256 pairs); the vector path is
// bound by the first-level cache, which hands it a piece of a selected row eight times over for eight pairs.
// Per launch of 20,000 points of 200 floats, R = 64, L = 128, inner product: 850 -> 405 us, the re-prunes
// beside each other 525 -> 142; builds: a million such points 311 -> 264 ms; squared L2, 100,000 points of 200
// floats 139 -> 82 ms, of 96 floats (R = 48, L = 96) 37.4 -> 26.3, of 48 (R = 32, L = 64) 18.0 -> 15.6.
// ---------------------------------------------------------------------------------------------
typedef float v16f_t __attribute__((ext_vector_type(16)));

// |S - D| <= E = GRAM_ERR * (|a'|^2 + |b'|^2) + GRAM_TINY, both norms as computed.  With u = 2^-24, rows
// of at most 256 elements and N = |a - p|^2 + |b - p|^2: rounding a' and b' moves the distance by at most
// 4 u N; the norms (chains of 64 fmas, two sums) are off by 66 u N; the inner product (chains of 32, three
// sums) by 35 u |a'||b'|, twice of which is 35 u N; putting S together costs 3 u N; and D itself, 38 u of a
// distance of at most 2 N, 76 u N.  In all 184 u N, where GRAM_ERR is 256 u: the rest covers the roundings
// of S + E and S - E and of the computed norms.  GRAM_TINY covers products and elements that underflow.
constexpr float GRAM_ERR = 0x1p-16f, GRAM_TINY = 1e-35f;

template <int KIND, int VEC, int NCH>
struct F32PruneOk {
  static constexpr bool value = !KindTraits<KIND>::is_int && VEC == 16 && NCH <= 8;
};

// Waves per SIMD of the prune kernel: what its walk's registers leave room for.  Byte rows above 128 bytes
// hold a block, the next one and a slice of selected rows, 32 registers each; float rows a block of
// candidates and a tile of selected rows, 8 * NCH registers each, beside 16 of products.  Squared L2 with seven
// pieces lacks five registers for three waves; they are put aside once per block of candidates, which costs
// less than the third wave brings (prune of 300,000 points of 200 floats, R = 64: 18.8 ms, by two waves 19.3; of
// a million at R = 32 20.8 and 22.1).
template <int KIND, int VEC, int NCH>
struct PruneWaves {
  static constexpr int value = F32PruneOk<KIND, VEC, NCH>::value ? (NCH <= 4 ? 4 : NCH <= 7 ? 3 : 2)
                               : MfmaPruneOk<KIND, VEC, NCH>::value && NCH == 2 ? 2 : 4;
};

// LDS of the walk: p's row, zero-padded to 8 * NCH pieces, the block's norms, the selected points' norms
struct F32Lds {
  float4* p;
  float* cnorm;    // 16
  float* selnorm;  // R
};
__host__ __device__ inline u32 f32_lds_bytes(u32 R, u32 npieces) {
  return ((npieces + 7u) & ~7u) * 16u + 64u + ((R * 4u + 15u) & ~15u) + ((R * 4u + 15u) & ~15u);
}
// `base` is 16-byte aligned; `out` gets the first R words
__device__ __forceinline__ F32Lds f32_lds_carve(unsigned char* base, u32 R, u32*& out) {
  F32Lds M;
  const u32 words = (R * 4u + 15u) & ~15u;
  out = reinterpret_cast<u32*>(base);
  M.selnorm = reinterpret_cast<float*>(base + words);
  M.cnorm = reinterpret_cast<float*>(base + 2u * words);
  M.p = reinterpret_cast<float4*>(base + 2u * words + 64u);
  return M;
}

template <int NCH>
struct F32Operand {
  float4 x[2][NCH];
};

// a row's pieces of this lane; L2: less p's
template <int KIND, int NCH>
__device__ __forceinline__ void f32_load(F32Operand<NCH>& o, const char* row, u32 npieces, u32 blk) {
#pragma unroll
  for (int u = 0; u < NCH; ++u)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const u32 pc = 8u * u + 4u * h + blk;
      o.x[h][u] = pc < npieces ? *reinterpret_cast<const float4*>(row + (u64)pc * 16u) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
}
template <int KIND, int NCH>
__device__ __forceinline__ void f32_centre(F32Operand<NCH>& o, const F32Lds& M, u32 npieces, u32 blk) {
  if constexpr (KIND == K_F32_L2) {
#pragma unroll
    for (int u = 0; u < NCH; ++u)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (8u * u + 4u * h < npieces) {  // (uniform; the LDS copy of p has zeros up to a multiple of 8 pieces)
          const float4 p = M.p[8u * u + 4u * h + blk];
          o.x[h][u].x -= p.x;
          o.x[h][u].y -= p.y;
          o.x[h][u].z -= p.z;
          o.x[h][u].w -= p.w;
        }
      }
  }
}

// inner products of rows a (4 * (lane / 16) + v) and columns b (lane % 16)
template <int NCH>
__device__ __forceinline__ void f32_products(const F32Operand<NCH>& a, const F32Operand<NCH>& b, u32 npieces,
                                             float (&dot)[4]) {
  // one half of the partial sums after the other: the second half's pieces may still be on their way
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    v16f_t acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int u = 0; u < NCH; ++u) {
      // (an instance serves rows that leave its last pieces empty: a chain of them adds zeros)
      if (u + 2 < NCH || 8u * u + 4u * h < npieces) {
        acc = __builtin_amdgcn_mfma_f32_16x16x1f32(a.x[h][u].x, b.x[h][u].x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x1f32(a.x[h][u].y, b.x[h][u].y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x1f32(a.x[h][u].z, b.x[h][u].z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x1f32(a.x[h][u].w, b.x[h][u].w, acc, 0, 0, 0);
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float half = (acc[v] + acc[4 + v]) + (acc[8 + v] + acc[12 + v]);
      dot[v] = h == 0 ? half : dot[v] + half;
    }
  }
}

// What the products say of one pair: +1 the first removes the second, -1 it does not, 0 to be measured.
// na, nb: squared norms (L2); dpc = d(p, second).
template <int KIND>
__device__ __forceinline__ int f32_verdict(float dot, float na, float nb, float af, float dpc) {
  if constexpr (KIND == K_F32_IP) {
    return af * -dot <= dpc ? 1 : -1;
  } else {
    const float n = na + nb;
    const float S = __builtin_fmaf(-2.0f, dot, n), E = __builtin_fmaf(GRAM_ERR, n, GRAM_TINY);
    const float lo = S - E, hi = S + E;
    // (a NaN anywhere, as from an overflow, fails every comparison: measured)
    if (lo <= hi && af * hi <= dpc) return 1;
    return af * lo > dpc ? -1 : 0;
  }
}

// Which of the candidates first[j], j in `mask`, row `sel` removes, each measured with distance_key's sum.
__device__ __forceinline__ u32 f32_measured(const VecTable& T, u32 sel, const u64* first, u32 mask, float af, int lane) {
  const u32 sub = (u32)lane & 7u, grp = (u32)lane >> 3;
  u32 removed = 0;
  while (mask) {
    u32 rest = mask;
    for (u32 k = 0; k < grp; ++k) rest &= rest - 1u;  // this group's candidate: the grp-th of the mask
    const bool ok = rest != 0;
    const u32 j = ok ? (u32)__builtin_ctz(rest) : 0u;
    const u64 key = first[j];
    const char* x = T.base + (u64)sel * T.row_bytes;
    const char* y = T.base + (u64)(ok ? key_id(key) : sel) * T.row_bytes;
    float d = 0.0f;  // (rare: not worth the registers that all pieces at once would take)
#pragma unroll 1
    for (u32 pc = sub; pc < T.npieces; pc += 8u) {
      const float4 f = *reinterpret_cast<const float4*>(x + (u64)pc * 16u), g = *reinterpret_cast<const float4*>(y + (u64)pc * 16u);
      const float e0 = f.x - g.x, e1 = f.y - g.y, e2 = f.z - g.z, e3 = f.w - g.w;
      d = __builtin_fmaf(e3, e3, __builtin_fmaf(e2, e2, __builtin_fmaf(e1, e1, __builtin_fmaf(e0, e0, d))));
    }
    d = group_sum(d);
    const u64 hit = ballot(ok && af * d <= float_from_dkey(key_dkey(key)));
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      if (mask) {  // uniform
        if ((hit >> (8 * g)) & 1ull) removed |= mask & (0u - mask);
        mask &= mask - 1u;
      }
    }
  }
  return removed;
}

// prow: p's row (L2).  The rest as prune_sorted.
template <int KIND, int VEC, int NCH>
__device__ __forceinline__ u32 prune_sorted_f32(const VecTable& T, const F32Lds& M, const char* prow, const u64* cand, u32 m,
                                                u32 R, float af, u32* out, int lane, u32& pair_evals) {
  constexpr bool L2 = KIND == K_F32_L2;
  const u32 blk = (u32)lane >> 4, r = (u32)lane & 15u;
  u32 nout = 0;
  if (m == 0) return 0;
  if constexpr (L2) {
    const u32 np8 = (T.npieces + 7u) & ~7u;  // (at most 64)
    if ((u32)lane < np8)
      M.p[lane] = (u32)lane < T.npieces ? reinterpret_cast<const float4*>(prow)[lane] : make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();
  }
  for (u32 i0 = 0; i0 < m && nout < R; i0 += 16) {
    const u32 nb = m - i0 < 16u ? m - i0 : 16u;
    const u64* first = cand + i0;
    const u64 ckey = first[r < nb ? r : 0u];
    const float dpc = float_from_dkey(key_dkey(ckey));  // of column r
    F32Operand<NCH> b;
    f32_load<KIND, NCH>(b, T.base + (u64)key_id(ckey) * T.row_bytes, T.npieces, blk);
    f32_centre<KIND, NCH>(b, M, T.npieces, blk);
    float ncol = 0.0f;
    if constexpr (L2) {
#pragma unroll
      for (int u = 0; u < NCH; ++u)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const float4 x = b.x[h][u];
          ncol = __builtin_fmaf(x.x, x.x, ncol);
          ncol = __builtin_fmaf(x.y, x.y, ncol);
          ncol = __builtin_fmaf(x.z, x.z, ncol);
          ncol = __builtin_fmaf(x.w, x.w, ncol);
        }
      ncol += __shfl_xor(ncol, 16, 64);
      ncol += __shfl_xor(ncol, 32, 64);
      if (lane < 16) M.cnorm[lane] = ncol;
    }

    // removed by a point selected before this block?
    u32 removed = 0;  // bit j: candidate j of the block
    for (u32 s0 = 0; s0 < nout; s0 += 16) {
      F32Operand<NCH> a;  // (past the end: the last row again, which changes no verdict)
      f32_load<KIND, NCH>(a, T.base + (u64)out[s0 + r < nout ? s0 + r : nout - 1u] * T.row_bytes, T.npieces, blk);
      f32_centre<KIND, NCH>(a, M, T.npieces, blk);
      float dot[4];
      f32_products<NCH>(a, b, T.npieces, dot);
      bool rem = false;
      u32 open = 0;  // rows whose pair with this lane's column has to be measured
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const u32 row = s0 + 4u * blk + v;
        const float nrow = L2 ? M.selnorm[row < nout ? row : nout - 1u] : 0.0f;
        const int verdict = f32_verdict<KIND>(dot[v], nrow, ncol, af, dpc);
        rem = rem | (verdict > 0);
        if (L2 && verdict == 0 && row < nout) open |= 1u << v;
      }
      const u64 rm = ballot(rem);
      removed |= (u32)(rm | (rm >> 16) | (rm >> 32) | (rm >> 48)) & 0xFFFFu;
      if constexpr (L2) {
        if (ballot(open != 0)) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const u64 om = ballot((open >> v) & 1u);
            for (u32 q = 0; q < 4; ++q) {
              const u32 mask = (u32)(om >> (16u * q)) & 0xFFFFu & ~removed & ((1u << nb) - 1u);
              if (mask) removed |= f32_measured(T, out[s0 + 4u * q + v], first, mask, af, lane);
            }
          }
        }
      }
    }

    // which candidate of the block would remove which: rows[v] holds rows v, 4 + v, 8 + v, 12 + v, 16 bits each
    u64 rows[4], opens[4];
    {
      float dot[4];
      f32_products<NCH>(b, b, T.npieces, dot);
      __syncthreads();  // (the norms)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float nrow = L2 ? M.cnorm[4u * blk + v] : 0.0f;
        const int verdict = f32_verdict<KIND>(dot[v], nrow, ncol, af, dpc);
        rows[v] = ballot(verdict > 0);
        opens[v] = L2 ? ballot(verdict == 0) : 0ull;
      }
    }
    pair_evals += nb * nout + nb * (nb - 1) / 2;

    // settle the block in order
    u32 alive = ((1u << nb) - 1u) & ~removed;
    u32 selmask = 0, nsel = 0;
    while (alive != 0 && nout + nsel < R) {
      const u32 t = (u32)__builtin_ctz(alive);
      selmask |= 1u << t;
      ++nsel;
      alive &= ~(1u << t);
      const u32 v = t & 3u, sh = 16u * (t >> 2);
      const u64 row = v == 0 ? rows[0] : v == 1 ? rows[1] : v == 2 ? rows[2] : rows[3];
      alive &= ~((u32)(row >> sh) & 0xFFFFu);
      if constexpr (L2) {
        const u64 ow = v == 0 ? opens[0] : v == 1 ? opens[1] : v == 2 ? opens[2] : opens[3];
        const u32 mask = (u32)(ow >> sh) & alive;
        if (mask) alive &= ~f32_measured(T, key_id(first[t]), first, mask, af, lane);
      }
    }
    // commit: ids and norms of the selected candidates, in order
    if (lane < 16 && ((selmask >> lane) & 1u)) {
      const u32 slot = nout + (u32)__builtin_popcount(selmask & ((1u << lane) - 1u));
      out[slot] = key_id(ckey);
      if constexpr (L2) M.selnorm[slot] = ncol;
    }
    nout += nsel;
    __syncthreads();
  }
  return nout;
}

// The same walk over an UNSORTED key array that may live in device memory (very long lists):
// the next candidate is found by a minimum search, and taken out by overwriting it.
template <int KIND, int VEC, int NCH>
__device__ __forceinline__ u32 prune_unsorted(const VecTable& T, const SelStage& st, u64* cand, u32 m, u32 R,
                                              const AlphaParam& al, u32* out, int lane, u32& pair_evals) {
  u32 nout = 0;
  for (u32 step = 0; step < m && nout < R; ++step) {
    u64 best = KEY_INF;
    u32 besti = 0;
    for (u32 i = lane; i < m; i += 64) {
      const u64 k = cand[i];
      if (k < best) {
        best = k;
        besti = i;
      }
    }
    const u64 key = wave_min_u64(best);
    if (key == KEY_INF) break;
    if (best == key) cand[besti] = KEY_INF;  // keys are distinct: exactly one lane
    const QueryRegs<KIND, VEC, NCH> cur =
        load_query<KIND, VEC, NCH>(T.base + (u64)key_id(key) * T.row_bytes, T.npieces, lane);
    if (!removed_by_selected<KIND, VEC, NCH>(T, st, cur, key_dkey(key), out, nout, al, lane, pair_evals)) {
      __syncthreads();
      if (lane == 0) out[nout] = key_id(key);
      stage_selected<KIND, VEC, NCH>(T, st, cur, nout, lane);
      ++nout;
    }
    __syncthreads();
  }
  return nout;
}

// LDS bytes of a stage for R selected rows, or 0 if they would not fit the budget
__host__ __device__ inline u32 stage_stride(u32 row_bytes) { return (row_bytes + 15u) & ~15u; }
__host__ inline u32 stage_bytes(u32 R, u32 row_bytes, u32 budget) {
  const u64 need = (u64)R * stage_stride(row_bytes);
  return need <= budget ? (u32)need : 0u;
}

}  // namespace annmi
