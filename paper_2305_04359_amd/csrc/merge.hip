// Step 2 of BatchInsert (Alg. 3 of the paper): for every existing point b that was chosen by
// batch points, N_out(b) <- N_out(b) U N, and prune(b, N_out(b), R) if that exceeds R.
//
// The edge keys, grouped by destination, are cut into segments of equal destination by a planning kernel, which
// appends directly where the row has room and otherwise files the segment under one of three
// kinds of re-prune (one wavefront per row), each served by a kernel of its own, in smaller batches of
// byte rows two or all three of them by one (merge_launches):
//
//   fast     the row still starts with the output of its last prune (its "clean prefix": sorted
//            by distance to b and free of pairs where one removes the other, which is what prune
//            guarantees of what it keeps) and only a few entries are new.  Only pairs with a new
//            entry can change anything, so the wave measures every candidate against b and
//            against the new entries in one sweep and replays the scan on bit masks.
//   gram     u8/i8 rows (up to 256 bytes) of at most 96 candidates: all pair distances from the int8 Gram matrix
//            on the matrix cores (exact), then the scan on bit masks.
//   generic  everything else: the wave-wide scan of prune_device.hpp, candidates in LDS or, for
//            very long lists, in a spill arena in device memory.  Float rows of at most 128 candidates,
//            up to 16 of them new, form only the pairs with a new entry, on the fp32 matrix cores.
//
// Every path computes exactly prune(b, U, R) with U = old row followed by the new sources in
// batch order; they differ only in which distances they have to take.
#include <utility>

#include "ann_device.hpp"
#include "ann_internal.hpp"
#include "ann_dispatch.hpp"
#include "plan_device.hpp"
#include "prune_device.hpp"

namespace annmi {

// ---------------------------------------------------------------------------------------------
// planning: one thread per edge key; the first key of each segment does the work
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void plan_kernel(MergeArgs a) {
  __shared__ u32 cnt_lds[4];
  __shared__ u32 base_lds[4];
  __shared__ u32 stat_lds[2];  // appends, appended edges
  if (threadIdx.x < 4) cnt_lds[threadIdx.x] = 0;
  if (threadIdx.x < 2) stat_lds[threadIdx.x] = 0;
  __syncthreads();

  const u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x;
  int kind = -1;
  u32 slot = 0, cnt = 0, b = 0, m = 0;
  if (i < a.nkeys) {
    b = (u32)(a.keys[i] >> 32);
    const bool head = b != NONE_ID && (i == 0 || (u32)(a.keys[i - 1] >> 32) != b);
    if (head) {
      // length of the segment: gallop, then bisect (keys are sorted by destination)
      u64 lo = i, step = 1;
      while (i + step < a.nkeys && (u32)(a.keys[i + step] >> 32) == b) {
        lo = i + step;
        step <<= 1;
      }
      u64 hi = i + step < a.nkeys ? i + step : a.nkeys;
      while (hi - lo > 1) {
        const u64 mid = (lo + hi) >> 1;
        if ((u32)(a.keys[mid] >> 32) == b)
          lo = mid;
        else
          hi = mid;
      }
      cnt = (u32)(hi - i);
      m = a.meta[b];
      kind = plan_segment(a, b, m, cnt, stat_lds, [&](u32 j) { return (u32)(a.keys[i + j] & 0xFFFFFFFFull); });
      if (kind >= 0) slot = atomicAdd(&cnt_lds[kind], 1u);
    }
  }
  __syncthreads();
  plan_reserve(a, cnt_lds, base_lds, stat_lds);
  __syncthreads();
  if (kind >= 0) plan_file(a, kind, base_lds[kind] + slot, i, cnt, b, m);
}

// ---------------------------------------------------------------------------------------------
// Grouping and planning of a batch in one: the keys come dealt into buckets by the low bits of their
// destination (group_split), one workgroup per bucket groups its keys by the other bits, at most GROUP_HIGH_BITS, and plans
// the segments, whose lengths it has just counted.  Equal destinations need to stand together, in the order of the batch;
// the order of the groups has no influence on any result.  It replaces the second pass of the radix sort
// (three launches) and the planning launch: a build of a million points at R = 64 79.3 ->
// 76.7 ms, batches of 3,000 points 420 -> 403 us each.
// Four waves, each over its own quarter of the bucket, rank as the radix sort does (sort.hip), with counters of each wave's own.
// A bucket that holds most of a batch keeps its four waves longer than the radix sort's tiles did: 30,000 edges to one vertex of
// a million 4.5 -> 4.7 ms, of which that vertex's re-prune is nearly all (four rows requested ahead: no change).  Where
// crowded vertices are part of a build it pays all the same: 200,000 points on a shell about sixteen others,
// 50,000 edges to one of them, 20.6 -> 18.9 ms.
// ---------------------------------------------------------------------------------------------
constexpr u32 GROUP_WAVES = 4;
__global__ __launch_bounds__(64 * GROUP_WAVES) void group_plan_kernel(MergeArgs a, const u64* in, u64* out, const u32* bucket_total,
                                                                      u32 low_bits, u32 high_bits) {
  extern __shared__ u32 count[];  // GROUP_WAVES x 2^high_bits, then 2^high_bits: where a segment's filing stands
  __shared__ u32 cnt_lds[4], base_lds[4], stat_lds[2], part[GROUP_WAVES], wave_sum[GROUP_WAVES];
  const u32 t = threadIdx.x, lane = t & 63u, w = t >> 6, digits = 1u << high_bits, buckets = 1u << low_bits;
  u32* mine = count + w * digits;
  u32* filed = count + GROUP_WAVES * digits;
  if (t < 4) cnt_lds[t] = 0;
  if (t < 2) stat_lds[t] = 0;
  const u32 c = bucket_total[blockIdx.x];
  if (c == 0) return;
  // the bucket's first key: those of all buckets before it
  u32 before = 0;
  for (u32 i = t; i < buckets; i += 64u * GROUP_WAVES) before += i < blockIdx.x ? bucket_total[i] : 0u;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) before += (u32)__shfl_xor((int)before, off, 64);
  if (lane == 0) part[w] = before;
  for (u32 i = lane; i < digits; i += 64) mine[i] = 0;
  __syncthreads();
  u64 base = 0;
#pragma unroll
  for (u32 v = 0; v < GROUP_WAVES; ++v) base += part[v];
  // this wave's quarter, whole rows of 64
  const u32 rows = (c + 63u) / 64u, per = (rows + GROUP_WAVES - 1u) / GROUP_WAVES * 64u;
  const u32 lo = w * per < c ? w * per : c, hi = lo + per < c ? lo + per : c;
  for (u32 i = lo + lane; i < hi; i += 64) atomicAdd(&mine[(u32)(in[base + i] >> 32) >> low_bits], 1u);
  __syncthreads();
  // first places, digit by digit and in a digit wave by wave: a thread owns PL digits
  const u32 PL = (digits + 64u * GROUP_WAVES - 1u) / (64u * GROUP_WAVES);
  u32 total = 0;
  for (u32 j = 0; j < PL; ++j)
    if (PL * t + j < digits)
      for (u32 v = 0; v < GROUP_WAVES; ++v) total += count[v * digits + PL * t + j];
  u32 incl = total;
#pragma unroll
  for (u32 off = 1; off < 64; off <<= 1) {
    const u32 o = (u32)__shfl_up((int)incl, off, 64);
    if (lane >= off) incl += o;
  }
  if (lane == 63) wave_sum[w] = incl;
  __syncthreads();
  u32 run = incl - total;
  for (u32 v = 0; v < w; ++v) run += wave_sum[v];
  const u32 first_run = run;
  for (u32 j = 0; j < PL; ++j) {
    if (PL * t + j >= digits) break;
    for (u32 v = 0; v < GROUP_WAVES; ++v) {
      const u32 x = count[v * digits + PL * t + j];
      count[v * digits + PL * t + j] = run;
      run += x;
    }
  }
  __syncthreads();
  for (u32 i0 = lo; i0 < hi; i0 += 64) {
    const u32 i = i0 + lane;
    const bool valid = i < hi;
    const u64 key = valid ? in[base + i] : 0ull;
    const u32 dg = (u32)(key >> 32) >> low_bits;
    u64 match = ballot(valid);
    for (u32 bit = 0; bit < high_bits; ++bit) {
      const bool one = (dg >> bit) & 1u;
      const u64 bm = ballot(one);
      match &= one ? bm : ~bm;
    }
    u32 dst = 0;
    if (valid) dst = mine[dg] + (u32)__builtin_popcountll(match & lanemask_lt((int)lane));
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (valid && (match >> lane) == 1ull) mine[dg] += (u32)__builtin_popcountll(match);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (valid) out[base + dst] = key;
  }
  __syncthreads();  // (also before the appends read the keys back)
  // after the walk the last wave's counter of a digit is the end of its segment
  u32 from = first_run;
  for (u32 j = 0; j < PL; ++j) {
    const u32 dg = PL * t + j;
    if (dg >= digits) break;
    const u32 to = count[(GROUP_WAVES - 1u) * digits + dg];
    if (to > from) {
      const u32 b = (dg << low_bits) | blockIdx.x;
      const int kind = plan_segment(a, b, a.meta[b], to - from, stat_lds, [&](u32 k) { return (u32)(a.keys[base + from + k] & 0xFFFFFFFFull); });
      filed[dg] = kind < 0 ? 0xFFFFFFFFu : ((u32)kind << 30) | atomicAdd(&cnt_lds[kind], 1u);
    }
    from = to;
  }
  __syncthreads();
  plan_reserve(a, cnt_lds, base_lds, stat_lds);
  __syncthreads();
  from = first_run;
  for (u32 j = 0; j < PL; ++j) {
    const u32 dg = PL * t + j;
    if (dg >= digits) break;
    const u32 to = count[(GROUP_WAVES - 1u) * digits + dg];
    if (to > from && filed[dg] != 0xFFFFFFFFu) {
      const u32 b = (dg << low_bits) | blockIdx.x, kind = filed[dg] >> 30;
      plan_file(a, (int)kind, base_lds[kind] + (filed[dg] & 0x3FFFFFFFu), base + from, to - from, b, a.meta[b]);
    }
    from = to;
  }
}

hipError_t launch_group_plan(const MergeArgs& a, const u64* in, const u32* bucket_total, u32 low_bits, u32 high_bits,
                             hipStream_t s) {
  const u32 lds = (GROUP_WAVES + 1u) * (4u << high_bits);
  hipLaunchKernelGGL(group_plan_kernel, dim3(1u << low_bits), dim3(64 * GROUP_WAVES), lds, s, a, in, const_cast<u64*>(a.keys),
                     bucket_total, low_bits, high_bits);
  return hipGetLastError();
}

hipError_t launch_plan(const MergeArgs& a, hipStream_t s) {
  if (a.nkeys == 0) return hipSuccess;
  const u32 grid = (u32)((a.nkeys + 255) / 256);
  hipLaunchKernelGGL(plan_kernel, dim3(grid), dim3(256), 0, s, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// fast path: clean prefix plus at most FastAMax new entries
// ---------------------------------------------------------------------------------------------
template <int NCH>
struct FastAMax {
  static constexpr int value = NCH <= 2 ? 4 : (NCH <= 4 ? 2 : 1);
};

// lane-local part of the distance between a query and the row pieces x; `xx` is the shared
// <x,x> part for the integer kinds
template <int KIND, int VEC, int NCH>
__device__ __forceinline__ i32 xx_part(const Piece<VEC> (&x)[NCH]) {
  i32 xx = 0;
  if constexpr (KIND == K_U8) {
#pragma unroll
    for (int u = 0; u < NCH; ++u)
#pragma unroll
      for (int i = 0; i < VEC / 4; ++i) xx = (i32)__builtin_amdgcn_udot4(x[u].w[i], x[u].w[i], (u32)xx, false);
  } else if constexpr (KIND == K_I8) {
#pragma unroll
    for (int u = 0; u < NCH; ++u)
#pragma unroll
      for (int i = 0; i < VEC / 4; ++i) xx = __builtin_amdgcn_sdot4((i32)x[u].w[i], (i32)x[u].w[i], xx, false);
  }
  return xx;
}

template <int KIND, int VEC, int NCH>
__device__ __forceinline__ u32 distance_key_xx(const QueryRegs<KIND, VEC, NCH>& Q, const Piece<VEC> (&x)[NCH], i32 xx) {
  if constexpr (KIND == K_U8) {
    u32 qx = 0;
#pragma unroll
    for (int u = 0; u < NCH; ++u)
#pragma unroll
      for (int i = 0; i < VEC / 4; ++i) qx = __builtin_amdgcn_udot4(Q.q[u].w[i], x[u].w[i], qx, false);
    return dkey_from_int(group_sum(xx - 2 * (i32)qx) + Q.qq);
  } else if constexpr (KIND == K_I8) {
    i32 qx = 0;
#pragma unroll
    for (int u = 0; u < NCH; ++u)
#pragma unroll
      for (int i = 0; i < VEC / 4; ++i) qx = __builtin_amdgcn_sdot4((i32)Q.q[u].w[i], (i32)x[u].w[i], qx, false);
    return dkey_from_int(group_sum(xx - 2 * qx) + Q.qq);
  } else {
    return distance_key<KIND, VEC, NCH>(Q, x);
  }
}

// One row of the fast path with exactly NA new entries (a compile-time count keeps every loop
// over the new entries fully unrolled and free of guards).
template <int KIND, int VEC, int NCH, int NA>
__device__ __forceinline__ u32 fast_item(const MergeArgs& a, const VecTable& T, const AlphaParam& al, u32* ids_lds,
                                         u32 (*dk_lds)[64], u32 b, u32 i0, u32 clean, u32 stale, u32* row, u32 R,
                                         int lane) {
  // all nine passes (eight over the clean prefix, one over the new entries) requested at once when
  // the pieces fit the register file: one trip to memory instead of three
  constexpr int PBF = VEC * NCH <= 16 ? 9 : (VEC * NCH <= 32 ? 5 : (PassBatch<VEC, NCH>::value > 4 ? 4 : PassBatch<VEC, NCH>::value));
  constexpr u32 na = NA;
  const int sub = lane & (LPC - 1);
  const u32 grp = (u32)lane >> 3;
    const u32 myid = (u32)lane < clean ? row[lane] : NONE_ID;
    u32 mynew = NONE_ID;
    if ((u32)lane < na) mynew = (u32)lane < stale ? row[clean + lane] : (u32)(a.keys[i0 + (lane - stale)] & 0xFFFFFFFFull);
    ids_lds[lane] = myid;
    if ((u32)lane < na) ids_lds[64 + lane] = mynew;

    const QueryRegs<KIND, VEC, NCH> Qb = load_query<KIND, VEC, NCH>(T.base + (u64)b * T.row_bytes, T.npieces, lane);
    QueryRegs<KIND, VEC, NCH> Qn[NA];
    u32 nid[NA];
#pragma unroll
    for (int k = 0; k < NA; ++k) {
      nid[k] = readlane_u32(mynew, k);
      if ((u32)k < na)
        Qn[k] = load_query<KIND, VEC, NCH>(T.base + (u64)nid[k] * T.row_bytes, T.npieces, lane);
      else
        Qn[k] = Qb;
    }
    __syncthreads();

    // one sweep over the clean prefix and the new entries: candidate index c < clean is row
    // position c, index 64 + k is new entry k; each is measured against b and every new entry
    u32 res[1 + NA];
#pragma unroll
    for (int q = 0; q <= NA; ++q) res[q] = 0;
    u32 newres[1 + NA];  // the same for the pass over the new entries (valid in lanes 8k)
#pragma unroll
    for (int q = 0; q <= NA; ++q) newres[q] = 0;
    const u32 npass_clean = (clean + 7u) >> 3;
    for (u32 t0 = 0; t0 < npass_clean + 1; t0 += PBF) {
      Piece<VEC> x[PBF][NCH];
#pragma unroll
      for (int tt = 0; tt < PBF; ++tt) {
        const u32 t = t0 + tt;
        // passes 0..npass_clean-1 cover the clean prefix, pass npass_clean the new entries
        const bool newpass = t == npass_clean;
        const u32 c = newpass ? grp : 8u * t + grp;
        const bool ok = newpass ? (grp < na) : (t < npass_clean && c < clean);
        const u32 id = ok ? ids_lds[newpass ? 64 + grp : c] : 0u;
        const char* src = T.base + (u64)id * T.row_bytes;
#pragma unroll
        for (int u = 0; u < NCH; ++u) {
          const u32 pc = sub + LPC * u;
          x[tt][u] = (ok && pc < T.npieces) ? load_piece<VEC>(src + (u64)pc * VEC) : zero_piece<VEC>();
        }
      }
#pragma unroll
      for (int tt = 0; tt < PBF; ++tt) {
        const u32 t = t0 + tt;
        if (t <= npass_clean) {  // uniform
          const i32 xx = xx_part<KIND, VEC, NCH>(x[tt]);
          const bool newpass = t == npass_clean;
          const u32 d0 = distance_key_xx<KIND, VEC, NCH>(Qb, x[tt], xx);
          if (newpass)
            newres[0] = d0;
          else if ((u32)sub == t)
            res[0] = d0;
#pragma unroll
          for (int k = 0; k < NA; ++k) {
            if ((u32)k < na) {  // uniform
              const u32 dkk = distance_key_xx<KIND, VEC, NCH>(Qn[k], x[tt], xx);
              if (newpass)
                newres[1 + k] = dkk;
              else if ((u32)sub == t)
                res[1 + k] = dkk;
            }
          }
        }
      }
    }
    // lane l holds the results of row position cand_of_lane(l); bring them to lane = position
    {
      const u32 c = cand_of_lane(lane);
#pragma unroll
      for (int q = 0; q <= NA; ++q) dk_lds[q][c] = res[q];
    }
    __syncthreads();
    const bool isc = (u32)lane < clean;
    const u32 dB = dk_lds[0][lane];
    const u64 keyc = isc ? make_key(dB, myid) : KEY_INF;

    // per new entry k: its key, its place among the clean entries, what it removes, what removes it
    u64 keyn[NA];
    u32 rank[NA];
    u64 removes[NA], removed_by[NA];
    u32 dBn[NA];
#pragma unroll
    for (int k = 0; k < NA; ++k) {
      dBn[k] = readlane_u32(newres[0], 8 * k);
      keyn[k] = make_key(dBn[k], nid[k]);
      const u32 dkj = dk_lds[1 + k][lane];  // distance new entry k <-> clean entry `lane`
      rank[k] = (u32)__builtin_popcountll(ballot(isc && keyc < keyn[k]));
      removes[k] = ballot(isc && alpha_dominates<KIND>(al, dkj, dB));
      removed_by[k] = ballot(isc && alpha_dominates<KIND>(al, dkj, dBn[k]));
    }
    // replay the scan: clean entries never remove each other, so only the new entries matter
    u64 alive = clean >= 64 ? ~0ull : ((1ull << clean) - 1ull);
    u32 selnew = 0;
#pragma unroll
    for (int r = 0; r < NA; ++r) {
      // the new entry that is r-th among the new entries in (distance, id) order
#pragma unroll
      for (int k = 0; k < NA; ++k) {
        if ((u32)k < na) {
          u32 ord = 0;
#pragma unroll
          for (int l = 0; l < NA; ++l)
            if ((u32)l < na && keyn[l] < keyn[k]) ++ord;
          if (ord == (u32)r) {
            const u64 before = rank[k] >= 64 ? ~0ull : ((1ull << rank[k]) - 1ull);
            bool killed = (removed_by[k] & alive & before) != 0;
#pragma unroll
            for (int l = 0; l < NA; ++l) {
              if ((u32)l < na && l != k && ((selnew >> l) & 1u) && keyn[l] < keyn[k]) {
                // distance new l <-> new k: query l against candidate k of the new pass
                const u32 dlk = readlane_u32(newres[1 + l], 8 * k);
                killed = killed || alpha_dominates<KIND>(al, dlk, dBn[k]);
              }
            }
            if (!killed) {
              selnew |= 1u << k;
              alive &= ~(removes[k] & ~before);
            }
          }
        }
      }
    }
    // positions in the merged order, cut at R
    u32 pos = (u32)__builtin_popcountll(alive & lanemask_lt(lane));
    u32 newpos = 0;
#pragma unroll
    for (int k = 0; k < NA; ++k) {
      if ((u32)k < na && ((selnew >> k) & 1u)) {
        if (rank[k] <= (u32)lane) ++pos;  // new entry k precedes clean entry `lane`
        const u64 before = rank[k] >= 64 ? ~0ull : ((1ull << rank[k]) - 1ull);
        u32 pk = (u32)__builtin_popcountll(alive & before);
#pragma unroll
        for (int l = 0; l < NA; ++l)
          if ((u32)l < na && ((selnew >> l) & 1u) && keyn[l] < keyn[k]) ++pk;
        if (lane == k) newpos = pk;
      }
    }
    const u32 nsel = (u32)__builtin_popcountll(alive) + (u32)__builtin_popcount(selnew);
    const u32 kept = nsel < R ? nsel : R;
    __syncthreads();
    if (isc && ((alive >> lane) & 1ull) && pos < R) row[pos] = myid;
    if ((u32)lane < na && ((selnew >> lane) & 1u) && newpos < R) row[newpos] = mynew;
    for (u32 j = kept + lane; j < R; j += 64) row[j] = NONE_ID;
    if (lane == 0) a.meta[b] = make_meta(kept, kept);
    return kept;
}

// what a workgroup's re-prunes add to the counters
struct MergeStats {
  unsigned long long rep = 0, edges = 0, pair = 0;
  __device__ __forceinline__ void add(const MergeArgs& a, int lane) const {
    if (a.counters != nullptr && lane == 0 && rep) {
      atomicAdd(&block_counters(a.counters)->reprunes, rep);
      atomicAdd(&block_counters(a.counters)->edges, edges);
      atomicAdd(&block_counters(a.counters)->prune_evals, pair);
    }
  }
};

template <int NCH>
struct FastLds {
  static constexpr int AMAX = FastAMax<NCH>::value;
  u32 ids[64 + AMAX];    // clean ids by row position, then the new ids
  u32 dk[1 + AMAX][64];  // distance keys by row position: to b, to each new entry
};

template <int KIND, int VEC, int NCH>
__device__ __forceinline__ void merge_fast_one(const MergeArgs& a, const VecTable& T, FastLds<NCH>& L, u32 it, int lane,
                                               MergeStats& stats) {
  constexpr int AMAX = FastAMax<NCH>::value;
  const AlphaParam al{a.a16, a.af};
  const MergeItem item = a.list_items[0][it];
  const u32 i0 = item.i0, cnt = item.cnt, b = item.b, m = item.meta;
  const u32 deg = meta_deg(m), clean = meta_clean(m);
  const u32 stale = deg - clean;  // appended since the last prune
  const u32 na = stale + cnt;     // 1 <= na <= AMAX
  u32* row = a.graph + (u64)b * a.R;
  // uniform dispatch on the number of new entries
#define ANN_FAST_CASE(N)                                                                              \
  case N:                                                                                             \
    if constexpr (AMAX >= N)                                                                          \
      (void)fast_item<KIND, VEC, NCH, N>(a, T, al, L.ids, L.dk, b, i0, clean, stale, row, a.R, lane); \
    break;
  switch (na) {
    ANN_FAST_CASE(1)
    ANN_FAST_CASE(2)
    ANN_FAST_CASE(3)
    ANN_FAST_CASE(4)
    ANN_FAST_CASE(5)
    ANN_FAST_CASE(6)
    ANN_FAST_CASE(7)
    ANN_FAST_CASE(8)
    default: break;
  }
#undef ANN_FAST_CASE
  ++stats.rep;
  stats.edges += cnt;
  stats.pair += (unsigned long long)(clean + na) * (na + 1);
}

template <int KIND, int VEC, int NCH>
__global__ __launch_bounds__(64) void merge_fast_kernel(MergeArgs a, VecTable T) {
  __shared__ FastLds<NCH> lds;
  const int lane = threadIdx.x;
  const u32 nitems = a.list_count[0];
  MergeStats stats;
  for (u32 it = blockIdx.x; it < nitems; it += gridDim.x) merge_fast_one<KIND, VEC, NCH>(a, T, lds, it, lane, stats);
  stats.add(a, lane);
}

// ---------------------------------------------------------------------------------------------
// prune of a short candidate list of u8/i8 vectors with the matrix cores
//
// An overflowing row has R old entries plus a few new ones.  For such a list every pair
// distance the scan of prune() can ask for is an entry of the Gram matrix of the candidate
// vectors, a small dense contraction.  The wave stages the vectors in LDS (u8 shifted by -128 so
// that they are int8; distances are translation invariant), sorts the candidates by
// (d(b,.), id), forms the Gram matrix of the sorted list with v_mfma_i32_32x32x32_i8 (exact in
// int32), reduces each entry at once to the bit "i removes j" (alpha * D(i,j) <= d(b,j), as the
// equivalent D(i,j) <= floor(d(b,j) * 2^16 / a16)), and then replays the scan of prune() on bit
// masks with scalar instructions.
// ---------------------------------------------------------------------------------------------
constexpr u32 SM_TMAX = 96;     // candidates handled by this path

struct SmallLds {
  u64 key[SM_TMAX];   // by arrival index
  u32 uid[SM_TMAX];   // ids by arrival index
  u32 nrm[SM_TMAX];   // squared norms of the shifted vectors, by arrival index
  u32 sid[SM_TMAX];   // ids, sorted by (distance to b, id)
  u32 snrm[SM_TMAX];  // norms, sorted
  i32 sthr[SM_TMAX];  // largest D(i,j) that still removes j, sorted
  u32 inv[SM_TMAX];   // sorted position -> arrival index
  // the entries behind the clean prefix ("new"), by their index among the new entries
  u32 nnrm[32];  // norms
  i32 nthr[32];  // largest D that still removes the new entry
  u32 npos[32];  // sorted positions
};

template <int VEC, int NCH>
struct SmallPathOk {
  static constexpr bool value = (8 * NCH * VEC <= 256);
};

// One 32x32 tile of the Gram matrix of the sorted candidates: rows 32*RB.., columns 32*CB...
// Accumulator register r of lane l is entry (row 8*(r/4) + 4*(l/32) + r%4, column l%32), so one
// ballot per register yields the 32 "removes" bits of two rows, which go to the lanes that own
// those rows.
template <int RB, int CB, int R_>
__device__ __forceinline__ void gram_tile_reg(const v16i_t& acc, const SmallLds& S, bool colok, i32 ncol, i32 tcol,
                                              u32 half, u32& Klo, u32& Khi) {
  constexpr int mlo = 32 * RB + 8 * (R_ / 4) + (R_ % 4);
  const i32 nrow = (i32)S.snrm[mlo + 4 * half];
  const i32 D = nrow + ncol - 2 * acc[R_];
  const u64 bm = ballot(colok && D <= tcol);
  if constexpr (mlo < 64) {
    Klo = writelane_pair<mlo, mlo + 4>(Klo, bm);
  } else if constexpr (CB == 2) {
    Khi = writelane_pair<mlo - 64, mlo + 4 - 64>(Khi, bm);
  }
}

template <int RB, int CB, int... Rs>
__device__ __forceinline__ void gram_tile_regs(const v16i_t& acc, const SmallLds& S, bool colok, i32 ncol, i32 tcol,
                                               u32 half, u32& Klo, u32& Khi, std::integer_sequence<int, Rs...>) {
  (gram_tile_reg<RB, CB, Rs>(acc, S, colok, ncol, tcol, half, Klo, Khi), ...);
}

template <int NCH, int RB, int CB>
__device__ __forceinline__ void gram_tile(const unsigned char* Xs, const SmallLds& S, u32 total, u32 ksteps, int lane,
                                          u32& Klo, u32& Khi) {
  constexpr u32 KS = 4u * NCH, SM_STRIDE = mm_stride(128u * NCH);
  const u32 half = (u32)lane >> 5;
  const u32 ia = 32u * RB + (lane & 31), ib = 32u * CB + (lane & 31);
  const u32 ra = ia < total ? S.inv[ia] : 0u;
  const u32 rb = ib < total ? S.inv[ib] : 0u;
  const unsigned char* pa = Xs + ra * SM_STRIDE + 16u * half;
  const unsigned char* pb = Xs + rb * SM_STRIDE + 16u * half;
  v16i_t acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  // all k-steps unconditionally: operands beyond the row's last step are zeroed
  v4i_t av[KS], bv[KS];
#pragma unroll
  for (u32 ks = 0; ks < KS; ++ks) {
    const u32 kk = ks < ksteps ? ks : ksteps - 1u;
    const v4i_t x = *reinterpret_cast<const v4i_t*>(pa + 32u * kk);
    const v4i_t y = *reinterpret_cast<const v4i_t*>(pb + 32u * kk);
    av[ks] = ks < ksteps ? x : v4i_t{0, 0, 0, 0};
    bv[ks] = y;
  }
#pragma unroll
  for (u32 ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(av[ks], bv[ks], acc, 0, 0, 0);
  const bool colok = ib < total;
  const i32 ncol = colok ? (i32)S.snrm[ib] : 0;
  const i32 tcol = colok ? S.sthr[ib] : -1;
  gram_tile_regs<RB, CB>(acc, S, colok, ncol, tcol, half, Klo, Khi, std::make_integer_sequence<int, 16>{});
}

// The same tile with the NEW entries as rows (new entry t in row t, at most 32 of them) and the
// sorted candidates 32*CB.. as columns.  Each accumulator register that holds rows below `na`
// yields two ballots: "new t removes sorted candidate j" (alpha * D <= d(b, j)) and "sorted
// candidate j removes new t" (alpha * D <= d(b, t)); lane t collects word CB of both masks.
template <int CB, int R_>
__device__ __forceinline__ void newrow_tile_reg(const v16i_t& acc, const i32 (&rown)[16], const i32 (&rowt)[16], u32 na,
                                                bool colok, i32 ncol, i32 tcol, u32 half, u32& rem, u32& rby) {
  constexpr int mlo = 8 * (R_ / 4) + (R_ % 4);
  if (na > (u32)(8 * (R_ / 4))) {  // uniform: rows 8*(R_/4).. exist
    const u32 t = (u32)mlo + 4u * half;
    const bool ok = colok && t < na;
    const i32 D = rown[R_] + ncol - 2 * acc[R_];
    const u64 b1 = ballot(ok && D <= tcol);
    const u64 b2 = ballot(ok && D <= rowt[R_]);
    rem = writelane_pair<mlo, mlo + 4>(rem, b1);
    rby = writelane_pair<mlo, mlo + 4>(rby, b2);
  }
}
template <int CB, int... Rs>
__device__ __forceinline__ void newrow_tile_regs(const v16i_t& acc, const i32 (&rown)[16], const i32 (&rowt)[16], u32 na,
                                                 bool colok, i32 ncol, i32 tcol, u32 half, u32& rem, u32& rby,
                                                 std::integer_sequence<int, Rs...>) {
  (newrow_tile_reg<CB, Rs>(acc, rown, rowt, na, colok, ncol, tcol, half, rem, rby), ...);
}
template <int NCH, int CB>
__device__ __forceinline__ void newrow_tile(const unsigned char* Xs, const SmallLds& S, const i32 (&rown)[16],
                                            const i32 (&rowt)[16], u32 clean, u32 na, u32 total, u32 ksteps, int lane,
                                            u32& rem, u32& rby) {
  constexpr u32 KS = 4u * NCH, SM_STRIDE = mm_stride(128u * NCH);
  const u32 half = (u32)lane >> 5;
  const u32 t = (u32)lane & 31u;
  const u32 ib = 32u * CB + t;
  const u32 ra = clean + (t < na ? t : na - 1u);
  const u32 rb = ib < total ? S.inv[ib] : 0u;
  const unsigned char* pa = Xs + ra * SM_STRIDE + 16u * half;
  const unsigned char* pb = Xs + rb * SM_STRIDE + 16u * half;
  v4i_t av[KS], bv[KS];
#pragma unroll
  for (u32 ks = 0; ks < KS; ++ks) {
    const u32 kk = ks < ksteps ? ks : ksteps - 1u;
    const v4i_t x = *reinterpret_cast<const v4i_t*>(pa + 32u * kk);
    const v4i_t y = *reinterpret_cast<const v4i_t*>(pb + 32u * kk);
    av[ks] = ks < ksteps ? x : v4i_t{0, 0, 0, 0};
    bv[ks] = y;
  }
  v16i_t acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (u32 ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(av[ks], bv[ks], acc, 0, 0, 0);
  const bool colok = ib < total;
  const i32 ncol = colok ? (i32)S.snrm[ib] : 0;
  const i32 tcol = colok ? S.sthr[ib] : -1;
  newrow_tile_regs<CB>(acc, rown, rowt, na, colok, ncol, tcol, half, rem, rby, std::make_integer_sequence<int, 16>{});
}

// S.uid[0..total) holds the candidate ids (old row entries first), the first `clean` of which
// are the row's clean prefix: sorted, none removing another.  Writes the pruned row and
// returns its length.
template <int KIND, int VEC, int NCH>
__device__ __forceinline__ u32 reprune_small_int(const VecTable& T, const QueryRegs<KIND, VEC, NCH>& Q,
                                                 unsigned char* Xs, SmallLds& S, u32 total, u32 clean, u32 R,
                                                 i64 a16, u32* row, int lane) {
  // every pass of eight candidates is requested before the first is used (a pass is at most
  // eight registers here): one trip to memory for the whole list
  constexpr int PB = SM_TMAX / 8;
  constexpr u32 SM_STRIDE = mm_stride(128u * NCH);
  const int sub = lane & (LPC - 1);
  const u32 grp = (u32)lane >> 3;
  const u32 npass = (total + 7u) >> 3;
  const u32 flip = KIND == K_U8 ? 0x80808080u : 0u;

  // stage the vectors, take d(b, x) and the norms
  for (u32 t0 = 0; t0 < npass; t0 += PB) {
    Piece<VEC> x[PB][NCH];
    u32 ids[PB];
#pragma unroll
    for (int tt = 0; tt < PB; ++tt) {
      const u32 c = 8u * (t0 + tt) + grp;
      const bool ok = c < total;
      ids[tt] = ok ? S.uid[c] : 0u;
      const char* src = T.base + (u64)ids[tt] * T.row_bytes;
#pragma unroll
      for (int u = 0; u < NCH; ++u) {
        const u32 pc = sub + LPC * u;
        x[tt][u] = (ok && pc < T.npieces) ? load_piece<VEC>(src + (u64)pc * VEC) : zero_piece<VEC>();
      }
    }
#pragma unroll
    for (int tt = 0; tt < PB; ++tt) {
      if (t0 + tt >= npass) break;  // uniform
      const u32 c = 8u * (t0 + tt) + grp;
      const u32 dk = distance_key<KIND, VEC, NCH>(Q, x[tt]);
      i32 nn = 0;
#pragma unroll
      for (int u = 0; u < NCH; ++u) {
        const u32 pc = sub + LPC * u;
        u32 wv[VEC / 4];
#pragma unroll
        for (int i = 0; i < VEC / 4; ++i) {
          wv[i] = pc < T.npieces ? (x[tt][u].w[i] ^ flip) : 0u;
          nn = __builtin_amdgcn_sdot4((i32)wv[i], (i32)wv[i], nn, false);
        }
        if (c < total) {
          unsigned char* dst = Xs + c * SM_STRIDE + pc * VEC;
          if constexpr (VEC == 16) {
            *reinterpret_cast<uint4*>(dst) = make_uint4(wv[0], wv[1], wv[2], wv[3]);
          } else {
#pragma unroll
            for (int i = 0; i < VEC / 4; ++i) *reinterpret_cast<u32*>(dst + 4 * i) = wv[i];
          }
        }
      }
      nn = group_sum(nn);
      if (sub == 0 && c < total) {
        S.key[c] = make_key(dk, ids[tt]);
        S.nrm[c] = (u32)nn;
      }
    }
  }
  __syncthreads();

  // rank of every candidate under (distance, id); keys are distinct.  With at most 32 entries
  // behind the clean prefix only those are compared against everything: a clean entry's rank is
  // its place in the prefix plus the new entries below it.
  const u32 na = total - clean;
  const bool by_new_rows = na <= 32u;
  {
    const u32 j0 = lane, j1 = lane + 64;
    const u64 k0 = j0 < total ? S.key[j0] : KEY_INF;
    const u64 k1 = j1 < total ? S.key[j1] : KEY_INF;
    u32 r0 = 0, r1 = 0;
    if (by_new_rows) {
      const bool c0 = j0 < clean, c1 = j1 < clean;
      u32 below0 = 0, below1 = 0;  // for a new entry: clean entries below it
      for (u32 k = clean; k < total; ++k) {
        const u64 kk = S.key[k];
        const bool g0 = kk < k0, g1 = kk < k1;
        r0 += g0 ? 1u : 0u;
        r1 += g1 ? 1u : 0u;
        const u32 above = (u32)__builtin_popcountll(ballot(g0 && c0)) + (u32)__builtin_popcountll(ballot(g1 && c1));
        if (j0 == k) below0 = clean - above;
        if (j1 == k) below1 = clean - above;
      }
      r0 += c0 ? j0 : below0;
      r1 += c1 ? j1 : below1;
    } else {
      for (u32 i = 0; i < total; ++i) {
        const u64 ki = S.key[i];
        r0 += ki < k0 ? 1u : 0u;
        r1 += ki < k1 ? 1u : 0u;
      }
    }
    if (j0 < total) {
      const i32 thr = alpha_threshold(int_from_dkey(key_dkey(k0)), a16);
      S.sid[r0] = key_id(k0);
      S.snrm[r0] = S.nrm[j0];
      S.sthr[r0] = thr;
      S.inv[r0] = j0;
      if (by_new_rows && j0 >= clean) {
        S.nnrm[j0 - clean] = S.nrm[j0];
        S.nthr[j0 - clean] = thr;
        S.npos[j0 - clean] = r0;
      }
    }
    if (j1 < total) {
      const i32 thr = alpha_threshold(int_from_dkey(key_dkey(k1)), a16);
      S.sid[r1] = key_id(k1);
      S.snrm[r1] = S.nrm[j1];
      S.sthr[r1] = thr;
      S.inv[r1] = j1;
      if (by_new_rows && j1 >= clean) {
        S.nnrm[j1 - clean] = S.nrm[j1];
        S.nthr[j1 - clean] = thr;
        S.npos[j1 - clean] = r1;
      }
    }
  }
  __syncthreads();

  const u32 nb = (total + 31u) >> 5;
  const u32 ksteps = (u32)((T.row_bytes + 31) / 32);
  if (by_new_rows) {
    // distances between the new entries and everything, reduced at once to two 96-bit masks per
    // new entry (lane t: new entry t)
    u32 REM[3] = {0u, 0u, 0u}, RBY[3] = {0u, 0u, 0u};
    // norm and threshold of the row each accumulator register holds in this lane (the same in
    // every tile); rows that do not exist are never looked at
    i32 rown[16], rowt[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      rown[r] = 0;
      rowt[r] = -1;
      if (na > (u32)(8 * (r / 4))) {  // uniform
        const u32 t = (u32)(8 * (r / 4) + (r % 4)) + 4u * ((u32)lane >> 5);
        rown[r] = (i32)S.nnrm[t];
        rowt[r] = S.nthr[t];
      }
    }
    newrow_tile<NCH, 0>(Xs, S, rown, rowt, clean, na, total, ksteps, lane, REM[0], RBY[0]);
    if (nb > 1) newrow_tile<NCH, 1>(Xs, S, rown, rowt, clean, na, total, ksteps, lane, REM[1], RBY[1]);
    if (nb > 2) newrow_tile<NCH, 2>(Xs, S, rown, rowt, clean, na, total, ksteps, lane, REM[2], RBY[2]);
    const u32 mypos = (u32)lane < na ? S.npos[lane] : 0xFFFFFFFFu;

    // replay of the scan of prune() on positions of the sorted list: the clean entries are all
    // selected until a selected new entry in front of them removes them; the new entries are
    // decided in sorted order
    const u32 nlo = total < 64u ? total : 64u;
    u64 sel_lo = nlo == 64u ? ~0ull : ((1ull << nlo) - 1ull);
    u32 sel_hi = total > 64u ? ((total - 64u) >= 32u ? ~0u : ((1u << (total - 64u)) - 1u)) : 0u;
    u64 new_lo = 0;  // positions held by new entries
    u32 new_hi = 0;
    for (u32 t = 0; t < na; ++t) {
      const u32 p = readlane_u32(mypos, (int)t);
      if (p < 64u)
        new_lo |= 1ull << p;
      else
        new_hi |= 1u << (p - 64u);
    }
    sel_lo &= ~new_lo;
    sel_hi &= ~new_hi;
    u64 todo_lo = new_lo;
    u32 todo_hi = new_hi;
    while (todo_lo != 0 || todo_hi != 0) {
      u32 p;
      if (todo_lo != 0) {
        p = (u32)__builtin_ctzll(todo_lo);
        todo_lo &= todo_lo - 1ull;
      } else {
        p = 64u + (u32)__builtin_ctz(todo_hi);
        todo_hi &= todo_hi - 1u;
      }
      const int t = __builtin_ctzll(ballot(mypos == p));  // the new entry at position p
      const u64 before_lo = p >= 64u ? ~0ull : ((1ull << p) - 1ull);
      const u32 before_hi = p >= 64u ? ((1u << (p - 64u)) - 1u) : 0u;
      const u64 rby_lo = (u64)readlane_u32(RBY[0], t) | ((u64)readlane_u32(RBY[1], t) << 32);
      const u32 rby_hi = readlane_u32(RBY[2], t);
      const bool killed = ((rby_lo & sel_lo & before_lo) | (u64)(rby_hi & sel_hi & before_hi)) != 0;
      if (!killed) {
        const u64 rem_lo = (u64)readlane_u32(REM[0], t) | ((u64)readlane_u32(REM[1], t) << 32);
        const u32 rem_hi = readlane_u32(REM[2], t);
        sel_lo &= ~(rem_lo & ~before_lo);
        sel_hi &= ~(rem_hi & ~before_hi);
        if (p < 64u)
          sel_lo |= 1ull << p;
        else
          sel_hi |= 1u << (p - 64u);
      }
    }
    // the first R selected positions, in order
    const u32 cnt_lo = (u32)__builtin_popcountll(sel_lo);
    const u32 nsel = cnt_lo + (u32)__builtin_popcount(sel_hi);
    const u32 nout = nsel < R ? nsel : R;
    if ((sel_lo >> lane) & 1ull) {
      const u32 at = (u32)__builtin_popcountll(sel_lo & lanemask_lt(lane));
      if (at < R) row[at] = S.sid[lane];
    }
    if (lane < 32 && ((sel_hi >> lane) & 1u)) {
      const u32 at = cnt_lo + (u32)__builtin_popcount(sel_hi & ((1u << lane) - 1u));
      if (at < R) row[at] = S.sid[64 + lane];
    }
    for (u32 j = nout + lane; j < R; j += 64) row[j] = NONE_ID;
    __syncthreads();
    return nout;
  }

  // Gram matrix tile by tile; K0[c] of lane i = bits "sorted candidate i removes candidate 32c+j",
  // K1 the same for candidates 64..95 (only column block 2 matters there)
  u32 K0[3] = {0u, 0u, 0u};
  u32 K1 = 0u;
  gram_tile<NCH, 0, 0>(Xs, S, total, ksteps, lane, K0[0], K1);
  if (nb > 1) {
    gram_tile<NCH, 0, 1>(Xs, S, total, ksteps, lane, K0[1], K1);
    gram_tile<NCH, 1, 1>(Xs, S, total, ksteps, lane, K0[1], K1);
  }
  if (nb > 2) {
    gram_tile<NCH, 0, 2>(Xs, S, total, ksteps, lane, K0[2], K1);
    gram_tile<NCH, 1, 2>(Xs, S, total, ksteps, lane, K0[2], K1);
    gram_tile<NCH, 2, 2>(Xs, S, total, ksteps, lane, K0[2], K1);
  }

  // the scan of prune(): walk the sorted list, select what is still alive, remove what it removes
  const u32 nlo = total < 64u ? total : 64u;
  u64 rem_lo = nlo == 64u ? ~0ull : ((1ull << nlo) - 1ull);
  u32 rem_hi = total > 64u ? ((total - 64u) >= 32u ? ~0u : ((1u << (total - 64u)) - 1u)) : 0u;
  u64 sel_lo = 0;
  u32 sel_hi = 0, nout = 0;
  while (rem_lo != 0 && nout < R) {
    const int i = __builtin_ctzll(rem_lo);
    sel_lo |= 1ull << i;
    ++nout;
    const u64 klo = (u64)readlane_u32(K0[0], i) | ((u64)readlane_u32(K0[1], i) << 32);
    rem_lo &= ~klo;
    rem_lo &= ~(1ull << i);
    rem_hi &= ~readlane_u32(K0[2], i);
  }
  while (rem_hi != 0 && nout < R) {
    const int i = __builtin_ctz(rem_hi);
    sel_hi |= 1u << i;
    ++nout;
    rem_hi &= ~readlane_u32(K1, i);
    rem_hi &= ~(1u << i);
  }

  // write the row: selected ids in sorted order, then padding
  if ((sel_lo >> lane) & 1ull) row[__builtin_popcountll(sel_lo & lanemask_lt(lane))] = S.sid[lane];
  if (lane < 32 && ((sel_hi >> lane) & 1u))
    row[__builtin_popcountll(sel_lo) + __builtin_popcount(sel_hi & ((1u << lane) - 1u))] = S.sid[64 + lane];
  for (u32 j = nout + lane; j < R; j += 64) row[j] = NONE_ID;
  __syncthreads();
  return nout;
}

// ---------------------------------------------------------------------------------------------
// gram path kernel
// ---------------------------------------------------------------------------------------------
template <int NCH>
struct GramLds {
  __align__(16) unsigned char Xs[SM_TMAX * mm_stride(128u * NCH)];
  SmallLds small;
};

template <int KIND, int VEC, int NCH>
__device__ __forceinline__ void merge_gram_one(const MergeArgs& a, const VecTable& T, GramLds<NCH>& L, u32 it, int lane,
                                               MergeStats& stats) {
  const MergeItem item = a.list_items[1][it];
  const u32 i0 = item.i0, cnt = item.cnt, b = item.b;
  const u32 deg = meta_deg(item.meta), clean = meta_clean(item.meta);
  const u32 total = deg + cnt;
  u32* row = a.graph + (u64)b * a.R;
  for (u32 j = lane; j < total; j += 64)
    L.small.uid[j] = j < deg ? row[j] : (u32)(a.keys[i0 + (j - deg)] & 0xFFFFFFFFull);
  __syncthreads();
  const QueryRegs<KIND, VEC, NCH> Qb = load_query<KIND, VEC, NCH>(T.base + (u64)b * T.row_bytes, T.npieces, lane);
  const u32 kept = reprune_small_int<KIND, VEC, NCH>(T, Qb, L.Xs, L.small, total, clean, a.R, a.a16, row, lane);
  if (lane == 0) a.meta[b] = make_meta(kept, kept);
  ++stats.rep;
  stats.edges += cnt;
  // pairs whose distance was formed: all of them, or only those with a new entry in them
  stats.pair += total - clean <= 32u ? (unsigned long long)(total - clean) * total : (unsigned long long)total * (total + 1) / 2;
}

template <int KIND, int VEC, int NCH>
__global__ __launch_bounds__(64) void merge_gram_kernel(MergeArgs a, VecTable T) {
  if constexpr (KindTraits<KIND>::is_int && SmallPathOk<VEC, NCH>::value) {
    __shared__ GramLds<NCH> lds;
    const int lane = threadIdx.x;
    const u32 nitems = a.list_count[1];
    MergeStats stats;
    for (u32 it = blockIdx.x; it < nitems; it += gridDim.x) merge_gram_one<KIND, VEC, NCH>(a, T, lds, it, lane, stats);
    stats.add(a, lane);
  }
}

// prune(b, U, R) of float rows whose list is a clean prefix and at most F32_NEW_MAX further entries: as in the
// fast path only pairs with a new entry can change anything.  The new entries are the columns of the
// products, the whole list, 16 rows at a time, the other operand: (total / 16) tiles instead of the
// tiles of every block against everything selected.  cand[0..total): sorted keys, bit 0 set in the new ones.
// One verdict per pair serves, "the earlier removes the later".  Writes the row, returns its length.
// Bound by the matrix cores' 32 cycles per element and tile, as the walk is.  Squared L2, 300,000 points of 200 floats, R = 64,
// L = 128: build 208 -> 160 ms; 100,000 of 96, R = 48: 26.9 -> 25.5; layered,
// 50,000 of 120: 36.2 -> 33.9.  16 new entries are one tile of columns; 128 positions are two words of masks.
constexpr u32 F32_NEW_MAX = 16, F32_LIST_MAX = 128;
template <int KIND, int NCH>
__device__ __forceinline__ u32 reprune_new_f32(const VecTable& T, const F32Lds& M, const char* prow, const u64* cand,
                                               u32 total, u32 R, float af, u32* row, int lane) {
  constexpr bool L2 = KIND == K_F32_L2;
  const u32 blk = (u32)lane >> 4, r = (u32)lane & 15u;
  if constexpr (L2) {
    const u32 np8 = (T.npieces + 7u) & ~7u;
    if ((u32)lane < np8)
      M.p[lane] = (u32)lane < T.npieces ? reinterpret_cast<const float4*>(prow)[lane] : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  const u64 k0 = (u32)lane < total ? cand[lane] : 0ull, k1 = (u32)lane + 64u < total ? cand[lane + 64] : 0ull;
  const u64 new_lo = ballot(k0 & 1ull), new_hi = ballot(k1 & 1ull);
  const u32 na_lo = (u32)__builtin_popcountll(new_lo), na = na_lo + (u32)__builtin_popcountll(new_hi);
  // this lane's column: the r-th new entry (the last one again behind the end)
  u32 mypos;
  {
    const u32 c = r < na ? r : na - 1u;
    u64 w = c < na_lo ? new_lo : new_hi;
    for (u32 k = c < na_lo ? c : c - na_lo; k > 0; --k) w &= w - 1ull;
    mypos = (u32)__builtin_ctzll(w) + (c < na_lo ? 0u : 64u);
  }
  const u64 ckey = cand[mypos];
  const float dcol = float_from_dkey(key_dkey(ckey));
  __syncthreads();
  F32Operand<NCH> b;
  f32_load<KIND, NCH>(b, T.base + (u64)key_id(ckey) * T.row_bytes, T.npieces, blk);
  f32_centre<KIND, NCH>(b, M, T.npieces, blk);
  auto norm_of = [](const F32Operand<NCH>& o) {
    float n = 0.0f;
#pragma unroll
    for (int u = 0; u < NCH; ++u)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float4 x = o.x[h][u];
        n = __builtin_fmaf(x.x, x.x, n);
        n = __builtin_fmaf(x.y, x.y, n);
        n = __builtin_fmaf(x.z, x.z, n);
        n = __builtin_fmaf(x.w, x.w, n);
      }
    n += __shfl_xor(n, 16, 64);
    n += __shfl_xor(n, 32, 64);
    return n;
  };
  const float ncol = L2 ? norm_of(b) : 0.0f;
  // of this lane's column: the positions whose pair with it ends in a removal, and those to be measured
  u64 hit_lo = 0, hit_hi = 0, open_lo = 0, open_hi = 0;
  for (u32 i0 = 0; i0 < total; i0 += 16) {
    F32Operand<NCH> a;
    f32_load<KIND, NCH>(a, T.base + (u64)key_id(cand[i0 + r < total ? i0 + r : total - 1u]) * T.row_bytes, T.npieces, blk);
    f32_centre<KIND, NCH>(a, M, T.npieces, blk);
    if constexpr (L2) {
      const float n = norm_of(a);
      if (lane < 16) M.cnorm[lane] = n;
      __syncthreads();
    }
    float dot[4];
    f32_products<NCH>(a, b, T.npieces, dot);
    u32 hit = 0, open = 0;
#pragma unroll
    for (u32 v = 0; v < 4; ++v) {
      const u32 i = i0 + 4u * blk + v;
      const float drow = float_from_dkey(key_dkey(cand[i < total ? i : total - 1u]));
      const float nrow = L2 ? M.cnorm[4u * blk + v] : 0.0f;
      const int verdict = f32_verdict<KIND>(dot[v], nrow, ncol, af, i > mypos ? drow : dcol);
      hit |= (verdict > 0 ? 1u : 0u) << (4u * blk + v);
      open |= (verdict == 0 ? 1u : 0u) << (4u * blk + v);
    }
    hit |= (u32)__shfl_xor((int)hit, 16, 64);
    hit |= (u32)__shfl_xor((int)hit, 32, 64);
    (i0 < 64u ? hit_lo : hit_hi) |= (u64)hit << (i0 & 63u);
    if constexpr (L2) {
      open |= (u32)__shfl_xor((int)open, 16, 64);
      open |= (u32)__shfl_xor((int)open, 32, 64);
      (i0 < 64u ? open_lo : open_hi) |= (u64)open << (i0 & 63u);
      __syncthreads();  // (the norms, before the next tile's)
    }
  }
  // replay of the scan on positions, as in reprune_small_int
  const u64 all_lo = total >= 64u ? ~0ull : (1ull << total) - 1ull;
  const u64 all_hi = total <= 64u ? 0ull : total >= 128u ? ~0ull : (1ull << (total - 64u)) - 1ull;
  u64 sel_lo = all_lo & ~new_lo, sel_hi = all_hi & ~new_hi;
  for (u32 t = 0; t < na; ++t) {
    const u32 p = readlane_u32(mypos, (int)t);
    const u64 bit_lo = p < 64u ? 1ull << p : 0ull, bit_hi = p < 64u ? 0ull : 1ull << (p - 64u);
    const u64 before_lo = p < 64u ? bit_lo - 1ull : ~0ull, before_hi = p < 64u ? 0ull : bit_hi - 1ull;
    const u64 h_lo = readlane_u64(hit_lo, (int)t), h_hi = readlane_u64(hit_hi, (int)t);
    bool killed = ((h_lo & sel_lo & before_lo) | (h_hi & sel_hi & before_hi)) != 0;
    u64 o_lo = 0, o_hi = 0;
    if constexpr (L2) {
      o_lo = readlane_u64(open_lo, (int)t);
      o_hi = readlane_u64(open_hi, (int)t);
      for (u32 w = 0; w < 2; ++w) {
        u64 m = w == 0 ? o_lo & sel_lo & before_lo : o_hi & sel_hi & before_hi;
        for (; m != 0 && !killed; m &= m - 1ull)
          killed = f32_measured(T, key_id(cand[64u * w + (u32)__builtin_ctzll(m)]), cand + p, 1u, af, lane) != 0;
      }
    }
    if (killed) continue;
    sel_lo &= ~(h_lo & ~before_lo & ~bit_lo);
    sel_hi &= ~(h_hi & ~before_hi & ~bit_hi);
    if constexpr (L2) {
      const u64 rest_lo = o_lo & sel_lo & ~before_lo & ~bit_lo, rest_hi = o_hi & sel_hi & ~before_hi & ~bit_hi;
      for (u32 q = 0; (rest_lo | rest_hi) != 0 && q < 8; ++q) {
        const u32 mask = (u32)((q < 4 ? rest_lo : rest_hi) >> (16u * (q & 3u))) & 0xFFFFu;
        if (!mask) continue;
        const u64 gone = (u64)f32_measured(T, key_id(cand[p]), cand + 16u * q, mask, af, lane) << (16u * (q & 3u));
        if (q < 4)
          sel_lo &= ~gone;
        else
          sel_hi &= ~gone;
      }
    }
    sel_lo |= bit_lo;
    sel_hi |= bit_hi;
  }
  // the first R selected positions, in order
  const u32 cnt_lo = (u32)__builtin_popcountll(sel_lo), nsel = cnt_lo + (u32)__builtin_popcountll(sel_hi);
  const u32 kept = nsel < R ? nsel : R;
  if ((sel_lo >> lane) & 1ull) {
    const u32 at = (u32)__builtin_popcountll(sel_lo & lanemask_lt(lane));
    if (at < R) row[at] = key_id(k0);
  }
  if ((sel_hi >> lane) & 1ull) {
    const u32 at = cnt_lo + (u32)__builtin_popcountll(sel_hi & lanemask_lt(lane));
    if (at < R) row[at] = key_id(k1);
  }
  for (u32 j = kept + lane; j < R; j += 64) row[j] = NONE_ID;
  return kept;
}

// ---------------------------------------------------------------------------------------------
// generic path kernel
// ---------------------------------------------------------------------------------------------
// CAP: candidate keys the kernel sorts in LDS.  Two instances: MERGE_SPILL_MIN for the few rows
// with long lists (hub vertices; beyond it the list goes to the arena), and MERGE_MEDIUM_MAX for
// the rows in between, which are many when batches hold millions of points: with the large
// buffer three waves fit a compute unit, with the small one sixteen.
// (Byte rows above 128 bytes: left alone, the compiler takes registers for one wave per SIMD.)
template <int KIND, int VEC, int NCH, u32 CAP>
__device__ __forceinline__ void merge_generic_one(const MergeArgs& a, const VecTable& T, u64* cand_lds, unsigned char* smem, u32 it,
                                                  int lane, MergeStats& stats) {
  constexpr int LIST = CAP == MERGE_SPILL_MIN ? 2 : 3;
  constexpr bool kF32 = F32PruneOk<KIND, VEC, NCH>::value;
  u32* out = reinterpret_cast<u32*>(smem);  // R entries
  SelStage st;
  st.stride = stage_stride(T.row_bytes);
  st.xx = out + a.R;
  unsigned char* blk = smem + ((a.R * 8u + 15u) & ~15u);  // 8 rows + 8 norms
  st.vec = a.stage_bytes ? blk + 8u * st.stride + 32u : nullptr;
  F32Lds F{};
  if constexpr (kF32) F = f32_lds_carve(smem, a.R, out);
  constexpr bool kMfma = MfmaPruneOk<KIND, VEC, NCH>::value;
  const MfmaLds M = mfma_lds_carve(smem + ((a.R * 4u + 15u) & ~15u), a.R, T.row_bytes);  // used when a.use_mfma
  const AlphaParam al{a.a16, a.af};
  const MergeItem item = a.list_items[LIST][LIST == 3 ? -(long long)it : (long long)it];
  const u32 i0 = item.i0, cnt = item.cnt, b = item.b;
  const u32 deg = meta_deg(item.meta);
  const u32 total = deg + cnt;
  u32* row = a.graph + (u64)b * a.R;
  // a clean prefix and few new entries (meta holds no prefix where one cannot be relied on)
  const u32 clean = meta_clean(item.meta);
  const bool by_new = kF32 && CAP == MERGE_MEDIUM_MAX && clean > 0 && total - clean <= F32_NEW_MAX && total <= F32_LIST_MAX;

  // candidate list U = N_out(b) followed by the new sources
  u64* cand;
  const bool in_lds = total <= CAP;
  if (in_lds) {
    cand = cand_lds;
  } else {
    unsigned long long off = 0;
    if (lane == 0) off = atomicAdd(a.arena_top, (unsigned long long)total);
    off = readlane_u64(off, 0);
    if (off + total > a.arena_cap) {  // cannot happen with the arena sized by the host
      if (lane == 0) *a.error_flag = 1u;
      return;
    }
    cand = a.arena + off;
  }
  for (u32 j = lane; j < total; j += 64) {
    const u32 id = j < deg ? row[j] : (u32)(a.keys[i0 + (j - deg)] & 0xFFFFFFFFull);
    cand[j] = make_key(0u, id);
  }
  __syncthreads();

  // distances d(b, x) for every x in U
  const QueryRegs<KIND, VEC, NCH> Q = load_query<KIND, VEC, NCH>(T.base + (u64)b * T.row_bytes, T.npieces, lane);
  for (u32 base = 0; base < total; base += 64) {
    const u32 c64 = total - base < 64u ? total - base : 64u;
    const u64* cb = cand + base;
    const u32 dk = eval_up_to_64<KIND, VEC, NCH>(T, Q, [cb](u32 i) { return key_id(cb[i]); }, c64, lane);
    const u32 c = cand_of_lane(lane);
    const u32 id = c < c64 ? key_id(cb[c]) : 0u;
    __syncthreads();
    if (c < c64) cand[base + c] = make_key(dk, id) | (by_new && base + c >= clean ? 1ull : 0ull);
  }
  __syncthreads();

  u32 pair_evals = total;
  u32 kept;
  if (in_lds) {
    u32 n2 = 64;
    while (n2 < total) n2 <<= 1;
    for (u32 j = total + lane; j < n2; j += 64) cand[j] = KEY_INF;
    __syncthreads();
    bitonic_sort_keys(cand, n2, lane);
    bool done = false;
    if constexpr (kMfma) {
      if (MfmaPruneOk<KIND, VEC, NCH>::always || a.use_mfma) {
        kept = prune_sorted_mfma<KIND, VEC, NCH>(T, M, cand, total, a.R, a.a16, out, lane, pair_evals);
        done = true;
      }
    }
    if constexpr (kF32 && CAP == MERGE_MEDIUM_MAX) {
      if (by_new) {
        kept = reprune_new_f32<KIND, NCH>(T, F, T.base + (u64)b * T.row_bytes, cand, total, a.R, a.af, row, lane);
        if (lane == 0) a.meta[b] = make_meta(kept, kept);
        __syncthreads();
        ++stats.rep;
        stats.edges += cnt;
        stats.pair += (unsigned long long)total * (total - clean + 1u);
        return;
      }
    }
    if constexpr (kF32)
      kept = prune_sorted_f32<KIND, VEC, NCH>(T, F, T.base + (u64)b * T.row_bytes, cand, total, a.R, a.af, out, lane, pair_evals);
    else if constexpr (!MfmaPruneOk<KIND, VEC, NCH>::always)
      if (!done) kept = prune_sorted<KIND, VEC, NCH>(T, st, blk, cand, total, a.R, al, out, lane, pair_evals);
  } else {
    // (the staged-vector areas are laid out for the walk in use; the minimum-search walk reads
    // the selected vectors from device memory when the matrix-core layout is active)
    SelStage st2 = st;
    if (a.use_mfma) st2.vec = nullptr;
    kept = prune_unsorted<KIND, VEC, NCH>(T, st2, cand, total, a.R, al, out, lane, pair_evals);
  }
  __syncthreads();
  for (u32 j = lane; j < a.R; j += 64) row[j] = j < kept ? out[j] : NONE_ID;
  if (lane == 0) a.meta[b] = make_meta(kept, kept);
  __syncthreads();
  ++stats.rep;
  stats.edges += cnt;
  stats.pair += pair_evals;
}

template <int KIND, int VEC, int NCH, u32 CAP>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(KindTraits<KIND>::is_int && NCH == 2 ? 2 : 1))) void merge_generic_kernel(MergeArgs a, VecTable T) {
  __shared__ u64 cand_lds[CAP];
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x;
  const u32 nitems = a.list_count[CAP == MERGE_SPILL_MIN ? 2 : 3];
  MergeStats stats;
  for (u32 it = blockIdx.x; it < nitems; it += gridDim.x) merge_generic_one<KIND, VEC, NCH, CAP>(a, T, cand_lds, smem, it, lane, stats);
  stats.add(a, lane);
}

// All three kinds in one launch, for batches with few segments: three launches one after the other take 24 us in a batch
// of 200 points, this one 14.  A workgroup has the LDS and the registers of the largest kind: with the buffer of 4,096 keys
// three share a compute unit, with that of 512 (CAP; longer lists have a launch of their own) eight, or five on rows
// above 128 bytes, whose gram buffers are 32 KB.  The fast kind needs neither and has its own launch (launches == 3) where its
// items are many.  The longest lists first; merge_launches says where this pays.
template <int KIND, int VEC, int NCH, u32 CAP>
__global__ __launch_bounds__(64) void merge_all_kernel(MergeArgs a, VecTable T) {
  if constexpr (KindTraits<KIND>::is_int && SmallPathOk<VEC, NCH>::value) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x;
    const u32 nfast = a.launches == 3 ? 0u : a.list_count[0], ngram = a.list_count[1], nlong = a.list_count[CAP == MERGE_SPILL_MIN ? 2 : 3];
    MergeStats stats;
    for (u32 it = blockIdx.x; it < nlong + ngram + nfast; it += gridDim.x) {
      if (it < nlong)
        merge_generic_one<KIND, VEC, NCH, CAP>(a, T, reinterpret_cast<u64*>(smem), smem + CAP * 8u, it, lane, stats);
      else if (it < nlong + ngram)
        merge_gram_one<KIND, VEC, NCH>(a, T, *reinterpret_cast<GramLds<NCH>*>(smem), it - nlong, lane, stats);
      else
        merge_fast_one<KIND, VEC, NCH>(a, T, *reinterpret_cast<FastLds<NCH>*>(smem), it - nlong - ngram, lane, stats);
      __syncthreads();
    }
    stats.add(a, lane);
  }
}
template <int KIND, int VEC, int NCH, u32 CAP>
static hipError_t launch_merge_all(const MergeArgs& a, const VecTable& T, u32 grid, u32 lds, hipStream_t s) {
  u32 all = CAP * 8u + lds;
  all = all > sizeof(GramLds<NCH>) ? all : (u32)sizeof(GramLds<NCH>);
  const auto kernel = merge_all_kernel<KIND, VEC, NCH, CAP>;
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)all);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(64), all, s, a, T);
  return hipGetLastError();
}

// The three kernels work on disjoint rows, so they may run side by side: s_gram and s_generic are
// side streams the caller has already made wait for the planning kernel.
template <int KIND, int VEC, int NCH>
static hipError_t launch_merge_t(const MergeArgs& a, const VecTable& T, u32 grid, hipStream_t s, hipStream_t s_gram,
                                 hipStream_t s_generic, hipStream_t s_medium) {
  // the generic kernel's few, long items first, so that they start at once instead of waiting
  // for LDS that the other two kernels' workgroups hold; a small grid serves its short list
  const u32 lds = F32PruneOk<KIND, VEC, NCH>::value ? f32_lds_bytes(a.R, T.npieces)
                  : a.use_mfma ? ((a.R * 4u + 15u) & ~15u) + mfma_lds_bytes(a.R, T.row_bytes)
                            : ((a.R * 8u + 15u) & ~15u) + 8u * stage_stride(T.row_bytes) + 32u + a.stage_bytes;
  if constexpr (KindTraits<KIND>::is_int && SmallPathOk<VEC, NCH>::value) {
    if (a.launches == 1)
      return launch_merge_all<KIND, VEC, NCH, MERGE_SPILL_MIN>(a, T, grid < 1024u ? grid : 1024u, lds, s);
    if (a.launches >= 2) {
      hipLaunchKernelGGL((merge_generic_kernel<KIND, VEC, NCH, MERGE_SPILL_MIN>), dim3(grid < 1024u ? grid : 1024u), dim3(64), lds, s, a, T);
      const hipError_t e = launch_merge_all<KIND, VEC, NCH, MERGE_MEDIUM_MAX>(a, T, grid < 4096u ? grid : 4096u, lds, s);
      if (a.launches == 2 || e != hipSuccess) return e;
      hipLaunchKernelGGL((merge_fast_kernel<KIND, VEC, NCH>), dim3(grid), dim3(64), 0, s, a, T);
      return hipGetLastError();
    }
  }
  const u32 grid_generic = (grid < 1024u || a.force_prune) ? grid : 1024u;
  hipLaunchKernelGGL((merge_generic_kernel<KIND, VEC, NCH, MERGE_SPILL_MIN>), dim3(grid_generic), dim3(64), lds,
                     s_generic, a, T);
  if (a.medium_max)
    hipLaunchKernelGGL((merge_generic_kernel<KIND, VEC, NCH, MERGE_MEDIUM_MAX>), dim3(grid), dim3(64), lds, s_medium, a,
                       T);
  // the caller's stream takes the kernel that usually ends last, so that its waits for the other
  // two streams are already satisfied when it reaches them
  if (a.gram_ok) {
    hipLaunchKernelGGL((merge_fast_kernel<KIND, VEC, NCH>), dim3(grid), dim3(64), 0, s_gram, a, T);
    hipLaunchKernelGGL((merge_gram_kernel<KIND, VEC, NCH>), dim3(grid), dim3(64), 0, s, a, T);
  } else {
    hipLaunchKernelGGL((merge_fast_kernel<KIND, VEC, NCH>), dim3(grid), dim3(64), 0, s, a, T);
  }
  return hipGetLastError();
}

hipError_t launch_merge(const DistCfg& cfg, const MergeArgs& a, u32 grid, hipStream_t s, hipStream_t s_gram,
                        hipStream_t s_generic, hipStream_t s_medium) {
  if (grid == 0) return hipSuccess;
  VecTable T{a.points, (u32)cfg.row_bytes, cfg.npieces};
  ANN_DISPATCH_CFG(launch_merge_t, a, T, grid, s, s_gram, s_generic, s_medium);
}

// Batches of byte rows whose re-prunes go in one launch, in two, or in three (two and the fast kind), on one stream; in larger
// ones each kind has a launch, and from 2,048 points on a stream.  What counts is how many rows there are to prune, four to
// five per point, and of what kind: the fast ones want many waves per compute unit (joined, they get eight or five), the longest
// lists want the 512-key buffer.  Whole builds, each kind apart / in one launch / in two / in three:
//  - rows of up to 128 bytes, uint8 and int8 of 128 at R = 40: batches of 1,020 points 10.2 / 9.6 / 9.8 / 10.2 ms and
//    12.0 / 11.7 / 10.8 / 11.1; 2,800 14.2 / - / 13.2 / 13.6 and 17.1 / - / 17.2 / 17.0; 4,000 17.5 / - / 17.0 / 17.0 and
//    21.9 / - / 23.7 / 22.9 (at R = 104 46.1 / - / 39.1 / 38.0); 5,200 19.9 / - / 19.9 / 19.6 and 25.8 / - / 29.7 / 28.3.
//  - rows of up to 256 bytes (256 registers), uint8 of 200 and int8 of 256 at R = 48 and 64: batches of 400 points 9.1 / 8.4 / 8.6
//    / 9.0, 14.9 / 13.9 / 14.0 / 14.5 and 10.8 / 10.1 / 9.6 / 9.8, 16.7 / 16.7 / 15.5 / 15.6; 1,000 11.2 / 10.1 / 10.2 / 10.7, 17.8 /
//    16.7 / 16.5 / 16.8 and 14.4 / 15.4 / 13.5 / 13.1, 22.1 / 25.3 / 22.2 / 21.1; 1,700 13.4 / - / 11.9 / 12.4, 20.0 / -
//    / 18.4 / 18.8 and 18.7 / - / 19.3 / 17.4, 27.3 / - / 29.2 / 26.3; 2,500 15.3 / - / 14.9 / 14.8, 22.3 / - / 21.2 / 21.6 and 21.9 / -
//    / 28.0 / 24.0, 31.6 / - / 38.0 / 32.9 (int8 of 140: 17.8 / - / 19.0 / 17.9, 29.1 / - / 31.6 / 29.6);
//    3,200 17.8 / - / 18.5 / 17.8 and 25.4 / - / 33.1 / 27.6.
u32 merge_launches(const DistCfg& cfg, u64 batch) {
  if (!gram_path_ok(cfg)) return 0;
  if (cfg.nch == 1) return batch <= 1024u ? 1 : batch <= 3072u ? 2 : batch <= 4096u ? 3 : 0;
  return batch <= 512u ? 1 : batch <= 1536u ? 2 : batch <= 2560u ? 3 : 0;
}

bool gram_path_ok(const DistCfg& cfg) { return cfg.kind <= 1 && 8 * cfg.nch * cfg.vec <= 256; }
u32 gram_path_tmax() { return SM_TMAX; }
bool mfma_prune_ok(u32 R, const DistCfg& cfg) {
  return cfg.kind <= 1 && 8 * cfg.nch * cfg.vec <= 256 && mfma_lds_bytes(R, (u32)cfg.row_bytes) <= MFMA_LDS_MAX;
}
u32 prune_stage_bytes(u32 R, const DistCfg& cfg) { return cfg.kind <= 1 ? stage_bytes(R, (u32)cfg.row_bytes, STAGE_BUDGET) : 0u; }
u32 fast_path_amax(const DistCfg& cfg) { return cfg.nch <= 2 ? 4u : (cfg.nch <= 4 ? 2u : 1u); }

// rows given from outside: degree from the row itself, no clean prefix known
__global__ __launch_bounds__(256) void meta_from_rows_kernel(const u32* graph, u64 n, u32 R, u32* meta) {
  const u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const u32* row = graph + i * R;
  u32 deg = 0;
  while (deg < R && row[deg] != NONE_ID) ++deg;
  meta[i] = make_meta(deg, 0u);
}
__global__ __launch_bounds__(256) void meta_forget_clean_kernel(u64 n, u32* meta) {
  const u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) meta[i] &= 0xFFFFu;
}

hipError_t launch_meta_from_rows(const u32* graph, u64 n, u32 R, u32* meta, hipStream_t s) {
  hipLaunchKernelGGL(meta_from_rows_kernel, dim3((u32)((n + 255) / 256)), dim3(256), 0, s, graph, n, R, meta);
  return hipGetLastError();
}
hipError_t launch_meta_forget_clean(u64 n, u32* meta, hipStream_t s) {
  hipLaunchKernelGGL(meta_forget_clean_kernel, dim3((u32)((n + 255) / 256)), dim3(256), 0, s, n, meta);
  return hipGetLastError();
}

}  // namespace annmi
