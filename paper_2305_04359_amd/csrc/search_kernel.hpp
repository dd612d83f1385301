// Batched greedy beam search, one wavefront per search (Alg. 1 of the paper).
//
// The beam (at most L candidates ordered by (distance, id), each with a "processed" flag) lives
// in registers, striped over the wave: entry i is held by lane i % 64 in slot i / 64.  LDS is the
// exchange medium when new candidates are merged in.  The visited filter of Sec. 4.5 (a lossy
// hash of vertex ids with one-sided error) is a per-wave LDS table of 16-byte buckets, newest
// entry first: a lost entry only causes a repeated distance evaluation, and the repeated
// candidate is then recognised as a duplicate of a beam entry or is worse than the beam's last
// entry, so results do not depend on the table.  A bucket holds four 32-bit ids, or, when the
// vertex count allows, eight 16-bit or six 21-bit tags: the id is passed through a bijection y
// of its B bits, bucket = floor(y * buckets / 2^B) (from the top 24 bits of y), tag = the low
// B - floor(log2 buckets) bits of y (at most 15, or 20).  Two ids of one bucket differ by less
// than 2^B / buckets in y, so equal tags mean equal ids: a tag match still identifies the vertex
// exactly while the table remembers up to twice as many vertices.  The bucket count need not be
// a power of two; it is chosen so that the wave's LDS lands on an occupancy step.
#pragma once
#include <atomic>
#include <cstddef>
#include <type_traits>

#include "ann_device.hpp"
#include "ann_internal.hpp"
#include "sketch.hpp"
#include "wave_sort.hpp"

namespace annmi {

// a bijection of the low `bits` bits: multiplication by an odd constant modulo 2^bits (its top
// bits, which choose the bucket, depend on all bits of x); the 24-bit multiply serves ids of at
// most 24 bits
__device__ __forceinline__ u32 mix_id(u32 x, u32 mask, u32 bits) {
  return (bits <= 24u ? (u32)__umul24(x, 0x9E3779u) : x * 0x9E3779B1u) & mask;
}

// high 16 bits of the 48-bit product of two 24-bit numbers (both operands in vector registers:
// nothing here reads a scalar register that a vector instruction may just have written)
__device__ __forceinline__ u32 umulhi24(u32 a, u32 b) {
  u32 r;
  asm("v_mul_hi_u32_u24 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

typedef unsigned short us2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u32 pk_min_u16(u32 a, u32 b) {
  return __builtin_bit_cast(u32, __builtin_elementwise_min(__builtin_bit_cast(us2_t, a), __builtin_bit_cast(us2_t, b)));
}

// The key no candidate may reach to enter a beam of L entries of which `size` are taken.  (FLAGS:
// the low bits of a beam entry that are no part of its key.)
template <int NSLOT, u64 FLAGS>
__device__ __forceinline__ u64 beam_worst(const u64 (&A)[NSLOT], u32 L, u32 size) {
  u64 worst = KEY_INF;
  if (size == L) {
#pragma unroll
    for (int s = 0; s < NSLOT; ++s)
      if ((int)((L - 1) >> 6) == s) worst = readlane_u64(A[s], (int)((L - 1) & 63)) | FLAGS;
  }
  return worst;
}

// the wave's keys moved down by one lane: lane l gets lane l + 1's, lane 63 gets `top`
__device__ __forceinline__ u64 shift_down_one(u64 k, u64 top) {
  const u32 lo = (u32)__builtin_amdgcn_update_dpp((int)(u32)top, (int)(u32)k, 0x130, 0xF, 0xF, false);
  const u32 hi = (u32)__builtin_amdgcn_update_dpp((int)(u32)(top >> 32), (int)(u32)(k >> 32), 0x130, 0xF, 0xF, false);
  return ((u64)hi << 32) | lo;
}

// beam <- the L closest of the beam and `ns` survivors (KEY_INF in the other lanes), by a sorting
// network: the smaller of each pair (entry of the beam's last slot, survivor in descending order),
// then a merge.  LAST_ROW: the survivors are in lanes 48 to 63.  False, and the beam unchanged, if
// a survivor is in the beam already (the filter lost it): it then stands next to the entry it repeats,
// in the beam or at its end.
template <int NSLOT, u64 FLAGS, bool LAST_ROW>
__device__ __forceinline__ bool insert_sorted(u64 (&A)[NSLOT], u64 survivor, u32 ns, u32 L, u32& size, int lane) {
  u64 B[NSLOT];
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) B[s] = A[s];
  u64 v[1] = {survivor};
  if constexpr (LAST_ROW)
    BitonicStage<1, 2, false, 16>::run(v);  // the rows of odd number end in descending order
  else
    BitonicStage<1, 2, true, 64>::run(v);
  const u64 last = B[NSLOT - 1];
  const bool keep = last < v[0];
  const u64 out = keep ? v[0] : last;
  B[NSLOT - 1] = keep ? last : v[0];
  bitonic_merge<NSLOT>(B);
  u64 next_first = KEY_INF;  // the smallest key of the next slot, for lane 63
  bool dup = false;
#pragma unroll
  for (int s = NSLOT - 1; s >= 0; --s) {
    const u64 up = shift_down_one(B[s], next_first);
    dup = dup || (B[s] != KEY_INF && (up | FLAGS) == (B[s] | FLAGS));
    next_first = readlane_u64(B[s], 0);
  }
  const u64 end = readlane_u64(B[NSLOT - 1], 63);
  dup = dup || (out != KEY_INF && (out | FLAGS) == (end | FLAGS));
  if (ballot(dup) != 0) return false;
  size = size + ns < L ? size + ns : L;
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) A[s] = (u32)(s * 64 + lane) < size ? B[s] : KEY_INF;
  return true;
}

// beam <- the L closest of the beam and the lanes' candidates (KEY_INF: none); returns how many
// candidates were below the beam's last entry and not in the beam already.  Called by one whole
// wave; `sync` orders its LDS accesses before and after against each other.
//
// NETWORK: from 20 survivors on they go in by the sorting network (search_network says when).  With
// the chip full it takes as many vector instructions as ranks by bisection and counting at 45
// survivors of a two-slot beam, at 20 of a one-slot beam.
template <int NSLOT, bool NETWORK, class Sync>
__device__ __forceinline__ void beam_insert(u64 (&A)[NSLOT], u64* beam, u64* skeys, u64 mykey, u32 L, u32& size,
                                            u32& n_surv, u32& n_ins, int lane, Sync sync) {
  constexpr u64 FLAGS = 1;
  const u64 worst = beam_worst<NSLOT, FLAGS>(A, L, size);
  bool surv = mykey < worst;
  u64 sm = ballot(surv);
  if (NETWORK && __builtin_popcountll(sm) >= 20) {
    const u32 ns = (u32)__builtin_popcountll(sm);
    if (insert_sorted<NSLOT, FLAGS, false>(A, surv ? mykey : KEY_INF, ns, L, size, lane)) {
#pragma unroll
      for (int s = 0; s < NSLOT; ++s) beam[s * 64 + lane] = A[s];
      sync();
      n_surv += ns;
      ++n_ins;
      return;
    }
  }
  if (sm) {
    u32 myrA = 0, myrB = 0, ns = 0;
    u32 shift[NSLOT];
#pragma unroll
    for (int s = 0; s < NSLOT; ++s) shift[s] = 0;
    if (__builtin_popcountll(sm) >= 4) {
      // many survivors: each finds its rank among the beam entries by bisection in the LDS
      // copy of the beam; a survivor that is already in the beam (the filter lost it) sits
      // exactly at its rank there and is dropped
      // the rank is at most 64 * NSLOT - 1 (a survivor lies below the last entry of a full
      // beam): one step per bit of it, each keeping the bit if that many entries lie below
      // the key; entries past `size` are never counted (the read stays inside the array)
      constexpr int BITS = (NSLOT == 1 ? 6 : NSLOT == 2 ? 7 : NSLOT == 4 ? 8 : NSLOT == 8 ? 9 : NSLOT == 16 ? 10 : 11);
      const u64 sk1 = mykey | FLAGS;
      u32 lo = 0;
#pragma unroll
      for (int bit = BITS - 1; bit >= 0; --bit) {
        const u32 t = lo + (1u << bit);
        const u64 v = beam[t - 1u] | FLAGS;
        lo = (t <= size && v < sk1) ? t : lo;
      }
      myrA = lo;
      if (surv && lo < size && (beam[lo] | FLAGS) == sk1) surv = false;
      sm = ballot(surv);
      ns = (u32)__builtin_popcountll(sm);
      if (surv) skeys[__builtin_popcountll(sm & lanemask_lt(lane))] = mykey;
      sync();
      // ranks among the survivors, and how far each beam entry moves
      // (a lane without a survivor counts too: its sum is never read)
      for (u32 j = 0; j < ns; ++j) {
        const u64 sj = skeys[j];
        myrB += (sj < mykey) ? 1u : 0u;
#pragma unroll
        for (int s = 0; s < NSLOT; ++s) shift[s] += (sj < A[s]) ? 1u : 0u;
      }
      sync();
    } else {
      // few survivors: one at a time, ranks from wave-wide compares
      for (u64 it = sm; it; it &= it - 1) {
        const int l = __builtin_ctzll(it);
        const u64 sk = readlane_u64(mykey, l);
        u32 rA = 0;
#pragma unroll
        for (int s = 0; s < NSLOT; ++s) rA += __builtin_popcountll(ballot(A[s] < sk));
        u64 at = KEY_INF;
#pragma unroll
        for (int s = 0; s < NSLOT; ++s)
          if ((int)(rA >> 6) == s) at = readlane_u64(A[s], (int)(rA & 63));
        const bool dup = (at | FLAGS) == (sk | FLAGS);
        if (lane == l) {
          myrA = rA;
          if (dup) surv = false;
        }
      }
      sm = ballot(surv);
      for (u64 it = sm; it; it &= it - 1) {
        const int l = __builtin_ctzll(it);
        const u64 sk = readlane_u64(mykey, l);
        const u32 rB = __builtin_popcountll(ballot(surv && mykey < sk));
#pragma unroll
        for (int s = 0; s < NSLOT; ++s) shift[s] += (sk < A[s]) ? 1u : 0u;
        if (lane == l) myrB = rB;
        ++ns;
      }
    }
    if (sm) {
#pragma unroll
      for (int s = 0; s < NSLOT; ++s) {
        const u32 np = (u32)(s * 64 + lane) + shift[s];
        if (A[s] != KEY_INF && np < L) beam[np] = A[s];
      }
      if (surv) {
        const u32 np = myrA + myrB;
        if (np < L) beam[np] = mykey;
      }
      n_surv += ns;
      ++n_ins;
      size = size + ns < L ? size + ns : L;
      sync();
#pragma unroll
      for (int s = 0; s < NSLOT; ++s) {
        const u32 idx = (u32)(s * 64 + lane);
        A[s] = idx < size ? beam[idx] : KEY_INF;
      }
      sync();
    }
  }
}

// An entry pk of the beam is beyond the bound that its k-th entry kk sets.
// Integers: d * 2^16 > d_k * (2^16 + eps16), exact; floats: d > d_k + eps * |d_k|, one fp32
// product and one fp32 sum.
template <int KIND>
__device__ __forceinline__ bool beyond_eps(u64 pk, u64 kk, const SearchArgs& a) {
  if constexpr (KindTraits<KIND>::is_int) {
    const long long d = int_from_dkey(key_dkey(pk)), dk = int_from_dkey(key_dkey(kk));
    return d * 65536ll > dk * (65536ll + a.eps16);
  } else {
    const float d = float_from_dkey(key_dkey(pk)), dk = float_from_dkey(key_dkey(kk));
    return d > __fadd_rn(dk, __fmul_rn(a.epsf, __builtin_fabsf(dk)));
  }
}
// entry i of the beam (wave-uniform)
template <int NSLOT>
__device__ __forceinline__ u64 beam_entry(const u64 (&A)[NSLOT], u32 i) {
  u64 k = 0;
#pragma unroll
  for (int s = 0; s < NSLOT; ++s)
    if ((int)(i >> 6) == s) k = readlane_u64(A[s], (int)(i & 63u));
  return k;
}

// Stands at the end of a branch that some lanes take, where uniform branches around it end too.  Without
// it the compiler lets all of them end in one place, and takes a value that differs between the
// uniform paths to that place (a list's pointer, a count) for one that differs between lanes: it, the
// branches it decides and in the end the state of the loop then live in vector registers and
// execution masks.
__device__ __forceinline__ void keep_join() { __builtin_amdgcn_wave_barrier(); }

// Entry nv of search qi's visited list.  (vptr, vcap) are wave-uniform; vptr turns null when the
// list is lost (it fits neither its slot nor a spill chunk: the prune kernel sees nv > room and
// reports it).
__device__ __forceinline__ void visited_append(const SearchArgs& a, u32 qi, u64*& vptr, u32& vcap, u32 nv, u64 pk,
                                               int lane) {
  if (vptr == nullptr) return;
  if (nv == vcap) {  // the list is full
    u64* moved = nullptr;
    u32 newcap = 0;
    if (vcap == a.vis_cap && a.spill != nullptr) {  // still in its slot: move to a spill chunk
      const u64 need = (u64)vcap + a.spill_chunk;
      unsigned long long off = 0;
      if (lane == 0) off = atomicAdd(a.spill_top, (unsigned long long)need);
      off = readlane_u64(off, 0);
      if (off + need <= a.spill_cap) {
        __threadfence();
        u64* dst = a.spill + off;
        for (u32 i = lane; i < vcap; i += 64)
          dst[i] = __hip_atomic_load(vptr + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (lane == 0) a.vis_where[qi] = off;
        moved = dst;
        newcap = (u32)need;
      }
    }
    vptr = reinterpret_cast<u64*>(readlane_u64(reinterpret_cast<u64>(moved), 0));
    vcap = readlane_u32(newcap, 0);
  }
  if (vptr != nullptr && lane == 0) vptr[nv] = pk;
  keep_join();
}

// The first k entries of the beam as search qi's results.
template <int KIND, int NSLOT>
__device__ __forceinline__ void write_results(const u64 (&A)[NSLOT], const SearchArgs& a, u32 qi, int lane) {
  if (a.out_ids == nullptr) return;
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) {
    const u32 idx = (u32)(s * 64 + lane);
    if (idx < a.k) {
      const bool ok = A[s] != KEY_INF;
      const u64 o = (u64)qi * a.k + idx;
      a.out_ids[o] = ok ? key_id(A[s]) : NONE_ID;
      if (a.out_dists != nullptr) {
        if constexpr (KindTraits<KIND>::is_int)
          reinterpret_cast<i32*>(a.out_dists)[o] = ok ? int_from_dkey(key_dkey(A[s])) : 0x7FFFFFFF;
        else
          reinterpret_cast<float*>(a.out_dists)[o] = ok ? float_from_dkey(key_dkey(A[s])) : __builtin_inff();
      }
    }
  }
}

// the words of a batch's counters that the steps after the searches count in
__device__ __forceinline__ void zero_batch_counters(u32* c) {
  c[0] = 0;
  c[4] = 0;
  c[5] = 0;
  c[8] = 0;
  c[9] = 0;
  c[10] = 0;
  c[11] = 0;
}

// The query of a search in registers, or (SK > 0) in LDS.
template <int KIND, int VEC, int NCH>
struct SearchQuery : QueryRegs<KIND, VEC, NCH> {
  __device__ __forceinline__ SearchQuery(const QueryRegs<KIND, VEC, NCH>& Q, Piece<VEC>*, int)
      : QueryRegs<KIND, VEC, NCH>(Q) {}
};
template <int KIND, int VEC, int NCH>
struct SearchQueryLds {
  const Piece<VEC>* mine;
  __device__ __forceinline__ SearchQueryLds(const QueryRegs<KIND, VEC, NCH>& Q, Piece<VEC>* lds, int lane) {
    if (lane < LPC) {
#pragma unroll
      for (int u = 0; u < NCH; ++u) lds[LPC * u + lane] = Q.q[u];
    }
    __syncthreads();
    mine = lds + (lane & (LPC - 1));
  }
  static constexpr bool in_lds = true;
  __device__ __forceinline__ Piece<VEC> piece(int u) const { return mine[LPC * u]; }
};

// EPS: the (1 + eps) rule is compiled in.  TAG16: the filter holds 16-bit tags (graphs of up to
// a few million points); the other two layouts share the second variant, so that their code does
// not weigh on the registers of the first.
// OWN: every search has a start vertex of its own and reports the closest vertex it found (the
// layered index); compiled apart so that the flat graph's searches do not carry its arguments.
// NETWORK: see beam_insert.
// SK: 16-byte pieces per lane of the vertices' sketches (0: there are none).  Once the beam is full, a row's
// candidates whose sketch puts them certainly beyond the beam's last entry are dropped unread.
template <int KIND, int VEC, int NCH, int NSLOT, bool EPS, bool TAG16, bool OWN, bool NETWORK>
__global__ __launch_bounds__(64) void search_kernel(SearchArgs a, VecTable T) {
  constexpr int SK = 0;
  constexpr SketchTable K{};
#include "search_body.inc"
}

// On rows with sketches.  A search waits for memory 70 % of its time, so registers go to waves: the query and
// its planes live in LDS (read once per pass of 8 to 32 candidates), and the bound keeps the compiler from spending the
// registers again.  200 floats: four waves with the query in registers 198 ms a build, five 188; a sixth would spill.
constexpr int sketch_waves(int NCH) { return NCH <= 4 ? 6 : NCH <= 7 ? 5 : 4; }
template <int KIND, int NCH, int NSLOT, bool EPS, bool TAG16, bool OWN, bool NETWORK, int SK>
__global__ __launch_bounds__(64, sketch_waves(NCH)) void search_sketch_kernel(SearchArgs a, VecTable T, SketchTable K) {
  constexpr int VEC = 16;
#include "search_body.inc"
}

// launches of the variants that other translation units compile: with the (1 + eps) rule
// (search_eps.hip), with start vertices of their own (search_own.hip), with both (search_own_eps.hip)
hipError_t launch_search_eps(const DistCfg& cfg, const SearchArgs& a, const VecTable& T, hipStream_t s, SearchPlan* plan);
hipError_t launch_search_own(const DistCfg& cfg, const SearchArgs& a, const VecTable& T, hipStream_t s, SearchPlan* plan);
hipError_t launch_search_own_eps(const DistCfg& cfg, const SearchArgs& a, const VecTable& T, hipStream_t s, SearchPlan* plan);
// the same on rows with sketches (sketch.hip, sketch_eps.hip, sketch_own.hip)
hipError_t launch_search_sketch(const DistCfg& cfg, const SearchArgs& a, const VecTable& T, hipStream_t s);
hipError_t launch_search_sketch_eps(const DistCfg& cfg, const SearchArgs& a, const VecTable& T, hipStream_t s);
hipError_t launch_search_sketch_own(const DistCfg& cfg, const SearchArgs& a, const VecTable& T, hipStream_t s);
// the filter's size and layout for an instance whose registers leave room for `waves` waves per SIMD (search.hip)
void search_set_filter(SearchArgs& a, u32 waves, u32 lds_more = 0);
// Several waves per search (search_wide.hip): rows of at most 64 ids, beams of at most 256, ids of
// at most 24 bits (beam entries and the 16-bit tags of a filter of 512 buckets).
constexpr u32 WIDE_BUCKETS = 512;
constexpr u64 WIDE_MAX_POINTS = 1ull << 24;
hipError_t launch_search_wide(const DistCfg& cfg, const SearchArgs& a, const VecTable& T, u32 waves, hipStream_t s);
// One wave per search with the next hops' memory requested ahead (search_ahead.hip): byte rows, rows of at
// most 64 ids, beams of at most 128, ids that 16-bit tags of a filter of AHEAD_BUCKETS hold.
constexpr u32 AHEAD_BUCKETS = 480;
constexpr u64 AHEAD_MAX_POINTS = 1ull << 23;
hipError_t launch_search_ahead(const DistCfg& cfg, const SearchArgs& a, const VecTable& T, hipStream_t s);

// beam slots per lane: the smallest power of two that holds L entries (beams of up to 2,048)
inline u32 search_nslot_for(u32 L) {
  u32 ns = 1;
  while (ns * 64u < L && ns < 32u) ns *= 2u;
  return ns;
}

// Whether searches with one-slot beams carry the sorting network.  It pays where 20 survivors of one
// row are common: long rows, or a beam that is still filling (10,000 uint8 queries, a million points,
// R = 64: 182 -> 174 us at L = 16, 416 -> 410 at L = 64; 200,000 points, R = 48: 183 -> 176 at L = 16,
// 385 -> 394 at L = 64).  Rows of 32 ids never repay the second path that the loop then holds (20,000
// uint8 points, 40,000 queries at L = 64: 753 -> 780 us; 48 floats, 2,000 queries: 151 -> 157).
// In the float variants with start vertices of their own, rows of up to 64 elements, it would also
// cost the wave per SIMD that they hold at 64 registers.
template <int KIND, int NCH, bool OWN>
constexpr bool search_network_compiled = !(OWN && !KindTraits<KIND>::is_int && NCH <= 2);
// The second path is repaid all the same where the searches are few and wait for their own chains, of
// which the network's is the shorter (56,000 uint8 points, R = 32, 7 queries at L = 18, eps = 0.25: 36.5 ->
// 34.3), and with the (1 + eps) rule, where a search ends soon after its beam has filled (341,000 uint8
// points, R = 48, 2,698 queries at L = 34, eps = 0.05: 115.5 -> 109.6).
inline bool search_network(const SearchArgs& a) {
  return a.R >= 64u || (a.R > 32u && (a.L <= 24u || a.eps16 >= 0)) || a.nq <= 256u;
}

// Waves per SIMD that the registers of one instance leave room for (0: the runtime does not say), asked for once.
template <int KIND, int VEC, int NCH, int NSLOT, bool EPS, bool TAG16, bool OWN, bool NETWORK, int SK = 0>
inline u32 search_instance_waves() {
  static std::atomic<u32> known{0};
  u32 waves = known.load(std::memory_order_relaxed);
  if (waves == 0) {
    hipFuncAttributes f{};
    const void* kernel;
    if constexpr (SK > 0)
      kernel = reinterpret_cast<const void*>(search_sketch_kernel<KIND, NCH, NSLOT, EPS, TAG16, OWN, NETWORK, SK>);
    else
      kernel = reinterpret_cast<const void*>(search_kernel<KIND, VEC, NCH, NSLOT, EPS, TAG16, OWN, NETWORK>);
    if (hipFuncGetAttributes(&f, kernel) != hipSuccess || f.numRegs < 1) return 0;
    waves = 512u / (((u32)f.numRegs + 7u) & ~7u);  // 512 registers per lane and SIMD, in units of 8
    waves = waves > 8u ? 8u : waves < 1u ? 1u : waves;
    known.store(waves, std::memory_order_relaxed);
  }
  return waves;
}

template <int KIND, int VEC, int NCH, int NSLOT, bool EPS, bool OWN, bool NETWORK, int SK = 0>
inline hipError_t launch_search_instance(SearchArgs a, const VecTable& T, hipStream_t s, SearchPlan* plan) {
  constexpr u32 more = SK > 0 ? LPC * (NCH + 2 * SK) * VEC : 0;  // LDS beside that of every search: the query and its planes
  // (the size decides whether 16-bit tags do, and with them the instance)
  u32 waves = search_instance_waves<KIND, VEC, NCH, NSLOT, EPS, true, OWN, NETWORK, SK>();
  if (waves != 0) search_set_filter(a, waves, more);
  if (waves != 0 && a.tag_width != 16u) {
    waves = search_instance_waves<KIND, VEC, NCH, NSLOT, EPS, false, OWN, NETWORK, SK>();
    if (waves != 0) search_set_filter(a, waves, more);
  }
  if (waves == 0) return hipErrorInvalidDeviceFunction;
  if (plan != nullptr) {
    *plan = SearchPlan{waves, 4u * a.hash_buckets, a.tag_width};
    return hipSuccess;
  }
  const u32 lds = search_lds_bytes(a.L, a.hash_buckets) + more;
  const dim3 grid(a.nq), block(64);
  if constexpr (SK > 0) {
    const SketchTable K{a.sketch};
    if (a.tag_width == 16u)
      hipLaunchKernelGGL((search_sketch_kernel<KIND, NCH, NSLOT, EPS, true, OWN, NETWORK, SK>), grid, block, lds, s, a, T, K);
    else
      hipLaunchKernelGGL((search_sketch_kernel<KIND, NCH, NSLOT, EPS, false, OWN, NETWORK, SK>), grid, block, lds, s, a, T, K);
  } else if (a.tag_width == 16u) {
    hipLaunchKernelGGL((search_kernel<KIND, VEC, NCH, NSLOT, EPS, true, OWN, NETWORK>), grid, block, lds, s, a, T);
  } else {
    hipLaunchKernelGGL((search_kernel<KIND, VEC, NCH, NSLOT, EPS, false, OWN, NETWORK>), grid, block, lds, s, a, T);
  }
  return hipGetLastError();
}

// One launch for a fixed choice of EPS and OWN; the beam slots are picked here.
template <int KIND, int VEC, int NCH, bool EPS, bool OWN>
inline hipError_t launch_search_variant(const SearchArgs& a, const VecTable& T, hipStream_t s, SearchPlan* plan) {
  constexpr bool NETWORK = search_network_compiled<KIND, NCH, OWN>;
  switch (search_nslot_for(a.L)) {
    case 1:
      if (NETWORK && search_network(a)) return launch_search_instance<KIND, VEC, NCH, 1, EPS, OWN, NETWORK>(a, T, s, plan);
      return launch_search_instance<KIND, VEC, NCH, 1, EPS, OWN, false>(a, T, s, plan);
    case 2: return launch_search_instance<KIND, VEC, NCH, 2, EPS, OWN, false>(a, T, s, plan);
    case 4: return launch_search_instance<KIND, VEC, NCH, 4, EPS, OWN, false>(a, T, s, plan);
    case 8: return launch_search_instance<KIND, VEC, NCH, 8, EPS, OWN, false>(a, T, s, plan);
    case 16: return launch_search_instance<KIND, VEC, NCH, 16, EPS, OWN, false>(a, T, s, plan);
    default: return launch_search_instance<KIND, VEC, NCH, 32, EPS, OWN, false>(a, T, s, plan);
  }
}

// The same on rows with sketches (beams of up to SEARCH_SKETCH_BEAM).
template <int KIND, int NCH, int SK, bool EPS, bool OWN>
inline hipError_t launch_search_sketched(const SearchArgs& a, const VecTable& T, hipStream_t s) {
  switch (search_nslot_for(a.L)) {
    case 1:
      if (search_network(a)) return launch_search_instance<KIND, 16, NCH, 1, EPS, OWN, true, SK>(a, T, s, nullptr);
      return launch_search_instance<KIND, 16, NCH, 1, EPS, OWN, false, SK>(a, T, s, nullptr);
    case 2: return launch_search_instance<KIND, 16, NCH, 2, EPS, OWN, false, SK>(a, T, s, nullptr);
    default: return hipErrorInvalidConfiguration;
  }
}

}  // namespace annmi
