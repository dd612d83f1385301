// The beam search of search_kernel.hpp with several wavefronts per search, for launches of few
// searches.
//
// What bounds a lone search is its chain: every hop reads a row, then the vectors it names (two
// dependent trips to memory), and the next vertex is known only when the beam has been updated.
// But late in a search most hops insert nothing, so the vertices the next hops will expand are
// mostly in the beam already.  One workgroup of W waves therefore shares a search: the first wave
// runs it in the one-wave kernel's order, hop by hop, and whenever the other waves are idle it hands
// them the next W - 1 entries of the beam that have not been expanded.  They expand them ahead,
// one per wave: row, filter, distances, and of those the keys that could still enter the beam, left
// in an LDS list.  A list is offered to the beam only when its vertex's turn comes, so the hops,
// their order and every result are the one-wave kernel's; a vertex that falls out of the beam
// first has been expanded for nothing.  A vertex whose turn comes before anybody has taken it is
// expanded by the first wave itself.
//
// The filter: an expansion ahead may only enter a vertex that is settled for good, because a list
// that is never offered must not hide its vertices from later hops.  Settled are those at or
// beyond the last entry of a full beam (that entry never grows); the others enter when their list
// is offered, where those that another list brought first are dropped.  Waves update buckets side
// by side without atomics: a 32-bit word is written whole and holds two whole tags, and a tag that
// a lost update drops only costs a repeated evaluation.
//
// A beam entry is its key with the id moved up to make room for the entry's state:
// (distance) << 32 | id << 8 | state << 1 | processed.
#include "ann_dispatch.hpp"
#include "search_kernel.hpp"

namespace annmi {

constexpr u32 WIDE_MAX_WAVES = 8;
constexpr u32 WIDE_MAX_LISTS = 32;
constexpr u64 WIDE_FLAGS = 0xFF;
// states: not expanded; 1 + i: expanded into list i; STATE_TAKEN + i: being expanded into list i;
// expanded, and nothing could enter the beam (also what the empty slots of a beam read as)
constexpr u32 STATE_NEW = 0, STATE_TAKEN = 64, STATE_EMPTY = 127;

__device__ __forceinline__ u64 wide_key(u32 dkey, u32 id) { return ((u64)dkey << 32) | ((u64)id << 8); }
__device__ __forceinline__ u32 wide_id(u64 k) { return (u32)k >> 8; }
__device__ __forceinline__ u32 wide_state(u64 k) { return ((u32)k & 0xFFu) >> 1; }
__device__ __forceinline__ u64 plain_key(u64 k) { return make_key(key_dkey(k), wide_id(k)); }

// What the first wave tells the others.  `go` changes when there is work: (batch number) << 8 | how
// many waves it is for, or WIDE_STOP.  It is one word so that a wave without work in one batch,
// which nobody waits for, cannot take that batch's number with the next one's work.  The rest of a
// batch is written before `go` and stays until `done` has counted all its waves.
constexpr u32 WIDE_STOP = 0xFFFFFFFFu;
struct WideCtrl {
  u64 worst;                  // candidates at or beyond this key cannot enter the beam any more
  u64 key[WIDE_MAX_WAVES];    // the vertices to expand, as beam entries ...
  u32 list[WIDE_MAX_WAVES];   // ... and the list each one's candidates go to
  u32 count[WIDE_MAX_LISTS];  // length of every list
  u32 go;
  u32 done;
  u32 pad_[4];
};
static_assert(sizeof(WideCtrl) % 16 == 0, "the filter's 16-byte buckets lie behind it");
__device__ __forceinline__ u32 lds_acquire(const u32* p) {
  return readlane_u32(__hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP), 0);
}

// eight 16-bit tags per bucket, as in search_kernel.hpp
struct WideFilter {
  uint4* bucket;
  u32 id_bits, idmask, tagmask, yshl, nb8;
  __device__ __forceinline__ bool seen(u32 x, u32& h, u32& tag, uint4& e) const {
    const u32 y = mix_id(x, idmask, id_bits);
    h = umulhi24(y << yshl, nb8);
    tag = y & tagmask;
    const u32 tt = tag * 0x10001u;
    e = bucket[h];
    const u32 mz = pk_min_u16(pk_min_u16(e.x ^ tt, e.y ^ tt), pk_min_u16(e.z ^ tt, e.w ^ tt));
    return (mz & 0xFFFFu) == 0u || (mz >> 16) == 0u;
  }
  __device__ __forceinline__ bool seen(u32 x) const {
    u32 h, tag;
    uint4 e;
    return seen(x, h, tag, e);
  }
  // newest in front; false if the vertex was there
  __device__ __forceinline__ bool enter(u32 x) const {
    u32 h, tag;
    uint4 e;
    if (seen(x, h, tag, e)) return false;
    bucket[h] = make_uint4((e.x << 16) | tag, (e.y << 16) | (e.x >> 16), (e.z << 16) | (e.y >> 16),
                           (e.w << 16) | (e.z >> 16));
    return true;
  }
};

// orders a wave's own LDS accesses (the hardware keeps them in order; the compiler must, too)
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// beam_insert for a wave that runs alone: always the sorting network, whose cost hardly depends on the
// number of survivors (880 cycles for a one-slot beam and up to 16 survivors, in lanes 48 to 63,
// `last_row`; 1,400 for two slots; 600 more otherwise), where one to three survivors inserted one at
// a time take 700 to 2,000 cycles, and more of them by bisection 1,200 and 180 each, most of it LDS
// latency.
template <int NSLOT>
__device__ __forceinline__ u32 wide_insert(u64 (&A)[NSLOT], u64 mykey, bool last_row, u32 L, u32& size, int lane) {
  const u64 worst = beam_worst<NSLOT, WIDE_FLAGS>(A, L, size);
  if (mykey >= worst) mykey = KEY_INF;
  for (;;) {
    const u64 sm = ballot(mykey != KEY_INF);
    const u32 ns = (u32)__builtin_popcountll(sm);
    if (ns == 0u) return 0;
    if (last_row ? insert_sorted<NSLOT, WIDE_FLAGS, true>(A, mykey, ns, L, size, lane)
                 : insert_sorted<NSLOT, WIDE_FLAGS, false>(A, mykey, ns, L, size, lane))
      return ns;
    // some are in the beam already (the filter lost them): drop those
    bool dropped = false;
    for (u64 it = sm; it; it &= it - 1) {
      const int l = __builtin_ctzll(it);
      const u64 k = readlane_u64(mykey, l) | WIDE_FLAGS;
      bool same = false;
#pragma unroll
      for (int s = 0; s < NSLOT; ++s) same = same || (A[s] | WIDE_FLAGS) == k;
      if (ballot(same) != 0) {
        dropped = true;
        if (lane == l) mykey = KEY_INF;
      }
    }
    // A row named a vertex twice: drop all but its last, so that the loop ends whatever the rows hold.  (Apart
    // from the drop above, which is taken often: in it, the test cost 1 to 3 % of a search.)
    if (!dropped) {
      for (u64 it = sm; it; it &= it - 1) {
        const u64 k = readlane_u64(mykey, __builtin_ctzll(it));
        if (mykey == k && lane < 63 - __builtin_clzll(ballot(mykey == k))) mykey = KEY_INF;
      }
    }
  }
}

// The kernel's arguments, read where they are used: named through `a` they are all fetched at the
// kernel's start and held in scalar registers for the whole search, which then spill.
__device__ __forceinline__ const SearchArgs& args_here() {
  const void* p = (const void*)__builtin_amdgcn_kernarg_segment_ptr();  // (the arguments come first)
  asm volatile("" : "+s"(p));
  return *reinterpret_cast<const SearchArgs*>(p);
}

// Four waves per SIMD: 512 searches of eight waves, or 1,024 of four, are then on the chip at once.  It
// holds the kernel to 128 registers, and three float instances of 8 pieces per lane spill 2 to 7 of
// them.  Free to take up to 139 they do not spill, but beyond 384 searches a second generation
// waits for the first (300,000 points of 256 floats, R = 32, 512 searches, L = 100: 556 -> 810 us).
//
// FIRST: the first wave, whose chain the search is, goes before the waves that work ahead (launch_wide_slots).
template <int KIND, int VEC, int NCH, int NSLOT, bool FIRST>
__global__ __launch_bounds__(64 * WIDE_MAX_WAVES, 4) void search_wide_kernel(SearchArgs a, VecTable T, u32 nlists) {
  extern __shared__ __align__(16) unsigned char smem[];
  u64* lists = reinterpret_cast<u64*>(smem);  // nlists x 64
  WideCtrl* ctrl = reinterpret_cast<WideCtrl*>(lists + (u64)nlists * 64);
  const u32 nb = a.hash_buckets;
  WideFilter F;
  F.bucket = reinterpret_cast<uint4*>(ctrl + 1);
  F.id_bits = a.id_bits;
  F.idmask = (1u << a.id_bits) - 1u;
  F.tagmask = (1u << (a.id_bits - (31u - (u32)__builtin_clz(nb)))) - 1u;
  F.yshl = 24u - a.id_bits;  // (ids of at most 24 bits)
  F.nb8 = nb << 8;

  const int lane = threadIdx.x & 63;
  const u32 wave = readlane_u32(threadIdx.x >> 6, 0);
  const u32 W = blockDim.x >> 6;
  const u32 qi = blockIdx.x;
  const u32 L = a.L;

  const u32 qrow = a.qidx ? a.qidx[qi] : qi;
  const QueryRegs<KIND, VEC, NCH> Q =
      load_query<KIND, VEC, NCH>(a.queries + (u64)qrow * a.qrow_bytes, T.npieces, lane);
  for (u32 i = threadIdx.x; i < nb; i += blockDim.x) F.bucket[i] = make_uint4(NONE_ID, NONE_ID, NONE_ID, NONE_ID);
  if (a.batch_counters != nullptr && qi == 0 && threadIdx.x == 0) zero_batch_counters(a.batch_counters);

  if (threadIdx.x == 0) {
    ctrl->go = 0;
    ctrl->done = 0;
  }
  __syncthreads();  // the filter is clear

  u32 evals = 0, n_pass = 0;  // statistics only: of this wave
  const u32 rlane = (u32)lane < a.R ? (u32)lane : a.R - 1u;  // (lanes past the row: its last id, not looked at)
  auto load_row = [&](u32 v) { return a.graph[(u64)v * a.R + rlane]; };
  // the candidates of a row (x: one id per lane) that are not below `worst` enter the filter, the
  // others go to a list; returns how many those are
  auto expand = [&](u32 x, u64 worst, u64* out) {
    u32* cid = reinterpret_cast<u32*>(out);  // the ids first, then the keys
    const bool fresh = x != NONE_ID && (u32)lane < a.R && !F.seen(x);
    const u64 fm = ballot(fresh);
    const u32 m = (u32)__builtin_popcountll(fm);
    if (m == 0u) return 0u;
    if (fresh) cid[__builtin_popcountll(fm & lanemask_lt(lane))] = x;
    wave_lds_fence();
    const u32 dk = eval_up_to_64_full_rows<KIND, VEC, NCH>(T, Q, [cid](u32 c) { return cid[c]; }, m, lane);
    const u32 c = cand_of_lane(lane);
    const u32 id = c < m ? cid[c] : 0u;
    wave_lds_fence();
    const u64 key = wide_key(dk, id);
    const bool open = c < m && key < worst;
    const u64 om = ballot(open);
    if (open)
      out[__builtin_popcountll(om & lanemask_lt(lane))] = key;
    else if (c < m)
      F.enter(id);
    keep_join();
    evals += m;
    n_pass += (m + 7u) >> 3;
    return (u32)__builtin_popcountll(om);
  };

  // The joins kept apart below (keep_join) leave the state of the first wave's loop in scalar registers:
  // a query on a million points 62.5 -> 62.0 us, 37 of them on 200,000 156.7 -> 155.2, a build of 10,000
  // points 8.49 -> 8.31 ms, and 78 vector registers instead of 87 for two-slot uint8 beams.
  u64 A[NSLOT];  // the beam: the first wave's
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) A[s] = KEY_INF;
  u32 nv = 0, n_surv = 0, n_ins = 0;
  if (wave != 0) {
    u32 batch = 0;
    for (;;) {  // ends: the first wave always comes to its end and then stops the others
      u32 go;
      while ((go = lds_acquire(&ctrl->go)) == batch) __builtin_amdgcn_s_sleep(1);
      if (go == WIDE_STOP) break;
      batch = go;
      if (wave <= (go & 0xFFu)) {
        const u32 x = load_row(wide_id(readlane_u64(ctrl->key[wave - 1u], 0)));
        const u32 list = readlane_u32(ctrl->list[wave - 1u], 0);
        const u32 cnt = expand(x, readlane_u64(ctrl->worst, 0), lists + (u64)list * 64);
        if (lane == 0) {
          ctrl->count[list] = cnt;
          __hip_atomic_fetch_add(&ctrl->done, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        keep_join();
      }
    }
  } else {
    if constexpr (FIRST) __builtin_amdgcn_s_setprio(3);
    u32 st = a.start;
    if (a.starts != nullptr) st = a.starts[a.slot != nullptr ? a.slot[qi] : qi];
    const u32 dk = readlane_u32(eval_up_to_64<KIND, VEC, NCH>(T, Q, [st](u32) { return st; }, 1u, lane), 0);
    if (lane == 0) {
      A[0] = wide_key(dk, st);
      F.enter(st);
    }
    evals = 1;
    u32 size = 1;
    u64* vptr = a.vis != nullptr ? a.vis + (u64)qi * a.vis_cap : nullptr;
    u32 vcap = a.vis_cap;
    if (a.vis_where != nullptr && lane == 0) a.vis_where[qi] = ~0ull;

    // Lane i keeps list i: the key of the vertex expanded there (KEY_INF: free) and its length.
    // List 0 takes what this wave expands itself and is used up at once.
    u64 lkey = KEY_INF;
    u32 lcount = 0;
    u32 batch = 0, taken = 0;  // the last batch handed out; waves still at it
    // the other waves are through: their lists
    auto collect = [&] {
      taken = 0;
      lcount = (u32)lane < nlists ? ctrl->count[lane] : 0u;
      if (lcount == 0u) lkey = KEY_INF;
#pragma unroll
      for (int s = 0; s < NSLOT; ++s) {
        const u32 state = wide_state(A[s]);
        if (state >= STATE_TAKEN && state != STATE_EMPTY) {
          const u32 list = state - STATE_TAKEN;
          const u32 now = ctrl->count[list] != 0u ? 1u + list : STATE_EMPTY;
          A[s] = (A[s] & ~0xFEull) | (u64)(now << 1);
        }
      }
      keep_join();
    };
    for (;;) {
      // The turn of every entry before the first one that has yet to be expanded, whose expansion
      // has something to offer, or that lies beyond the (1 + eps) bound: nothing changes the
      // beam up to there.
      const bool eps = a.eps16 >= 0 && size >= a.k;
      const u64 kk = eps ? beam_entry<NSLOT>(A, a.k - 1u) : 0ull;
      u32 stop = (u32)NSLOT * 64u;
#pragma unroll
      for (int s = NSLOT - 1; s >= 0; --s) {
        const bool b = !(A[s] & 1ull) && (wide_state(A[s]) != STATE_EMPTY || (eps && beyond_eps<KIND>(A[s], kk, a)));
        const u64 bm = ballot(b);
        if (bm) stop = (u32)(s * 64) + (u32)__builtin_ctzll(bm);
      }
#pragma unroll
      for (int s = 0; s < NSLOT; ++s) {
        const bool turn = !(A[s] & 1ull) && (u32)(s * 64 + lane) < stop;
        const u64 tm = ballot(turn);
        if (tm == 0ull) continue;
        const u32 cnt = (u32)__builtin_popcountll(tm);
        if (vptr != nullptr) {
          if (nv + cnt <= vcap) {
            if (turn) vptr[nv + (u32)__builtin_popcountll(tm & lanemask_lt(lane))] = plain_key(A[s]);
            keep_join();
          } else {
            u32 at = nv;
            for (u64 it = tm; it; it &= it - 1, ++at)
              visited_append(args_here(), qi, vptr, vcap, at, plain_key(readlane_u64(A[s], __builtin_ctzll(it))), lane);
          }
        }
        nv += cnt;
        if (turn) A[s] |= 1ull;
      }
      if (stop == (u32)NSLOT * 64u) break;
      const u64 pk = beam_entry<NSLOT>(A, stop);
      if (eps && beyond_eps<KIND>(pk, kk, a)) break;
      const u32 state = wide_state(pk);
      if (state >= STATE_TAKEN) {  // (p*'s expansion is under way; empty ones were passed above)
        while (lds_acquire(&ctrl->done) != taken) __builtin_amdgcn_s_sleep(1);  // ends: they only expand
        collect();
        continue;
      }
      if (vptr != nullptr) {
        if (nv < vcap) {
          if (lane == 0) vptr[nv] = plain_key(pk);
          keep_join();
        } else {
          visited_append(args_here(), qi, vptr, vcap, nv, plain_key(pk), lane);
        }
      }
      ++nv;
#pragma unroll
      for (int s = 0; s < NSLOT; ++s)
        if ((u32)(s * 64 + lane) == stop) A[s] |= 1ull;
      u32 from = 0, cnt = 0;
      if (state == STATE_NEW) {
        const u32 x = load_row(wide_id(pk));  // travels while the others get their work
        const u64 worst = beam_worst<NSLOT, WIDE_FLAGS>(A, L, size);
        if (taken != 0u && lds_acquire(&ctrl->done) == taken) collect();
        if (taken == 0u) {
          if (lkey >= worst) lkey = KEY_INF;  // fallen out of the beam
          const bool room = lane > 0 && (u32)lane < nlists && lkey == KEY_INF;
          const u64 roomm = ballot(room);
          u32 ahead = (u32)__builtin_popcountll(roomm);
          if (ahead > W - 1u) ahead = W - 1u;
          // the r-th free list takes the r-th entry
          const u32 r = (u32)__builtin_popcountll(roomm & lanemask_lt(lane));
          if (room && r < ahead) ctrl->list[r] = (u32)lane;
          wave_lds_fence();
          u32 before = 0;
#pragma unroll
          for (int s = 0; s < NSLOT; ++s) {
            const bool want = !(A[s] & 1ull) && wide_state(A[s]) == STATE_NEW;
            const u64 wm = ballot(want);
            const u32 e = before + (u32)__builtin_popcountll(wm & lanemask_lt(lane));
            if (want && e < ahead) {
              ctrl->key[e] = A[s];
              A[s] |= (u64)((STATE_TAKEN + ctrl->list[e]) << 1);
            }
            before += (u32)__builtin_popcountll(wm);
          }
          keep_join();
          if (ahead > before) ahead = before;
          if (ahead != 0u) {
            wave_lds_fence();
            if (room && r < ahead) lkey = ctrl->key[r];
            taken = ahead;
            batch = (batch + 1u) & 0xFFFFFFu;
            if (lane == 0) {
              ctrl->worst = worst;
              ctrl->done = 0;
              __hip_atomic_store(&ctrl->go, (batch << 8) | ahead, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            keep_join();
          }
        }
        cnt = expand(x, worst, lists);
        wave_lds_fence();
      } else {
        from = state - 1u;
        if ((u32)lane == from) lkey = KEY_INF;
        cnt = readlane_u32(lcount, (int)from);
      }
      // beam <- beam U N_out(p*), keep the L closest
      if (cnt != 0u) {
        const bool last_row = cnt <= 16u;  // up to 16 candidates sit in the last row of lanes
        const u32 i = last_row ? (u32)lane - 48u : (u32)lane;
        u64 mykey = KEY_INF;
        if (i < cnt) {
          mykey = lists[from * 64u + i];
          if (!F.enter(wide_id(mykey))) mykey = KEY_INF;
        }
        const u32 ns = wide_insert<NSLOT>(A, mykey, last_row, L, size, lane);
        n_surv += ns;
        n_ins += ns != 0u ? 1u : 0u;
      }
    }
    if (lane == 0) __hip_atomic_store(&ctrl->go, WIDE_STOP, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
  }

  const SearchArgs& z = args_here();
  if (wave == 0) {
    if (z.nvis != nullptr && lane == 0) z.nvis[qi] = nv;
#pragma unroll
    for (int s = 0; s < NSLOT; ++s)
      if (A[s] != KEY_INF) A[s] = plain_key(A[s]);
    if (z.next_start != nullptr && lane == 0) {
      // the beam's first entry is the closest vertex the search visited (it always holds one)
      const u32 best = key_id(A[0]);
      z.next_start[z.slot != nullptr ? z.slot[qi] : qi] = z.down != nullptr ? z.down[best] : best;
    }
    write_results<KIND, NSLOT>(A, z, qi, lane);
  }
  if (z.counters != nullptr && lane == 0) {
    DevCounters* c = block_counters(z.counters);
    if (wave == 0) {
      atomicAdd(&c->searches, 1ull);
      atomicAdd(&c->hops, (unsigned long long)nv);
      atomicAdd(&c->survivors, (unsigned long long)n_surv);
      atomicAdd(&c->insert_hops, (unsigned long long)n_ins);
    }
    atomicAdd(&c->evals, (unsigned long long)evals);
    atomicAdd(&c->passes, (unsigned long long)n_pass);
  }
}

template <int KIND, int VEC, int NCH, int NSLOT>
static void launch_wide_slots(const SearchArgs& a, const VecTable& T, u32 nlists, dim3 grid, dim3 block, u32 lds, hipStream_t s) {
  // The first wave before the others: where four waves and more share a SIMD (500 searches on 300,000 points, R = 48, L = 64,
  // 125.5 -> 119.5 us, on float rows 174.6 -> 169.5, 900 on 900,000 points 153.8 -> 151.6; builds of 25,000 points 14.3 ->
  // 13.9 ms), and in the upper layers of a layered build, beside which the bottom layer searches (200,000 points: 27.4 ->
  // 26.6 ms).  With fewer searches it only holds up the waves it will wait for (300 on 500,000 points 153.8 -> 155.4 us).
  if (a.nq > 384u || (a.starts != nullptr && a.vis != nullptr))
    hipLaunchKernelGGL((search_wide_kernel<KIND, VEC, NCH, NSLOT, true>), grid, block, lds, s, a, T, nlists);
  else
    hipLaunchKernelGGL((search_wide_kernel<KIND, VEC, NCH, NSLOT, false>), grid, block, lds, s, a, T, nlists);
}

template <int KIND, int VEC, int NCH>
static hipError_t launch_wide(const SearchArgs& a, const VecTable& T, u32 waves, hipStream_t s) {
  const u32 nlists = waves * 4u < WIDE_MAX_LISTS ? waves * 4u : WIDE_MAX_LISTS;
  const u32 ns = search_nslot_for(a.L);
  const u32 lds = nlists * 64u * 8u + (u32)sizeof(WideCtrl) + a.hash_buckets * 16u;
  const dim3 grid(a.nq), block(waves * 64u);
  switch (ns) {
    case 1: launch_wide_slots<KIND, VEC, NCH, 1>(a, T, nlists, grid, block, lds, s); break;
    case 2: launch_wide_slots<KIND, VEC, NCH, 2>(a, T, nlists, grid, block, lds, s); break;
    case 4: launch_wide_slots<KIND, VEC, NCH, 4>(a, T, nlists, grid, block, lds, s); break;
    default: return hipErrorInvalidConfiguration;
  }
  return hipGetLastError();
}

hipError_t launch_search_wide(const DistCfg& cfg, const SearchArgs& args, const VecTable& T, u32 waves, hipStream_t s) {
  if (waves < 2u || waves > WIDE_MAX_WAVES) return hipErrorInvalidConfiguration;
  SearchArgs a = args;
  // a filter of its own size: LDS is no concern with few searches
  a.hash_buckets = WIDE_BUCKETS;
  search_filter_mode(a.n, a.hash_buckets, &a.id_bits, &a.tag_width);
  if (a.tag_width != 16u) return hipErrorInvalidConfiguration;
  ANN_DISPATCH_CFG(launch_wide, a, T, waves, s);
}

}  // namespace annmi
