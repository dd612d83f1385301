// The beam search of search_kernel.hpp, one wavefront per search, with the memory of the next hops
// requested ahead: for launches that leave the chip half empty.
//
// What bounds a search there is its chain of hops: a row, then the vectors it names (two dependent trips to
// memory), and the instructions between them, of which a wave issues one every four cycles however idle
// the chip.  Of 130 hops (beam of 128) only some 30 insert anything, so the vertex behind p* in the
// beam is the next one in twelve of thirteen cases.  While p*'s distances are taken, its successor,
// whose row was requested a hop earlier, is expanded: its fresh neighbours enter the filter and their
// vectors are requested; and the row of the vertex behind that one is.  If an insertion brings
// another vertex to the front, the expansion is undone: every lane puts back what its bucket of the
// filter held.  The order of hops, of evaluations and of filter entries is the one-wave kernel's, and so
// are all results.  Expanding two vertices ahead gained nothing (the waits were no shorter, the
// instructions more: 218 us against 203).
//
// 2,000 uint8 queries at L = 128, R = 64: 233 -> 203 us on 100,000 points, 374 -> 325 on a million;
// 100,001 points built in batches of up to 2,000: 34.8 -> 32.9 ms.
//
// The visited list is written 64 entries at a time, from the registers of the wave.
#include "ann_dispatch.hpp"
#include "search_kernel.hpp"

namespace annmi {

// Survivors of one hop from which on the sorting network takes them: one at a time they cost some 20
// instructions each and 60 in all, the network of a two-slot beam 500.
constexpr u32 AHEAD_NETWORK = 24;

// 8-vertex passes whose vectors are requested ahead (rows with more fresh neighbours, early in a search, wait
// for them)
template <int NCH>
struct AheadPasses {
  static constexpr int value = NCH <= 1 ? 2 : 1;
};

// orders a wave's own LDS accesses (the hardware keeps them in order; the compiler must, too)
__device__ __forceinline__ void ahead_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The kernel's arguments, read where they are used (see search_wide.hip)
__device__ __forceinline__ const SearchArgs& ahead_args() {
  const void* p = (const void*)__builtin_amdgcn_kernarg_segment_ptr();  // (the arguments come first)
  asm volatile("" : "+s"(p));
  return *reinterpret_cast<const SearchArgs*>(p);
}

// beam <- the L closest of the beam and the lanes' candidates (KEY_INF: none), all below `worst`; returns how
// many of them were not in the beam already.
template <int NSLOT>
__device__ __forceinline__ u32 ahead_insert(u64 (&A)[NSLOT], u64* beam, u64 mykey, u32 L, u32& size, int lane) {
  constexpr u64 FLAGS = 1;
  u64 sm = ballot(mykey != KEY_INF);
  if ((u32)__builtin_popcountll(sm) > AHEAD_NETWORK) {
    const u32 ns = (u32)__builtin_popcountll(sm);
    if (insert_sorted<NSLOT, FLAGS, false>(A, mykey, ns, L, size, lane)) return ns;
  }
  u32 shift[NSLOT], at = 0, n = 0;
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) shift[s] = 0;
  for (; sm; sm &= sm - 1) {
    const int l = __builtin_ctzll(sm);
    const u64 sk = readlane_u64(mykey, l);
    u32 lt = 0, gt = 0;
    bool above[NSLOT];
#pragma unroll
    for (int s = 0; s < NSLOT; ++s) {
      lt += (u32)__builtin_popcountll(ballot(A[s] < sk));
      above[s] = A[s] > (sk | FLAGS);
      gt += (u32)__builtin_popcountll(ballot(above[s]));
    }
    if (lt + gt != 64u * NSLOT) {  // in the beam already (the filter lost it)
      if (lane == l) mykey = KEY_INF;
      continue;
    }
    ++n;
#pragma unroll
    for (int s = 0; s < NSLOT; ++s) shift[s] += above[s] ? 1u : 0u;
    at += sk < mykey ? 1u : 0u;
    if (lane == l) at += lt;
  }
  if (n == 0u) return 0;
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) {
    const u32 np = (u32)(s * 64 + lane) + shift[s];
    if (A[s] != KEY_INF && np < L) beam[np] = A[s];
  }
  if (mykey != KEY_INF && at < L) beam[at] = mykey;
  ahead_fence();
  size = size + n < L ? size + n : L;
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) {
    const u32 idx = (u32)(s * 64 + lane);
    A[s] = beam[idx];
    if (idx >= size) A[s] = KEY_INF;
  }
  ahead_fence();
  return n;
}

template <int KIND, int VEC, int NCH, int NSLOT>
__global__ __launch_bounds__(64, 4) void search_ahead_kernel(SearchArgs a, VecTable T) {
  constexpr int SP = AheadPasses<NCH>::value;
  extern __shared__ __align__(16) unsigned char smem[];
  u32* cid = reinterpret_cast<u32*>(smem);
  u64* beam = reinterpret_cast<u64*>(cid + 64);
  uint4* bucket = reinterpret_cast<uint4*>(beam + 64 * NSLOT);
  const int lane = threadIdx.x;
  const int sub = lane & (LPC - 1);
  const u32 grp = (u32)lane >> 3;
  const u32 qi = blockIdx.x;
  const u32 nb = a.hash_buckets;
  const u32 idmask = (1u << a.id_bits) - 1u;
  const u32 tagmask = (1u << (a.id_bits - (31u - (u32)__builtin_clz(nb)))) - 1u;
  const u32 yshl = 24u - a.id_bits;
  const u32 nb8 = nb << 8;
  const u32 L = a.L;

  const u32 qrow = a.qidx ? a.qidx[qi] : qi;
  const QueryRegs<KIND, VEC, NCH> Q = load_query<KIND, VEC, NCH>(a.queries + (u64)qrow * a.qrow_bytes, T.npieces, lane);
  for (u32 i = lane; i < nb; i += 64) bucket[i] = make_uint4(NONE_ID, NONE_ID, NONE_ID, NONE_ID);
  if (a.batch_counters != nullptr && qi == 0 && lane == 0) zero_batch_counters(a.batch_counters);

  // in the filter already? if not, enter it: h and e are the bucket and what it held before
  auto enter = [&](u32 x, bool ok, u32& h, uint4& e) -> bool {
    const u32 y = (u32)__umul24(x, 0x9E3779u) & idmask;
    h = umulhi24(y << yshl, nb8);
    const u32 tag = y & tagmask;
    const u32 tt = tag | (tag << 16);
    e = bucket[h];
    const u32 mz = pk_min_u16(pk_min_u16(e.x ^ tt, e.y ^ tt), pk_min_u16(e.z ^ tt, e.w ^ tt));
    const bool fresh = ok && !((mz & 0xFFFFu) == 0u || (mz >> 16) == 0u);
    if (fresh)
      bucket[h] = make_uint4((e.x << 16) | tag, (e.y << 16) | (e.x >> 16), (e.z << 16) | (e.y >> 16), (e.w << 16) | (e.z >> 16));
    return fresh;
  };
  const bool whole = T.npieces == (u32)(LPC * NCH);
  auto request = [&](u32 id, Piece<VEC> (&x)[NCH]) {
    const char* row = T.base + (u64)id * T.row_bytes;
    if (whole) {
#pragma unroll
      for (int u = 0; u < NCH; ++u) x[u] = load_piece<VEC>(row + (u64)(sub + LPC * u) * VEC);
    } else {
#pragma unroll
      for (int u = 0; u < NCH; ++u) {
        const u32 pc = sub + LPC * u;
        x[u] = pc < T.npieces ? load_piece<VEC>(row + (u64)pc * VEC) : zero_piece<VEC>();
      }
    }
  };

  u64 A[NSLOT];
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) {
    A[s] = KEY_INF;
    beam[s * 64 + lane] = KEY_INF;
  }
  u32 st = a.start;
  if (a.starts != nullptr) st = a.starts[a.slot != nullptr ? a.slot[qi] : qi];
  ahead_fence();
  {
    const u32 dk = readlane_u32(eval_up_to_64<KIND, VEC, NCH>(T, Q, [st](u32) { return st; }, 1u, lane), 0);
    u32 h;
    uint4 e;
    if (lane == 0) {
      A[0] = make_key(dk, st);
      (void)enter(st, true, h, e);
    }
  }
  ahead_fence();

  u32 size = 1, nv = 0, evals = 1, n_pass = 0, n_surv = 0, n_ins = 0;
  u64* vptr = a.vis != nullptr ? a.vis + (u64)qi * a.vis_cap : nullptr;
  u32 vcap = a.vis_cap;
  if (a.vis_where != nullptr && lane == 0) a.vis_where[qi] = ~0ull;
  u64 vk = 0;  // lane i: entry i of the visited list's last, unwritten run of 64
  auto flush = [&](u32 cnt) {  // entries nv - cnt .. nv - 1
    if (vptr == nullptr) return;
    const u32 first = nv - cnt;
    if (nv <= vcap) {
      if ((u32)lane < cnt) vptr[first + lane] = vk;
      keep_join();
    } else {
      for (u32 i = 0; i < cnt; ++i) visited_append(ahead_args(), qi, vptr, vcap, first + i, readlane_u64(vk, (int)i), lane);
    }
  };
  const u32 rlane = (u32)lane < a.R ? (u32)lane : a.R - 1u;  // (lanes past the row: its last id, not looked at)
  auto load_row = [&](u32 v) { return a.graph[(u64)v * a.R + rlane]; };

  u32 idS = NONE_ID, mS = 0;   // the vertex expanded ahead, its fresh neighbours' count
  bool freshS = false;         // to undo that expansion in the filter
  u32 hS = 0;
  uint4 eS = make_uint4(0, 0, 0, 0);
  u32 idB = NONE_ID - 1u, rowB = NONE_ID;  // the vertex whose row has been requested
  Piece<VEC> X[SP][NCH];
#pragma unroll
  for (int t = 0; t < SP; ++t)
#pragma unroll
    for (int u = 0; u < NCH; ++u) X[t][u] = zero_piece<VEC>();

  // row x: filter, list of fresh ids, request of their vectors
  auto expand = [&](u32 x) {
    freshS = enter(x, x != NONE_ID && (u32)lane < a.R, hS, eS);
    const u64 fm = ballot(freshS);
    mS = (u32)__builtin_popcountll(fm);
    if (mS != 0u) {
      if (freshS) cid[__builtin_popcountll(fm & lanemask_lt(lane))] = x;
      ahead_fence();
      if (mS <= 8u * SP) {
#pragma unroll
        for (int t = 0; t < SP; ++t) {
          if (t > 0 && mS <= 8u * t) break;
          const u32 c = 8u * t + grp;
          request(cid[c < mS ? c : 0u], X[t]);
        }
      }
    }
  };

  u64 worst = KEY_INF;
  u64 um[NSLOT];  // the unprocessed entries of the beam behind n2
  u32 changed = 1;
  // the first of them
  auto pop = [&]() -> u32 {
    u32 id = NONE_ID;
#pragma unroll
    for (int s = 0; s < NSLOT; ++s) {
      if (id == NONE_ID && um[s]) {
        id = readlane_u32((u32)A[s], __builtin_ctzll(um[s])) >> 1;
        um[s] &= um[s] - 1;
      }
    }
    return id;
  };
  u32 p = NONE_ID, n1 = NONE_ID, n2 = NONE_ID;  // p* and the two behind it
  u32 m = 0;             // candidates of p* waiting for their distances (their ids in cid, their vectors in X)
  u32 more = 0;          // rowB is to be expanded now: the successor's row, or p*'s own
  u32 forced = 0;        // p* was not expanded ahead: its row is rowB, its turn comes after the expansion
  u32 nextB = NONE_ID;   // the row to request next
  for (;;) {
    u64 mykey = KEY_INF;
    if (m != 0u) {
      u32 dk = 0;
      if (m <= 8u * SP) {
#pragma unroll
        for (int t = 0; t < SP; ++t) {
          if (t > 0 && m <= 8u * t) break;
          const u32 d = distance_key<KIND, VEC, NCH>(Q, X[t]);
          if (sub == t) dk = d;
        }
      } else {
        dk = eval_up_to_64_full_rows<KIND, VEC, NCH>(T, Q, [cid](u32 c) { return cid[c]; }, m, lane);
      }
      const u32 c = cand_of_lane(lane);
      const u32 id = cid[c];
      mykey = make_key(dk, id);
      if (c >= m || mykey >= worst) mykey = KEY_INF;
      ahead_fence();
      evals += m;
      n_pass += (m + 7u) >> 3;
    }
    // rowB is the last thing requested.  Waited for here, nothing is outstanding for the compiler to wait for
    // where the expansion takes registers that a request of another path might still fill.
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    if (more != 0u) expand(rowB);
    if (nextB != NONE_ID) {
      rowB = load_row(nextB);
      idB = nextB;
      nextB = NONE_ID;
    }
    if (ballot(mykey != KEY_INF) != 0ull) {
      const u32 ns = ahead_insert<NSLOT>(A, beam, mykey, L, size, lane);
      worst = beam_worst<NSLOT, 1ull>(A, L, size);
      changed = 1;
      n_surv += ns;
      n_ins += ns != 0u ? 1u : 0u;
    }
    if (forced == 0u) {
      // p* <- closest unprocessed member of the beam, and the two that follow it
      if (changed != 0u) {
#pragma unroll
        for (int s = 0; s < NSLOT; ++s) um[s] = ballot(!(A[s] & 1ull));  // (KEY_INF has the flag)
        p = pop();
        n1 = pop();
      } else {
        p = n1;
        n1 = n2;
      }
      n2 = pop();
      changed = 0;
      if (p == NONE_ID) break;
      u64 pk = 0;
#pragma unroll
      for (int s = 0; s < NSLOT; ++s) {
        const bool me = (u32)A[s] == p << 1;
        const u64 mm = ballot(me);
        const u64 k = readlane_u64(A[s], __builtin_ctzll(mm | (1ull << 63)));
        pk = mm != 0ull ? k : pk;
        A[s] |= me ? 1ull : 0ull;
      }
      if (a.eps16 >= 0 && size >= a.k) {
        if (beyond_eps<KIND>(pk, beam_entry<NSLOT>(A, a.k - 1u), a)) break;
      }
      if ((u32)lane == (nv & 63u)) vk = pk;
      ++nv;
      if ((nv & 63u) == 0u) flush(64u);
      if (p != idS) {
        if (idS != NONE_ID && freshS) bucket[hS] = eS;  // the vertex expanded ahead is not next
        ahead_fence();
        if (p != idB) rowB = load_row(p);
        idB = p;
        nextB = n1;
        idS = p;
        m = 0;
        more = 1;
        forced = 1;
        continue;
      }
    }
    forced = 0;
    m = mS;
    more = n1 == idB ? 1u : 0u;
    idS = more != 0u ? n1 : NONE_ID;  // the next vertex, if its row is here
    nextB = more != 0u ? n2 : n1;
  }

  if ((nv & 63u) != 0u) flush(nv & 63u);
  const SearchArgs& z = ahead_args();
  if (z.nvis != nullptr && lane == 0) z.nvis[qi] = nv;
  if (z.next_start != nullptr && lane == 0) {
    const u32 best = key_id(A[0]);
    z.next_start[z.slot != nullptr ? z.slot[qi] : qi] = z.down != nullptr ? z.down[best] : best;
  }
  write_results<KIND, NSLOT>(A, z, qi, lane);
  if (z.counters != nullptr && lane == 0) {
    DevCounters* c = block_counters(z.counters);
    atomicAdd(&c->searches, 1ull);
    atomicAdd(&c->hops, (unsigned long long)nv);
    atomicAdd(&c->evals, (unsigned long long)evals);
    atomicAdd(&c->passes, (unsigned long long)n_pass);
    atomicAdd(&c->survivors, (unsigned long long)n_surv);
    atomicAdd(&c->insert_hops, (unsigned long long)n_ins);
  }
}

template <int KIND, int VEC, int NCH>
static hipError_t launch_ahead(const SearchArgs& a, const VecTable& T, hipStream_t s) {
  const u32 lds = 64u * 4u + search_nslot_for(a.L) * 512u + a.hash_buckets * 16u;
  const dim3 grid(a.nq), block(64);
  switch (search_nslot_for(a.L)) {
    case 1: hipLaunchKernelGGL((search_ahead_kernel<KIND, VEC, NCH, 1>), grid, block, lds, s, a, T); break;
    case 2: hipLaunchKernelGGL((search_ahead_kernel<KIND, VEC, NCH, 2>), grid, block, lds, s, a, T); break;
    default: return hipErrorInvalidConfiguration;
  }
  return hipGetLastError();
}

#define ANN_AHEAD_CFG(KIND, NCH) \
  case KIND * 10 + NCH: return launch_ahead<KIND, 16, NCH>(a, T, s)
hipError_t launch_search_ahead(const DistCfg& cfg, const SearchArgs& args, const VecTable& T, hipStream_t s) {
  SearchArgs a = args;
  a.hash_buckets = AHEAD_BUCKETS;
  search_filter_mode(a.n, a.hash_buckets, &a.id_bits, &a.tag_width);
  if (a.tag_width != 16u || a.R > 64u || cfg.vec != 16) return hipErrorInvalidConfiguration;
  switch (cfg.kind * 10 + cfg.nch) {
    ANN_AHEAD_CFG(K_U8, 1);
    ANN_AHEAD_CFG(K_U8, 2);
    ANN_AHEAD_CFG(K_U8, 4);
    ANN_AHEAD_CFG(K_I8, 1);
    ANN_AHEAD_CFG(K_I8, 2);
    ANN_AHEAD_CFG(K_I8, 4);
    default: return hipErrorInvalidConfiguration;
  }
}
#undef ANN_AHEAD_CFG

}  // namespace annmi
