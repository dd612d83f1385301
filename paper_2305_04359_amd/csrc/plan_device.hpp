// Planning of step 2 of BatchInsert: what becomes of the segment of reversed edges that a destination receives.  Shared
// by the kernels that find the segments (sort.hip, merge.hip).
#pragma once
#include "ann_device.hpp"
#include "ann_internal.hpp"

namespace annmi {

__device__ __forceinline__ u32 meta_deg(u32 m) { return m & 0xFFFFu; }
__device__ __forceinline__ u32 meta_clean(u32 m) { return m >> 16; }
__device__ __forceinline__ u32 make_meta(u32 deg, u32 clean) { return deg | (clean << 16); }

// What becomes of a segment of cnt edges to b, whose meta word is m and whose sources are source(0 .. cnt - 1): appended here
// where the row has room (returns -1), else the work list it belongs on: 0 fast, 1 gram, 2 generic with a long
// candidate list, 3 generic with a list of up to 512.
template <class Source>
__device__ __forceinline__ int plan_segment(const MergeArgs& a, u32 b, u32 m, u32 cnt, u32* stat_lds, Source source) {
  const u32 deg = meta_deg(m), clean = meta_clean(m);
  if (!a.force_prune && deg + cnt <= a.R) {
    u32* row = a.graph + (u64)b * a.R;
    for (u32 j = 0; j < cnt; ++j) row[deg + j] = source(j);
    a.meta[b] = make_meta(deg + cnt, clean);
    if (a.counters != nullptr) {
      atomicAdd(&stat_lds[0], 1u);
      atomicAdd(&stat_lds[1], cnt);
    }
    return -1;
  }
  const u32 fresh = deg - clean + cnt;
  int kind = 2;
  if (a.force_prune)
    kind = (a.gram_ok && deg + cnt <= a.gram_tmax) ? 1 : 2;  // (the fast path presumes a clean prefix)
  else if (clean <= 64 && fresh <= a.fast_amax)
    kind = 0;
  else if (a.gram_ok && deg + cnt <= a.gram_tmax)
    kind = 1;
  return kind == 2 && deg + cnt <= a.medium_max ? 3 : kind;
}
// One global atomic per work list and workgroup; the order of a list has no influence on any result, every segment is
// processed on its own.
__device__ __forceinline__ void plan_reserve(const MergeArgs& a, const u32* cnt_lds, u32* base_lds, const u32* stat_lds) {
  if (threadIdx.x < 4 && cnt_lds[threadIdx.x] != 0)
    base_lds[threadIdx.x] = atomicAdd(&a.list_count[threadIdx.x], cnt_lds[threadIdx.x]);
  if (a.counters != nullptr && threadIdx.x == 0 && stat_lds[0] != 0) {
    atomicAdd(&block_counters(a.counters)->appends, (unsigned long long)stat_lds[0]);
    atomicAdd(&block_counters(a.counters)->edges, (unsigned long long)stat_lds[1]);
  }
}
__device__ __forceinline__ void plan_file(const MergeArgs& a, int kind, u32 at_, u64 i0, u32 cnt, u32 b, u32 m) {
  const long long at = (long long)at_;
  a.list_items[kind][kind == 3 ? -at : at] = MergeItem{(u32)i0, cnt, b, m};
}

}  // namespace annmi
