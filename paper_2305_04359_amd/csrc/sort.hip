// Grouping of reversed edges by destination: a stable least-significant-digit radix sort of
// 64-bit keys (destination << 32 | source) on the destination bits only (by default; a caller
// may name another run of key bits).  It takes the place of
// the semisort in BatchInsert (Alg. 3): equal destinations become consecutive, and, the sort
// being stable, the sources of one destination stay in the order they were emitted (batch order).
//
// One wavefront owns a tile of consecutive keys and walks it 64 keys at a time, so ranking inside
// a tile needs no cross-wave coordination: a key's rank among equal digits of its 64-key row is
// a popcount over a match mask built from one ballot per digit bit.  Digits are up to 10 bits
// wide.  Equal destinations need only stand together, so where their bits are at most 21 one pass
// does (group_split), and merge.hip groups each of its buckets; more bits take all passes.  At most
// 12,288 keys are sorted by one workgroup.
#include "ann_device.hpp"
#include "ann_internal.hpp"
#include "plan_device.hpp"

namespace annmi {

constexpr u32 RS_DIGIT_BITS = 10;  // at most this many key bits per pass
constexpr u32 RS_RADIX = 1u << RS_DIGIT_BITS;

static u64 rs_tile_keys(u64 count) {
  // at least 1024 keys per tile, at most 8192 tiles
  u64 t = (count + 8191) / 8192;
  if (t < 1024) t = 1024;
  return (t + 63) / 64 * 64;
}
static u64 rs_tiles(u64 count) { return (count + rs_tile_keys(count) - 1) / rs_tile_keys(count); }

// RS_RADIX x tiles counters and RS_RADIX digit totals, enough for any sort of AT MOST `count`
// keys.  (The number of tiles is not monotone in the key count: 8,192 x 1,024 keys make 8,192
// tiles, a few more keys make tiles of 1,088 keys and fewer of them.)
u64 radix_hist_entries(u64 count) {
  u64 tiles = (count + 1023) / 1024 + 1;
  if (tiles > 8192) tiles = 8192;
  return RS_RADIX * (tiles + 1);
}

// DROP: keys of all ones (unused slots) are left out.
template <bool DROP>
__global__ __launch_bounds__(64) void rs_hist_kernel(const u64* keys, u64 count, u64 tile_keys, u32 tiles,
                                                     u32 shift, u32 mask, u32* hist) {
  __shared__ u32 cnt[RS_RADIX];
  const int lane = threadIdx.x;
  for (u32 i = lane; i < RS_RADIX; i += 64) cnt[i] = 0;
  __syncthreads();
  const u64 lo = (u64)blockIdx.x * tile_keys;
  const u64 hi = lo + tile_keys < count ? lo + tile_keys : count;
  // four rows of 64 keys requested at a time: the walk waits for memory, not for arithmetic
  for (u64 i0 = lo + lane; i0 < hi; i0 += 256) {
    u64 k4[4];
#pragma unroll
    for (u32 q = 0; q < 4; ++q) k4[q] = i0 + 64u * q < hi ? keys[i0 + 64u * q] : 0ull;
#pragma unroll
    for (u32 q = 0; q < 4; ++q)
      if (i0 + 64u * q < hi && !(DROP && k4[q] == KEY_INF)) atomicAdd(&cnt[(u32)(k4[q] >> shift) & mask], 1u);
  }
  __syncthreads();
  for (u32 i = lane; i < RS_RADIX; i += 64) hist[(u64)i * tiles + blockIdx.x] = cnt[i];
}

// hist is a RS_RADIX x tiles table.  One workgroup per digit turns its row into an exclusive
// prefix over the tiles and leaves the row total in digit_total[digit] ...
__global__ __launch_bounds__(256) void rs_rowscan_kernel(u32* hist, u32 tiles, u32* digit_total) {
  __shared__ u32 part[256];
  const u32 t = threadIdx.x;
  u32* row = hist + (u64)blockIdx.x * tiles;
  const u32 per = (tiles + 255) / 256;
  const u32 lo = t * per < tiles ? t * per : tiles;
  const u32 hi = lo + per < tiles ? lo + per : tiles;
  u32 s = 0;
  for (u32 i = lo; i < hi; ++i) s += row[i];
  part[t] = s;
  __syncthreads();
  for (u32 off = 1; off < 256; off <<= 1) {
    const u32 v = t >= off ? part[t - off] : 0u;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  u32 run = t ? part[t - 1] : 0u;
  for (u32 i = lo; i < hi; ++i) {
    const u32 v = row[i];
    row[i] = run;
    run += v;
  }
  if (t == 255) digit_total[blockIdx.x] = part[255];
}

// ... and every scatter workgroup turns the RS_RADIX totals into the first output index of each
// digit for itself (an exclusive scan of 1,024 numbers in LDS costs a microsecond; a kernel of
// its own for it cost six, and a "last workgroup does it" ticket inside the row scan more still:
// RS_RADIX atomics on one address).
template <bool DROP>
__global__ __launch_bounds__(64) void rs_scatter_kernel(const u64* keys, u64* out, u64 count, u64 tile_keys,
                                                        u32 tiles, u32 shift, u32 mask, u32 nbits,
                                                        const u32* hist, const u32* digit_total) {
  __shared__ u32 base[RS_RADIX];
  const int lane = threadIdx.x;
  {
    // exclusive scan of the digit totals: lane l owns digits [PL*l, PL*(l+1))
    constexpr u32 PL = RS_RADIX / 64;
    u32 v[PL], sum = 0;
#pragma unroll
    for (u32 k = 0; k < PL; ++k) {
      v[k] = digit_total[PL * lane + k];
      sum += v[k];
    }
    u32 incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const u32 o = (u32)__shfl_up((int)incl, off, 64);
      if (lane >= off) incl += o;
    }
    u32 run = incl - sum;
#pragma unroll
    for (u32 k = 0; k < PL; ++k) {
      const u32 dgt = PL * lane + k;
      base[dgt] = run + hist[(u64)dgt * tiles + blockIdx.x];
      run += v[k];
    }
  }
  __syncthreads();
  const u64 lo = (u64)blockIdx.x * tile_keys;
  const u64 hi = lo + tile_keys < count ? lo + tile_keys : count;
  for (u64 i4 = lo; i4 < hi; i4 += 256) {
    u64 k4[4];  // four rows requested before the first is ranked
#pragma unroll
    for (u32 q = 0; q < 4; ++q) k4[q] = i4 + 64u * q + lane < hi ? keys[i4 + 64u * q + lane] : 0ull;
#pragma unroll
    for (u32 q = 0; q < 4; ++q) {
      const u64 i0 = i4 + 64u * q;
      if (i0 >= hi) break;  // uniform
      const u64 i = i0 + lane;
      const u64 key = k4[q];
      const bool valid = i < hi && !(DROP && key == KEY_INF);
      const u32 dg = (u32)(key >> shift) & mask;
      u64 match = ballot(valid);
      for (u32 b = 0; b < nbits; ++b) {
        const bool bit = (dg >> b) & 1u;
        const u64 bm = ballot(bit);
        match &= bit ? bm : ~bm;
      }
      const u32 rank = (u32)__builtin_popcountll(match & lanemask_lt(lane));
      u32 dst = 0;
      if (valid) dst = base[dg] + rank;
      __syncthreads();
      // the highest lane of each group of equal digits advances the group's counter
      if (valid && (match >> lane) == 1ull) base[dg] += (u32)__builtin_popcountll(match);
      __syncthreads();
      if (valid) out[dst] = key;
    }
  }
}

// Few keys: the whole sort in one workgroup.  The three launches of a pass take 18 us however few the
// keys are (each workgroup of the scan and of the scatter walks 1,024 digits), and a small batch
// waits for two passes of them.  Here 16 waves hold the keys in registers, wave w those from
// 64 ROWS w on; a pass ranks them as above, in counters of each wave's own, turns the counters into
// first positions (digit by digit, inside a digit wave by wave: stable) and exchanges the keys
// through LDS.  Bound by the chain of LDS round trips of a wave's rows.  6,400 keys
// on 14 bits: 37 us in six launches, 13.5 us here; 1,024 keys 7 us, 4,096 keys 11 us (build of 10,000
// points, R = 32: 9.65 -> 8.30 ms).
//
// PLAN: the keys are a batch's reversed edges, sorted by all bits of their destination, and the segments are planned in
// the same launch: a thread looks at the keys it holds after the last pass, and finds the end of a segment that starts with
// one of them in LDS.
constexpr u64 RS_ONE_MAX = 64ull * 12 * 16;

template <int WAVES, int ROWS, bool PLAN>
__global__ __launch_bounds__(64 * WAVES) void rs_one_kernel(u64* keys, u32 count, u32 first_bit, u32 key_bits,
                                                            u32 npass, MergeArgs a) {
  constexpr u32 D = RS_RADIX;
  constexpr u32 N = 64u * ROWS * WAVES;
  constexpr u32 PL = D / (64u * WAVES);  // digits a thread owns in the scan
  __shared__ u64 xch[N];
  __shared__ unsigned short cnt[WAVES * D];  // cnt[w * D + digit]
  __shared__ u32 wave_total[WAVES];
  const u32 t = threadIdx.x, lane = t & 63u, w = t >> 6;
  const u32 i0 = 64u * ROWS * w + lane;  // key of row q: i0 + 64 q
  unsigned short* mine = cnt + w * D;
  u64 k[ROWS];
#pragma unroll
  for (u32 q = 0; q < (u32)ROWS; ++q) k[q] = i0 + 64u * q < count ? keys[i0 + 64u * q] : ~0ull;

  const u32 per = (key_bits + npass - 1) / npass;
  u32 done = 0;
  for (u32 p = 0; p < npass; ++p) {
    const u32 nb = key_bits - done < per ? key_bits - done : per;
    const u32 shift = first_bit + done, digits = 1u << nb;
    done += nb;
    for (u32 i = lane; i < digits; i += 64) mine[i] = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    u32 rank[ROWS];
#pragma unroll
    for (u32 q = 0; q < (u32)ROWS; ++q) {
      rank[q] = 0;
      if (i0 - lane + 64u * q < count) {  // uniform
        const bool valid = i0 + 64u * q < count;
        const u32 dg = (u32)(k[q] >> shift) & (digits - 1u);
        u64 match = ballot(valid);
        for (u32 b = 0; b < nb; ++b) {
          const bool bit = (dg >> b) & 1u;
          const u64 bm = ballot(bit);
          match &= bit ? bm : ~bm;
        }
        if (valid) {
          const u32 before = mine[dg];  // read by the group's lanes before its highest lane writes
          rank[q] = before + (u32)__builtin_popcountll(match & lanemask_lt((int)lane));
          __builtin_amdgcn_wave_barrier();
          if ((match >> lane) == 1ull) mine[dg] = (unsigned short)(before + (u32)__builtin_popcountll(match));
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
    }
    __syncthreads();
    // thread t owns digits PL t to PL t + PL - 1: their total, then the exclusive scan
    u32 total = 0;
    if (PL * t < digits) {
      for (u32 j = 0; j < PL; ++j)
        if (PL * t + j < digits)
          for (u32 v = 0; v < (u32)WAVES; ++v) total += cnt[v * D + PL * t + j];
    }
    u32 incl = total;
#pragma unroll
    for (u32 off = 1; off < 64; off <<= 1) {
      const u32 o = (u32)__shfl_up((int)incl, off, 64);
      if (lane >= off) incl += o;
    }
    if (lane == 63) wave_total[w] = incl;
    __syncthreads();
    u32 run = incl - total;
    for (u32 v = 0; v < w; ++v) run += wave_total[v];
    for (u32 j = 0; j < PL; ++j) {
      if (PL * t + j >= digits) break;
      for (u32 v = 0; v < (u32)WAVES; ++v) {
        const u32 c = cnt[v * D + PL * t + j];
        cnt[v * D + PL * t + j] = (unsigned short)run;  // (at most count, which fits)
        run += c;
      }
    }
    __syncthreads();
#pragma unroll
    for (u32 q = 0; q < (u32)ROWS; ++q)
      if (i0 + 64u * q < count) xch[mine[(u32)(k[q] >> shift) & (digits - 1u)] + rank[q]] = k[q];
    __syncthreads();
#pragma unroll
    for (u32 q = 0; q < (u32)ROWS; ++q)
      if (i0 + 64u * q < count) k[q] = xch[i0 + 64u * q];
  }
#pragma unroll
  for (u32 q = 0; q < (u32)ROWS; ++q)
    if (i0 + 64u * q < count) keys[i0 + 64u * q] = k[q];
  if constexpr (PLAN) {
    __shared__ u32 cnt_lds[4], base_lds[4], stat_lds[2];
    if (t < 4) cnt_lds[t] = 0;
    if (t < 2) stat_lds[t] = 0;
    __syncthreads();
    u32 filed[ROWS], cnt[ROWS], m[ROWS];
#pragma unroll
    for (u32 q = 0; q < (u32)ROWS; ++q) {  // (all meta words requested before the first segment is measured)
      const u32 i = i0 + 64u * q, b = (u32)(k[q] >> 32);
      const bool head = i < count && b != NONE_ID && (i == 0 || (u32)(xch[i - 1u] >> 32) != b);
      cnt[q] = head ? 1u : 0u;
      m[q] = a.meta[head ? b : 0u];
    }
#pragma unroll
    for (u32 q = 0; q < (u32)ROWS; ++q) {
      filed[q] = NONE_ID;
      if (cnt[q] == 0) continue;
      const u32 i = i0 + 64u * q, b = (u32)(k[q] >> 32);
      u32 lo = i, step = 1;  // gallop, then bisect
      while (i + step < count && (u32)(xch[i + step] >> 32) == b) {
        lo = i + step;
        step <<= 1;
      }
      u32 hi = i + step < count ? i + step : count;
      while (hi - lo > 1) {
        const u32 mid = (lo + hi) >> 1;
        if ((u32)(xch[mid] >> 32) == b)
          lo = mid;
        else
          hi = mid;
      }
      cnt[q] = hi - i;
      const int kind = plan_segment(a, b, m[q], cnt[q], stat_lds, [&](u32 j) { return (u32)xch[i + j]; });
      if (kind >= 0) filed[q] = ((u32)kind << 30) | atomicAdd(&cnt_lds[kind], 1u);
    }
    __syncthreads();
    plan_reserve(a, cnt_lds, base_lds, stat_lds);
    __syncthreads();
#pragma unroll
    for (u32 q = 0; q < (u32)ROWS; ++q)
      if (filed[q] != NONE_ID) {
        const u32 b = (u32)(k[q] >> 32), kind = filed[q] >> 30;
        plan_file(a, (int)kind, base_lds[kind] + (filed[q] & 0x3FFFFFFFu), i0 + 64u * q, cnt[q], b, m[q]);
      }
  }
}

// One workgroup plans 1,024 keys in 3 us and so saves a launch; 6,400 keys, which are 25 workgroups' work, in 11, where the
// launch of its own takes 5.
constexpr u64 RS_PLAN_MAX = 64ull * 4 * 4;
bool sort_and_plan_ok(u64 count) { return count <= RS_PLAN_MAX; }
hipError_t launch_sort_and_plan(const MergeArgs& a, u64* keys, u32 key_bits, hipStream_t s) {
  if (a.nkeys == 0) return hipSuccess;
  const u32 npass = (key_bits + RS_DIGIT_BITS - 1) / RS_DIGIT_BITS;
  hipLaunchKernelGGL((rs_one_kernel<4, 4, true>), dim3(1), dim3(256), 0, s, keys, (u32)a.nkeys, 32u, key_bits, npass, a);
  return hipGetLastError();
}

hipError_t radix_sort_edges(u64* keys, u64* tmp, u32* hist, u64 hist_entries, u64 count, u32 key_bits,
                            hipStream_t s, u32 first_bit) {
  if (count < 2 || key_bits == 0) return hipSuccess;
  if ((u64)RS_RADIX * (rs_tiles(count) + 1) > hist_entries) return hipErrorInvalidValue;  // histogram too small
  if (first_bit + key_bits > 64) key_bits = 64 - first_bit;  // (callers sort within the key)
  const u32 npass = (key_bits + RS_DIGIT_BITS - 1) / RS_DIGIT_BITS;
  // One compute unit against the whole chip: six launches take 37 to 46 us up to 65,536 keys, one
  // workgroup 20 us at 8,192 keys and twenty bits and a third more per 4,096 keys; 12,288 keys is
  // what its LDS holds.  Few waves for few keys: a workgroup of sixteen waits for a compute unit that
  // has room for all of them (18 us a sort in the layered build, where layers overlap; 9 us so).
  if (count <= RS_ONE_MAX) {
#define RS_ONE(W, ROWS) \
  hipLaunchKernelGGL((rs_one_kernel<W, ROWS, false>), dim3(1), dim3(64 * W), 0, s, keys, (u32)count, first_bit, key_bits, npass, MergeArgs{})
    if (count <= 64u * 4 * 4)
      RS_ONE(4, 4);
    else if (count <= 64u * 8 * 8)
      RS_ONE(8, 8);
    else if (count <= 64u * 16 * 8)
      RS_ONE(16, 8);
    else
      RS_ONE(16, 12);
#undef RS_ONE
    return hipGetLastError();
  }
  const u64 tile_keys = rs_tile_keys(count);
  const u32 tiles = (u32)rs_tiles(count);
  const u32 per = (key_bits + npass - 1) / npass;
  u64* src = keys;
  u64* dst = tmp;
  u32 done = 0;
  for (u32 p = 0; p < npass; ++p) {
    const u32 nb = key_bits - done < per ? key_bits - done : per;
    const u32 shift = first_bit + done;
    const u32 mask = (1u << nb) - 1u;
    hipLaunchKernelGGL(rs_hist_kernel<false>, dim3(tiles), dim3(64), 0, s, src, count, tile_keys, tiles, shift, mask, hist);
    u32* digit_total = hist + (u64)RS_RADIX * tiles;
    hipLaunchKernelGGL(rs_rowscan_kernel, dim3(RS_RADIX), dim3(256), 0, s, hist, tiles, digit_total);
    hipLaunchKernelGGL(rs_scatter_kernel<false>, dim3(tiles), dim3(64), 0, s, src, dst, count, tile_keys, tiles, shift,
                       mask, nb, hist, digit_total);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    u64* t = src;
    src = dst;
    dst = t;
    done += nb;
  }
  if (src != keys) return hipMemcpyAsync(keys, src, count * sizeof(u64), hipMemcpyDeviceToDevice, s);
  return hipSuccess;
}

// The first half of grouping a batch's keys (the second: group_plan_kernel in merge.hip): one stable pass over the
// low bits of the destinations, unused slots left out.
bool group_split_plan(u64 count, u32 key_bits, u32* low_bits) {
  if (count <= RS_ONE_MAX || key_bits > RS_DIGIT_BITS + GROUP_HIGH_BITS) return false;
  // buckets of about 512 keys, so that there are some hundreds of workgroups
  u32 low = key_bits > GROUP_HIGH_BITS - 1u ? key_bits - (GROUP_HIGH_BITS - 1u) : 1u;
  while (low < RS_DIGIT_BITS && low < key_bits - 1u && (count >> low) > 512u) ++low;
  *low_bits = low < RS_DIGIT_BITS ? low : RS_DIGIT_BITS;
  return true;
}
// a wave's tile: a batch of a few thousand points needs more of them than rs_tile_keys gives
static u64 group_tile_keys(u64 count) { return count <= (1u << 18) ? 256 : count <= (1u << 19) ? 512 : rs_tile_keys(count); }
u64 group_hist_entries(u64 count) {
  if (count <= RS_ONE_MAX) return radix_hist_entries(count);
  const u64 tk = group_tile_keys(count), tiles = (count + tk - 1) / tk, most = radix_hist_entries(count);
  // (no larger for a smaller count: sizes below the lines take up to 1,024 tiles)
  const u64 need = RS_RADIX * ((tiles < 1024 ? 1024 : tiles) + 1);
  return need > most ? need : most;
}
hipError_t group_split(const u64* keys, u64* out, u32* hist, u64 hist_entries, u64 count, u32 low_bits, const u32** bucket_total,
                       hipStream_t s) {
  const u64 tile_keys = group_tile_keys(count);
  const u32 tiles = (u32)((count + tile_keys - 1) / tile_keys);
  if ((u64)RS_RADIX * (tiles + 1u) > hist_entries) return hipErrorInvalidValue;
  const u32 mask = (1u << low_bits) - 1u;
  u32* digit_total = hist + (u64)RS_RADIX * tiles;
  hipLaunchKernelGGL(rs_hist_kernel<true>, dim3(tiles), dim3(64), 0, s, keys, count, tile_keys, tiles, 32u, mask, hist);
  hipLaunchKernelGGL(rs_rowscan_kernel, dim3(RS_RADIX), dim3(256), 0, s, hist, tiles, digit_total);
  hipLaunchKernelGGL(rs_scatter_kernel<true>, dim3(tiles), dim3(64), 0, s, keys, out, count, tile_keys, tiles, 32u, mask, low_bits,
                     hist, digit_total);
  *bucket_total = digit_total;
  return hipGetLastError();
}

}  // namespace annmi
