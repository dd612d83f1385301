// The clustering-based builder of Sec. 4.3 (ParlayHCNNG) with the cluster trees of Sec. 3.2.
//
// Per group of trees: the points are split level by level (all splitting nodes of a level in one
// pass: every point takes the side of the nearer of its node's two pivots; a stable two-way split
// from running counts of left points puts the children in place, finished children straight into
// the final order); the leaves' vectors are gathered as int8 into tiles of 32 rows laid out as
// the matrix cores read them; one wavefront per 32 points of a leaf finds their l nearest
// neighbours inside the leaf on the matrix cores (32 x 32 inner products per instruction group,
// every lane keeping the best of the candidates it sees for its own point); one workgroup per
// leaf sorts the leaf's candidate pairs in LDS, and one wavefront per leaf runs Kruskal's scan
// with the degree bound, 64 pairs at a time (a pair that fails once fails for good, so the wave
// tests 64 in parallel and accepts at once all that no earlier one can change; the scan is a chain of
// dependent LDS trips, so thousands of leaves are scanned side by side).
// At the end every point's neighbours of all trees, each once (found where the trees left them, in places of the
// point's own, or, with many trees or a large degree bound, by sorting all arcs), are
// pruned with the alpha rule of Sec. 4.1 by the re-prune kernel of the flat graph's BatchInsert.
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <type_traits>

#include "ann_device.hpp"
#include "driver_internal.hpp"
#include "plan_device.hpp"

using namespace annmi;

namespace annmi {
namespace hcnng {

constexpr u32 HC_MAX_LS = 1024;       // points per leaf
constexpr u32 HC_MAX_L = 16;          // nearest neighbours per point that restrict the tree
constexpr u32 HC_MAX_PAIRS = 16384;   // candidate pairs per leaf (sorted in LDS)
constexpr u32 HC_MAX_DEPTH = 39;      // below this depth a node is cut in the middle of its order
constexpr u32 HC_NONE = 0xFFFFFFFFu;

typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef int v16i_t __attribute__((ext_vector_type(16)));

u64 stream_output(u64 seed, u64 k) {  // the (k+1)-th output of SplitMix64(seed)
  u64 z = seed + (k + 1) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
u64 mulhi64(u64 a, u64 b) { return (u64)(((unsigned __int128)a * (unsigned __int128)b) >> 64); }

u32 bits_to_hold(u64 count) {  // smallest b with 2^b - 1 >= count: indices below count never have all b bits set
  u32 b = 1;
  while (((1ull << b) - 1ull) < count) ++b;
  return b;
}

// A wavefront of the side kernels takes SIDE_PER_WAVE consecutive positions.  The node of its first
// position is found once, by a uniform search that the scalar unit runs; the later positions step
// forward from there.
constexpr u32 SIDE_PER_WAVE = 128, SIDE_PER_WAVE_F32 = 32;
__device__ inline u32 side_first_node(const u32* off, u32 nseg, u64 w0) {
  u32 lo = 0, hi = nseg;
  while (hi - lo > 1) {
    const u32 mid = (lo + hi) >> 1;
    if ((u64)off[mid] <= w0)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// The sides of one level's points: bit i % 32 of right[i / 32] is set if the point at position i is farther
// from the first pivot of its node than from the second.  ids: the point at each position; the nodes of the
// level are the position ranges off[s]..off[s+1]; a node that splits names the positions of its two
// pivots, the points of any other node are all left ones.
//
// A wavefront takes SIDE_PER_WAVE consecutive positions, whose vectors are all requested before the first
// is used, 32 at a time: the pivots of up to 16 nodes are the rows of a matrix product and the 32 points
// its columns, so that a point costs a quarter of a matrix instruction instead of 16 dot products and
// their sums across lanes, and hands on one bit instead of its key again.  Nearly always one node covers all 32.
// What bounds it: 128 bytes gathered per point.  30 trees over a million uint8 points of 128: 365 -> 247 us per
// level on average (39 levels), with the ids of 4 bytes and the sides of one bit that the split then reads
// (74 + 29 + 13 -> 52 + 4 + 4 us) the build 65.7 -> 59.4 ms.
template <bool SIGNED>
__global__ __launch_bounds__(256) void hc_side_kernel(const unsigned char* pts, u32 row_bytes, const u32* ids, u64 n,
                                                      const u32* off, u32 nseg, const u32* pos1, const u32* pos2,
                                                      u32* right) {
  const int lane = (int)(threadIdx.x & 63u);
  const u32 half = (u32)lane >> 5, col = (u32)lane & 31u;
  const u64 w0 = ((u64)blockIdx.x * 4u + (u32)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6))) * SIDE_PER_WAVE;
  if (w0 >= n) return;
  constexpr u32 NT = SIDE_PER_WAVE / 32u;
  const u32 npieces = row_bytes / 16u;  // at most 8
  constexpr u32 flip = SIGNED ? 0u : 0x80808080u;  // uint8 data moved down by 128: distances do not change
  auto load_row = [&](u32 id, v4i_t (&x)[4]) {
    const unsigned char* row = pts + (u64)id * row_bytes;
#pragma unroll
    for (u32 ks = 0; ks < 4; ++ks)
      x[ks] = 2u * ks + half < npieces ? *reinterpret_cast<const v4i_t*>(row + 16u * (2u * ks + half)) : v4i_t{0, 0, 0, 0};
  };
  auto to_int8 = [&](v4i_t (&x)[4]) {  // (the pieces behind the row's end stay zero)
#pragma unroll
    for (u32 ks = 0; ks < 4; ++ks) x[ks] = 2u * ks + half < npieces ? x[ks] ^ (int)flip : x[ks];
  };
  u32 id[NT];
#pragma unroll
  for (u32 q = 0; q < NT; ++q) {
    const u64 i = w0 + 32u * q + col;
    id[q] = ids[i < n ? i : n - 1u];
  }
  v4i_t x[NT][4];
#pragma unroll
  for (u32 q = 0; q < NT; ++q) load_row(id[q], x[q]);

  u32 seg = side_first_node(off, nseg, w0);
  u32 held = HC_NONE;  // the node whose pivots are rows 0 and 1 of the operand
  v4i_t pv[4];
  u32 splits = 0;  // row's node splits
  i32 norm = 0;    // the pivot's squared norm
  u32 word = 0;    // lane q: the sides of tile q
#pragma unroll
  for (u32 q = 0; q < NT; ++q) {
    const u64 t0 = w0 + 32u * q;
    if (t0 >= n) break;  // uniform
    const u64 t1 = t0 + 31u < n ? t0 + 31u : n - 1u;
    while ((u64)off[seg + 1] <= t0) ++seg;
    u32 last = seg;  // (a node that splits has 3 points or more, one that does not is deep: at most 12 nodes in 32
                     // positions, as the level holds only nodes of more points than a leaf)
    while ((u64)off[last + 1] <= t1) ++last;
    if (held == HC_NONE || seg < held || last > held + 15u || (seg == last && seg != held)) {  // uniform
      held = seg;
      const u32 node = held + (col >> 1) < nseg ? held + (col >> 1) : nseg - 1u;
      const u32 p = (col & 1u) ? pos2[node] : pos1[node];
      splits = p != HC_NONE ? 1u : 0u;
      load_row(splits ? ids[p] : 0u, pv);
      to_int8(pv);
      norm = 0;
#pragma unroll
      for (u32 ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int k = 0; k < 4; ++k) norm = __builtin_amdgcn_sdot4(pv[ks][k], pv[ks][k], norm, false);
      norm += __shfl_xor(norm, 32, 64);
    }
    to_int8(x[q]);
    v16i_t acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(pv[ks], x[q][ks], acc, 0, 0, 0);
    // |x-a|^2 <= |x-b|^2  <=>  |a|^2 - |b|^2 - 2 (<x,a> - <x,b>) <= 0.  Register r of a lane is row 8 (r / 4) +
    // 4 half + r % 4: the pivots of node held + k are registers 4 (k / 4) + 2 (k % 2) and the next, in the
    // lanes of half (k / 2) % 2.
    bool far;
    if (seg == last) {
      const i32 d = (i32)readlane_u32((u32)norm, 0) - (i32)readlane_u32((u32)norm, 1);
      far = readlane_u32(splits, 0) != 0 && d - 2 * (acc[0] - acc[1]) > 0;
    } else {
      const u64 i = t0 + col;
      u32 k = seg - held;
      while (held + k < last && (u64)off[held + k + 1] <= i) ++k;
      i32 v = 0;
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int e = 0; e < 2; ++e)
          if (k == (u32)(4 * g + e) + 2u * half) v = acc[4 * g + 2 * e] - acc[4 * g + 2 * e + 1];
      const i32 other = __shfl_xor(v, 32, 64);
      if (((k >> 1) & 1u) != half) v = other;
      const i32 d = __shfl(norm, (int)(2u * k), 64) - __shfl(norm, (int)(2u * k + 1u), 64);
      const u32 sp = (u32)__shfl((int)splits, (int)(2u * k), 64);
      far = sp != 0 && d - 2 * v > 0;
    }
    const u32 bits = (u32)ballot(far && half == 0 && t0 + col < n);
    if ((u32)lane == q) word = bits;
  }
  if ((u32)lane < NT && w0 + 32u * (u32)lane < n) right[w0 / 32u + (u32)lane] = word;
}

// Leaf vectors are kept in tiles of 32 consecutive points of ONE leaf (a leaf's tiles follow one
// another from tile_of_leaf[leaf]; the unused rows of its last tile are zero, and nothing that is
// kept is computed from them): inside a tile the 16-byte
// piece c of row r lies at (c * 32 + r) * 16, so that the matrix-core operand of the
// nearest-neighbour kernels -- lane (row, half) takes piece 2 ks + half of its row -- is 1 KB of
// consecutive bytes per load instead of 32 bytes out of each of 32 rows.
__device__ inline u32 leaf_of_tile(const u32* tile_of_leaf, u32 nleaves, u32 tile) {
  u32 lo = 0, hi = nleaves;  // uniform: the scalar unit runs this
  while (hi - lo > 1) {
    const u32 mid = (lo + hi) >> 1;
    if (tile_of_leaf[mid] <= tile)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// The vectors in that layout, as int8 (uint8 data moved down by 128: distances do not change),
// rows of lv_stride bytes (a multiple of 32, zero tail), and their squared norms (times 512, and a number below 16) by
// position.  One workgroup per tile, eight lanes per point.
template <bool SIGNED>
__global__ __launch_bounds__(256) void hc_gather_kernel(const unsigned char* pts, u32 row_bytes, const u64* keys,
                                                        const u32* leaf_off, const u32* tile_of_leaf, u32 nleaves,
                                                        u32 lv_stride, unsigned char* leafvec, i32* leafnorm) {
  const u32 tile = blockIdx.x;
  const u32 leaf = leaf_of_tile(tile_of_leaf, nleaves, tile);
  const u32 r = threadIdx.x >> 3, sub = threadIdx.x & 7u;
  const u32 in_leaf = 32u * (tile - tile_of_leaf[leaf]) + r;
  unsigned char* y = leafvec + (u64)tile * 32u * lv_stride;
  if (in_leaf >= leaf_off[leaf + 1] - leaf_off[leaf]) {  // an unused row of the leaf's last tile: zeros
    for (u32 pc = sub; pc < lv_stride / 16; pc += 8)
      *reinterpret_cast<uint4*>(y + ((u64)pc * 32u + r) * 16u) = make_uint4(0, 0, 0, 0);
    return;
  }
  const u64 i = (u64)leaf_off[leaf] + in_leaf;
  const u32 id = (u32)keys[i];
  const uint4* x = reinterpret_cast<const uint4*>(pts + (u64)id * row_bytes);
  i32 nn = 0;
  for (u32 pc = sub; pc < lv_stride / 16; pc += 8) {
    uint4 v = make_uint4(0, 0, 0, 0);
    if (pc < row_bytes / 16) {
      v = x[pc];
      if constexpr (!SIGNED) {
        v.x ^= 0x80808080u;
        v.y ^= 0x80808080u;
        v.z ^= 0x80808080u;
        v.w ^= 0x80808080u;
      }
    }
    *reinterpret_cast<uint4*>(y + ((u64)pc * 32u + r) * 16u) = v;
    nn = __builtin_amdgcn_sdot4((i32)v.x, (i32)v.x, nn, false);
    nn = __builtin_amdgcn_sdot4((i32)v.y, (i32)v.y, nn, false);
    nn = __builtin_amdgcn_sdot4((i32)v.z, (i32)v.z, nn, false);
    nn = __builtin_amdgcn_sdot4((i32)v.w, (i32)v.w, nn, false);
  }
  nn = group_sum(nn);
  // where the nearest-neighbour kernel's keys hold the distance, and which of its lane's 16 candidates of a tile it is
  if (sub == 0) leafnorm[i] = (nn << 9) | (i32)(4u * (r / 8u) + r % 4u);
}

// Which leaf and which 32 queries of it a block of the nearest-neighbour kernels takes.  A leaf's
// blocks all read the whole leaf, so they should run at the same time on one XCD and find it in
// that XCD's L2: blocks go to the XCDs in turn, so block b belongs to XCD b % 8, and the blocks of
// one XCD walk through the query tiles of a leaf before they move to the next leaf.
__device__ inline bool knn_block(u32 nleaves, u32 ny, u32& leaf, u32& q0) {
  const u32 xcd = blockIdx.x & 7u, k = blockIdx.x >> 3;
  leaf = 8u * (k / ny) + xcd;
  q0 = 32u * (k % ny);
  return leaf < nleaves;
}

__device__ __forceinline__ u32 med3_u32(u32 a, u32 b, u32 c) {
  u32 r;
  asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// best <- the N smallest of two ascending lists, ascending: the smaller of one list's i-th and the other's
// i-th from the end are the N smallest, rising up to some place and falling behind it; a merging network
// over the next power of two, with zeros in front, sorts them.
template <int N>
__device__ __forceinline__ void merge_lists(u64 (&best)[N], const u64 (&other)[N]) {
  constexpr int P = N <= 4 ? 4 : N <= 8 ? 8 : N <= 16 ? 16 : 32;
  u64 v[P];
#pragma unroll
  for (int i = 0; i < P; ++i) v[i] = 0ull;
#pragma unroll
  for (int i = 0; i < N; ++i) v[P - N + i] = best[i] < other[N - 1 - i] ? best[i] : other[N - 1 - i];
#pragma unroll
  for (int j = P / 2; j > 0; j >>= 1)
#pragma unroll
    for (int i = 0; i < P; ++i)
      if ((i & j) == 0) {
        const u64 lo = v[i] < v[i + j] ? v[i] : v[i + j], hi = v[i] < v[i + j] ? v[i + j] : v[i];
        v[i] = lo;
        v[i + j] = hi;
      }
#pragma unroll
  for (int i = 0; i < N; ++i) best[i] = v[P - N + i];
}

// a lane's own keys, ascending: a bitonic network over the next power of two
template <int N>
__device__ __forceinline__ void sort_list(u64 (&a)[N]) {
  constexpr int P = N <= 4 ? 4 : N <= 8 ? 8 : N <= 16 ? 16 : 32;
  u64 v[P];
#pragma unroll
  for (int i = 0; i < P; ++i) v[i] = i < P - N ? 0ull : a[i - (P - N)];
#pragma unroll
  for (int k = 2; k <= P; k <<= 1)
#pragma unroll
    for (int j = k / 2; j > 0; j >>= 1)
#pragma unroll
      for (int i = 0; i < P; ++i)
        if ((i & j) == 0) {
          const bool up = (i & k) == 0;
          const u64 lo = v[i] < v[i + j] ? v[i] : v[i + j], hi = v[i] < v[i + j] ? v[i + j] : v[i];
          v[i] = up ? lo : hi;
          v[i + j] = up ? hi : lo;
        }
#pragma unroll
  for (int i = 0; i < N; ++i) a[i] = v[P - N + i];
}

// The l nearest neighbours, inside its leaf, of each of 32 consecutive points of a leaf (block
// (leaf, 32-point block), one wavefront).  Matrix-core tile: rows = 32 candidates, columns = the
// 32 points; lane (half, col) then holds, for point col, the inner products with 16 of the 32
// candidates, and keeps the LCAP smallest (distance, position) keys it has seen in registers.
// The two lanes of a point merge their lists at the end.  knn_pos / knn_d: l entries per point,
// ascending; positions are relative to the leaf.
//
// What bounds it: vector instructions (84 % of the cycles), five per candidate to form, test and queue its key
// and ten (v_med3) per queue entry to put it in the list.  30 trees over a million uint8 points, leaves
// of up to 1,000, l = 10: 10.9 -> 8.3 ms (insertion by min and max, 100 exchanges per merge and tiles moved
// between registers before).  Longer queues (32, 40) gain nothing, nor do blocks of four waves that read
// a leaf side by side (10.9).
template <int LCAP>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(LCAP <= 10 ? 4 : 3, LCAP <= 10 ? 4 : 3))) void hc_knn_kernel(const unsigned char* leafvec, const i32* leafnorm, u32 lv_stride,
                                                    const u32* leaf_off, const u32* tile_of_leaf, u32 l,
                                                    unsigned short* knn_pos, i32* knn_d, u32 nleaves, u32 ny) {
  u32 leaf, q0;
  if (!knn_block(nleaves, ny, leaf, q0)) return;
  const u32 off = leaf_off[leaf];
  const u32 cnt = leaf_off[leaf + 1] - off;
  if (q0 >= cnt) return;
  const unsigned char* tiles = leafvec + (u64)tile_of_leaf[leaf] * 32u * lv_stride;  // the leaf's first tile
  const int lane = threadIdx.x;
  const u32 half = (u32)lane >> 5, col = (u32)lane & 31u;
  const u32 ksteps = lv_stride / 32u;  // at most 4
  const u32 q = q0 + col;
  const u32 qrow = q < cnt ? q : cnt - 1u;
  const u32 qn = (u32)leafnorm[off + qrow] & ~511u;  // (times 512, like the candidates' norms)
  v4i_t bq[4];
#pragma unroll
  for (u32 ks = 0; ks < 4; ++ks) {
    const u32 kk = ks < ksteps ? ks : ksteps - 1u;
    const v4i_t y = *reinterpret_cast<const v4i_t*>(tiles + (u64)q0 * lv_stride + ((2u * kk + half) * 32u + col) * 16u);
    bq[ks] = ks < ksteps ? y : v4i_t{0, 0, 0, 0};
  }
  // A lane meets the candidates c0 + 8 (r / 4) + 4 half + r % 4: numbered c0 / 2 + r (below 512)
  // they ascend with the candidate's position, and a squared distance of at most 128 bytes is
  // below 2^23, so (distance << 9 | number) orders a lane's candidates like (distance, position)
  // in one 32-bit word: an insertion step is a min and a max.
  constexpr u32 K32_INF = 0xFFFFFFFFu;
  u32 best32[LCAP];
#pragma unroll
  for (int i = 0; i < LCAP; ++i) best32[i] = K32_INF;
  // Candidates below the lane's worst kept key wait in a queue of the lane's own (LDS, one
  // column per lane) and are inserted when some lane's queue is full: the insertion code then
  // runs a few times per wave with most lanes busy, not once per candidate for one lane's sake.
  constexpr u32 QCAP = 24;  // a tile adds at most 16 per lane; drained once above 8
  __shared__ __align__(16) unsigned char pend[QCAP * 256];
  const u32 first = 4u * (u32)lane;
  u32 at = first;  // (bytes) where the lane's next entry goes
  u32 worst = K32_INF;
  auto drain = [&]() {
    // into an ascending list: every place takes the middle one of the key, its own entry and the one before
#pragma unroll 1
    for (u32 p = first; p < QCAP * 256u; p += 512u) {
      if (ballot(p < at) == 0ull) break;
      const u32 k0 = *reinterpret_cast<const u32*>(pend + p);  // (what lies behind the queue's end is not used)
      const u32 k1 = *reinterpret_cast<const u32*>(pend + p + 256u);
      const u32 key[2] = {p < at ? k0 : K32_INF, p + 256u < at ? k1 : K32_INF};
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int t = LCAP - 1; t > 0; --t) best32[t] = med3_u32(key[h], best32[t - 1], best32[t]);
        best32[0] = key[h] < best32[0] ? key[h] : best32[0];
      }
    }
    at = first;
    // The point's other lane has the other half of the candidates: half a list from each of the two is a
    // whole one, and what is farther than both halves' ends cannot enter it (8.6 -> 8.3 ms).
    const u32 mine = best32[LCAP / 2 - 1], theirs = (u32)__shfl_xor((int)mine, 32, 64);
    const u32 end = (mine > theirs ? mine : theirs) | 511u;  // (numbers of two lanes do not compare: all of that distance)
    worst = end < best32[LCAP - 1] ? end + 1u : best32[LCAP - 1];
  };

  struct Tile {
    v4i_t av[4], cn[4];
  };
  auto request = [&](u32 c0, Tile& t) {
#pragma unroll
    for (u32 ks = 0; ks < 4; ++ks) {
      const u32 kk = ks < ksteps ? ks : ksteps - 1u;
      t.av[ks] = *reinterpret_cast<const v4i_t*>(tiles + (u64)c0 * lv_stride + ((2u * kk + half) * 32u + col) * 16u);
    }
    // norms of this lane's 16 candidates: rows 8g + 4 half + 0..3, g = 0..3 (the array has a tail
    // of 64 entries, so reading past the leaf's end stays inside it)
#pragma unroll
    for (u32 g = 0; g < 4; ++g) t.cn[g] = *reinterpret_cast<const v4i_t*>(leafnorm + off + c0 + 8u * g + 4u * half);
  };
  auto use = [&](u32 c0, const Tile& tile) {
    if (ballot(at > first + 256u * (QCAP - 16u)) != 0ull) drain();  // room for this tile in every lane's queue
    v16i_t acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(tile.av[ks], bq[ks], acc, 0, 0, 0);
    // only the tile with the queries themselves and the leaf's last tile hold candidates to skip
    const u32 qn_tile = qn + (c0 >> 1);
    int minus_1024;  // (out of the compiler's sight, which makes two instructions of a known power of two)
    asm("s_movk_i32 %0, -1024" : "=s"(minus_1024));
    auto scan = [&](auto checked) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const u32 cand = c0 + 8u * (r / 4) + 4u * half + (r % 4);
        // (|q|^2 + |c|^2 - 2<q,c>) << 9 | number, from norms that come shifted and with the number in the tile:
        // a multiplication (an inner product over 128 bytes fits 24 bits) and a sum of three.  (No asm
        // statement may read the products: the compiler waits for the matrix unit only before its own
        // instructions.)
        const u32 packed = (u32)__mul24(acc[r], minus_1024) + ((u32)tile.cn[r / 4][r % 4] + qn_tile);
        const bool valid = !decltype(checked)::value || (cand < cnt && cand != q);
        const u32 key = valid ? packed : K32_INF;
        // written in any case, kept when the place moves on: no lane is masked, no branch taken
        *reinterpret_cast<u32*>(pend + at) = key;
        at += key < worst ? 256u : 0u;
      }
    };
    if (c0 == q0 || c0 + 32u > cnt)
      scan(std::true_type{});
    else
      scan(std::false_type{});
  };
  // the tile after the current one is requested before the current one is used (the last one asks
  // for itself again); two tiles in turn, so that none is moved from register to register
  Tile t0, t1;
  request(0, t0);
  for (u32 c0 = 0; c0 < cnt; c0 += 64u) {
    request(c0 + 32u < cnt ? c0 + 32u : c0, t1);
    use(c0, t0);
    if (c0 + 32u >= cnt) break;
    request(c0 + 64u < cnt ? c0 + 64u : c0, t0);
    use(c0 + 32u, t1);
  }
  drain();
  // back to (distance << 32 | position), then the other half of the candidates from the partner lane
  u64 best[LCAP];
#pragma unroll
  for (int i = 0; i < LCAP; ++i) {
    const u32 k = best32[i], nr = k & 511u;
    const u32 cand = 32u * (nr >> 4) + 8u * ((nr & 15u) >> 2) + 4u * half + (nr & 3u);
    best[i] = k == K32_INF ? KEY_INF : (((u64)(k >> 9) << 32) | cand);
  }
  u64 other[LCAP];
#pragma unroll
  for (int i = 0; i < LCAP; ++i) other[i] = (u64)__shfl_xor((unsigned long long)best[i], 32, 64);
  merge_lists<LCAP>(best, other);
  if (half == 0 && q < cnt) {
#pragma unroll
    for (int j = 0; j < LCAP; ++j) {
      if ((u32)j < l) {
        const u64 o = (u64)(off + q) * l + j;
        knn_pos[o] = best[j] == KEY_INF ? (unsigned short)0xFFFF : (unsigned short)(best[j] & 0xFFFFull);
        knn_d[o] = (i32)(best[j] >> 32);
      }
    }
  }
}

// ---- float data ------------------------------------------------------------------------------
// The same three steps for float vectors (squared L2, or the negative inner product).  Sums run in
// fp32 in a fixed order; which of two nearly equal distances is the smaller may come out
// differently from an fp64 computation, and with it a point's side, a neighbour or a tree edge.
typedef float v16f_t __attribute__((ext_vector_type(16)));

template <bool MIPS>
__global__ __launch_bounds__(256) void hc_side_f32_kernel(const unsigned char* pts, u32 row_bytes, const u32* ids,
                                                          u64 n, const u32* off, u32 nseg, const u32* pos1,
                                                          const u32* pos2, u32* right) {
  const u32 sub = threadIdx.x & 7u, grp = (threadIdx.x >> 3) & 7u;
  const u64 w0 = ((u64)blockIdx.x * 4u + (u32)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6))) * SIDE_PER_WAVE_F32;
  if (w0 >= n) return;
  u32 seg = side_first_node(off, nseg, w0);
  u32 word = 0;
  for (u32 it = 0; it < SIDE_PER_WAVE_F32 / 8u; ++it) {
    const u64 i = w0 + 8u * it + grp;
    const u32 id = ids[i < n ? i : n - 1u];
    while ((u64)off[seg + 1] <= (i < n ? i : n - 1u)) ++seg;
    bool far = false;
    const u32 p1 = pos1[seg];
    if (p1 != HC_NONE) {
      const u32 ida = ids[p1], idb = ids[pos2[seg]];
      const float4* x = reinterpret_cast<const float4*>(pts + (u64)id * row_bytes);
      const float4* a = reinterpret_cast<const float4*>(pts + (u64)ida * row_bytes);
      const float4* b = reinterpret_cast<const float4*>(pts + (u64)idb * row_bytes);
      float da = 0.0f, db = 0.0f;
      for (u32 pc = sub; pc < row_bytes / 16; pc += 8) {
        const float4 vx = x[pc], va = a[pc], vb = b[pc];
        const float fx[4] = {vx.x, vx.y, vx.z, vx.w}, fa[4] = {va.x, va.y, va.z, va.w}, fb[4] = {vb.x, vb.y, vb.z, vb.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if constexpr (MIPS) {
            da = __builtin_fmaf(-fx[k], fa[k], da);
            db = __builtin_fmaf(-fx[k], fb[k], db);
          } else {
            const float ea = fx[k] - fa[k], eb = fx[k] - fb[k];
            da = __builtin_fmaf(ea, ea, da);
            db = __builtin_fmaf(eb, eb, db);
          }
        }
      }
      da = group_sum(da);
      db = group_sum(db);
      far = da > db;
    }
    u64 m = ballot(far && i < n) & 0x0101010101010101ull;  // bit 8 g: point g of the eight
    m |= m >> 7;
    m |= m >> 14;
    m |= m >> 28;
    word |= ((u32)m & 0xFFu) << (8u * it);
  }
  if ((threadIdx.x & 63u) == 0) right[w0 / 32u] = word;
}

// vectors in leaf order (rows of lv_stride bytes, zero tail) and their squared norms
__global__ __launch_bounds__(256) void hc_gather_f32_kernel(const unsigned char* pts, u32 row_bytes, const u64* keys,
                                                            const u32* leaf_off, const u32* tile_of_leaf, u32 nleaves,
                                                            u32 lv_stride, unsigned char* leafvec, float* leafnorm) {
  const u32 tile = blockIdx.x;
  const u32 leaf = leaf_of_tile(tile_of_leaf, nleaves, tile);
  const u32 r = threadIdx.x >> 3, sub = threadIdx.x & 7u;
  const u32 in_leaf = 32u * (tile - tile_of_leaf[leaf]) + r;
  unsigned char* y = leafvec + (u64)tile * 32u * lv_stride;
  if (in_leaf >= leaf_off[leaf + 1] - leaf_off[leaf]) {  // an unused row of the leaf's last tile: zeros
    for (u32 pc = sub; pc < lv_stride / 16; pc += 8)
      *reinterpret_cast<float4*>(y + ((u64)pc * 32u + r) * 16u) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    return;
  }
  const u64 i = (u64)leaf_off[leaf] + in_leaf;
  const u32 id = (u32)keys[i];
  const float4* x = reinterpret_cast<const float4*>(pts + (u64)id * row_bytes);
  float nn = 0.0f;
  for (u32 pc = sub; pc < lv_stride / 16; pc += 8) {
    float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (pc < row_bytes / 16) v = x[pc];
    *reinterpret_cast<float4*>(y + ((u64)pc * 32u + r) * 16u) = v;
    nn = __builtin_fmaf(v.x, v.x, nn);
    nn = __builtin_fmaf(v.y, v.y, nn);
    nn = __builtin_fmaf(v.z, v.z, nn);
    nn = __builtin_fmaf(v.w, v.w, nn);
  }
  nn = group_sum(nn);
  if (sub == 0) leafnorm[i] = nn;
}

// Nearest neighbours inside the leaf on the fp32 matrix cores (v_mfma_f32_32x32x2f32: two
// elements of the inner product per instruction; a lane feeds it, one after the other, the four
// floats of a 16-byte piece, the lower half-wave taking bytes 0..15 of every 32 and the upper half
// bytes 16..31: a reordering of the sum's terms that both operands share).  Squared L2 comes out
// as |a|^2 + |b|^2 - 2<a,b>, clamped at zero, for the selection (as in the integer kernel); the
// distances of the l candidates selected are then taken again as sum (a - b)^2 (see the end of the
// kernel).  knn_d receives the order-preserving 32-bit image of the distance.
template <int LCAP, bool MIPS>
__global__ __launch_bounds__(64) void hc_knn_f32_kernel(const unsigned char* leafvec, const float* leafnorm,
                                                        u32 lv_stride, const u32* leaf_off, const u32* tile_of_leaf,
                                                        u32 l, unsigned short* knn_pos, i32* knn_d, u32 nleaves,
                                                        u32 ny) {
  u32 leaf, q0;
  if (!knn_block(nleaves, ny, leaf, q0)) return;
  const u32 off = leaf_off[leaf];
  const u32 cnt = leaf_off[leaf + 1] - off;
  if (q0 >= cnt) return;
  const int lane = threadIdx.x;
  const u32 half = (u32)lane >> 5, col = (u32)lane & 31u;
  const u32 ksteps = lv_stride / 32u;
  const u32 q = q0 + col;
  const u32 qrow = q < cnt ? q : cnt - 1u;
  const float qn = leafnorm[off + qrow];
  const unsigned char* tiles = leafvec + (u64)tile_of_leaf[leaf] * 32u * lv_stride;  // the leaf's first tile
  const u32 in_tile = (half * 32u + col) * 16u;  // piece 2 ks + half of row col: at in_tile + ks * 1024
  const unsigned char* qp = tiles + (u64)q0 * lv_stride + in_tile;
  u64 best[LCAP];
#pragma unroll
  for (int i = 0; i < LCAP; ++i) best[i] = KEY_INF;
  constexpr u32 QCAP = 24;  // a tile adds at most 16 per lane; drained once above 8
  __shared__ u64 pend[QCAP][64];
  u32 pc = 0;
  u64 worst = KEY_INF;
  auto drain = [&]() {
#pragma unroll 1
    for (u32 i = 0; i < QCAP; ++i) {
      if (ballot(i < pc) == 0ull) break;
      u64 key = i < pc ? pend[i][lane] : KEY_INF;
#pragma unroll
      for (int t = 0; t < LCAP; ++t) {
        const u64 lo = key < best[t] ? key : best[t];
        key = key < best[t] ? best[t] : key;
        best[t] = lo;
      }
    }
    pc = 0;
    // (half a list from each of the point's two lanes, as above; these keys compare)
    const u64 mine = best[LCAP / 2 - 1], theirs = (u64)__shfl_xor((unsigned long long)mine, 32, 64);
    const u64 end = mine > theirs ? mine : theirs;
    worst = end < best[LCAP - 1] ? end + 1u : best[LCAP - 1];
  };
  for (u32 c0 = 0; c0 < cnt; c0 += 32u) {
    if (ballot(pc > QCAP - 16u) != 0ull) drain();  // room for this tile in every lane's queue
    const unsigned char* cp = tiles + (u64)c0 * lv_stride + in_tile;
    v16f_t acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (u32 ks = 0; ks < ksteps; ++ks) {
      const float4 a = *reinterpret_cast<const float4*>(cp + 1024u * ks);
      const float4 b = *reinterpret_cast<const float4*>(qp + 1024u * ks);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b.x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b.y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b.z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b.w, acc, 0, 0, 0);
    }
    float cn[16];
#pragma unroll
    for (u32 g = 0; g < 4; ++g) {
      const float4 v = *reinterpret_cast<const float4*>(leafnorm + off + c0 + 8u * g + 4u * half);
      cn[4 * g] = v.x;
      cn[4 * g + 1] = v.y;
      cn[4 * g + 2] = v.z;
      cn[4 * g + 3] = v.w;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const u32 cand = c0 + 8u * (r / 4) + 4u * half + (r % 4);
      float dd;
      if constexpr (MIPS) {
        dd = -acc[r];
      } else {
        dd = (qn + cn[r]) - 2.0f * acc[r];
        dd = dd < 0.0f ? 0.0f : dd;
      }
      const u64 key = (cand < cnt && cand != q) ? (((u64)dkey_from_float(dd) << 32) | cand) : KEY_INF;
      const bool qual = key < worst;
      if (qual) {
        pend[pc][lane] = key;
        ++pc;
      }
    }
  }
  drain();
  u64 other[LCAP];
#pragma unroll
  for (int i = 0; i < LCAP; ++i) other[i] = (u64)__shfl_xor((unsigned long long)best[i], 32, 64);
  merge_lists<LCAP>(best, other);
  if constexpr (!MIPS) {
    // |a|^2 + |b|^2 - 2<a,b> loses the leading digits of a small distance (unit vectors a hundredth
    // apart: errors of a few 1e-5 of the value), which is fine for picking candidates but not for
    // what the pairs are sorted by, nor for deciding the last places of the list.  So the list
    // kept so far is longer than l (LCAP entries: the launch picks LCAP = 16 for l <= 10 and 24
    // beyond); the distances of all of them are taken again as sum (a - b)^2, a chain of fused
    // multiply-adds in the order of the elements, the list is put in (distance, position) order
    // once more and its first l entries are the result.  Both lanes of a point hold the same
    // merged list by now; each takes every other entry and the two exchange the results.
    const u32 npc = lv_stride / 16u;
    const unsigned char* qbase = tiles + (u64)(qrow >> 5) * 32u * lv_stride + (u64)(qrow & 31u) * 16u;
    u64 fresh[LCAP];
#pragma unroll
    for (int j = 0; j < LCAP; ++j) {
      fresh[j] = KEY_INF;
      if (((u32)j & 1u) == half && best[j] != KEY_INF) {
        const u32 cand = (u32)(best[j] & 0xFFFFull);
        const unsigned char* cbase = tiles + (u64)(cand >> 5) * 32u * lv_stride + (u64)(cand & 31u) * 16u;
        float dd = 0.0f;
        for (u32 c = 0; c < npc; ++c) {
          const float4 a = *reinterpret_cast<const float4*>(qbase + (u64)c * 512u);
          const float4 b = *reinterpret_cast<const float4*>(cbase + (u64)c * 512u);
          float t = a.x - b.x;
          dd = __builtin_fmaf(t, t, dd);
          t = a.y - b.y;
          dd = __builtin_fmaf(t, t, dd);
          t = a.z - b.z;
          dd = __builtin_fmaf(t, t, dd);
          t = a.w - b.w;
          dd = __builtin_fmaf(t, t, dd);
        }
        fresh[j] = ((u64)dkey_from_float(dd) << 32) | cand;
      }
    }
#pragma unroll
    for (int j = 0; j < LCAP; ++j) {
      const u64 o = (u64)__shfl_xor((unsigned long long)fresh[j], 32, 64);
      fresh[j] = ((u32)j & 1u) == half ? fresh[j] : o;
    }
    sort_list<LCAP>(fresh);
#pragma unroll
    for (int j = 0; j < LCAP; ++j) best[j] = fresh[j];
  }
  if (half == 0 && q < cnt) {
#pragma unroll
    for (int j = 0; j < LCAP; ++j) {
      if ((u32)j < l) {
        const u64 o = (u64)(off + q) * l + j;
        knn_pos[o] = best[j] == KEY_INF ? (unsigned short)0xFFFF : (unsigned short)(best[j] & 0xFFFFull);
        knn_d[o] = (i32)(best[j] >> 32);
      }
    }
  }
}

// NS consecutive steps of a bitonic merge (strides jtop, jtop / 2, ... >= 64) over the P keys in
// LDS, for the stage that builds runs of k2 keys: the keys whose positions differ only in the NS
// stride bits exchange among themselves alone, so one thread reads those 2^NS keys, takes the
// steps in registers and writes them back.
template <int NS>
__device__ __forceinline__ void lds_steps(u64* ek, u32 P, u32 k2, u32 jtop, u32 tid) {
  constexpr u32 NK = 1u << NS;
  const u32 jlow = jtop >> (NS - 1);
  for (u32 g = tid; g < (P >> NS); g += 1024) {
    const u32 i = ((g & ~(jlow - 1u)) << NS) | (g & (jlow - 1u));  // the stride bits clear
    const bool asc = (i & k2) == 0;
    u64 v[NK];
#pragma unroll
    for (u32 m = 0; m < NK; ++m) v[m] = ek[i + m * jlow];
#pragma unroll
    for (u32 bit = NK >> 1; bit > 0; bit >>= 1) {
#pragma unroll
      for (u32 m = 0; m < NK; ++m) {
        if ((m & bit) == 0) {
          const u64 a = v[m], b = v[m | bit];
          const bool swap = (a > b) == asc;
          v[m] = swap ? b : a;
          v[m | bit] = swap ? a : b;
        }
      }
    }
#pragma unroll
    for (u32 m = 0; m < NK; ++m) ek[i + m * jlow] = v[m];
  }
}

// One leaf, first half: its candidate pairs (every point with its k = min(l, cnt-1) nearest),
// each once (the entry of the larger end is dropped when the smaller end lists the pair too),
// sorted by (distance, smaller position, larger position) in LDS.  The sorted pairs, as
// (smaller << 16 | larger), replace the head of the leaf's part of knn_d (from knn_d[off * l]);
// their number goes to pair_cnt[leaf].
//
// A thread keeps its NK keys in registers.  A histogram over PAIR_SPANS equal spans between the leaf's least and
// greatest distance (most pairs lie in a tenth of them) says how many keys lie below a distance, about; that number
// deals the keys into PAIR_BUCKETS buckets of two to four each, and a key's place is its bucket's first plus the
// bucket's keys below it, which it counts itself.  Where a bucket holds more than PAIR_CROWD keys (many equal distances)
// the leaf is sorted by the bitonic network instead, whose 91 steps took 49 us for a leaf of 8,192
// keys, waiting for LDS and barriers.  30 trees of a million points: 8.1 -> 4.1 ms (5.7 with
// the lists looked up in memory).
constexpr u32 PAIR_SPANS = 1024, PAIR_BUCKETS = 2048, PAIR_CROWD = 48;
template <int NK>
__global__ __launch_bounds__(1024) void hc_pairs_kernel(const u32* leaf_list, const u32* leaf_off, u32 l,
                                                       const unsigned short* knn_pos, i32* knn_d, u32* pair_cnt) {
  extern __shared__ __align__(16) unsigned char hc_smem[];
  __shared__ u32 first[PAIR_BUCKETS + 1];  // counts, then the buckets' first places
  __shared__ u32 below[PAIR_SPANS + 1];    // counts, then the keys below the span
  __shared__ u32 least, greatest, crowd, wave_total[16];
  u64* ek = reinterpret_cast<u64*>(hc_smem);  // 1024 * NK
  const u32 leaf = leaf_list[blockIdx.x];  // the launch's leaves: those of one size class
  const u32 off = leaf_off[leaf];
  const u32 cnt = leaf_off[leaf + 1] - off;
  if (cnt < 2) {
    if (threadIdx.x == 0) pair_cnt[leaf] = 0;
    return;
  }
  const u32 tid = threadIdx.x;
  const int lane = (int)(tid & 63u);
  const u32 k = l < cnt - 1u ? l : cnt - 1u;
  const u32 E = cnt * k;  // at most 1024 * NK
  for (u32 i = tid; i < PAIR_BUCKETS; i += 1024) first[i] = 0;
  below[tid] = 0;
  if (tid == 0) {
    least = 0xFFFFFFFFu;
    greatest = 0;
    crowd = 0;
  }
  // The lists go through LDS (where the sorted keys will be), two entries per word: that a list holds a point
  // is looked up in half as many places as there are pairs, and by single entries from memory it was most of
  // the kernel's time.
  unsigned short* lists = reinterpret_cast<unsigned short*>(hc_smem);
  const u32 words = (l + 1u) / 2u;  // per list
  for (u32 i = tid; i < cnt * 2u * words; i += 1024) {
    const u32 a = i / (2u * words), j = i - a * 2u * words;
    lists[i] = j < k ? knn_pos[(u64)(off + a) * l + j] : (unsigned short)0xFFFFu;
  }
  u64 key[NK];
  u32 lo = 0xFFFFFFFFu, hi = 0;
#pragma unroll
  for (int q = 0; q < NK; ++q) {  // (the distances, requested together)
    const u32 e = tid + 1024u * q, a = e / k;
    key[q] = e < E ? (u64)(u32)knn_d[(u64)(off + a) * l + (e - a * k)] << 32 : KEY_INF;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NK; ++q) {
    const u32 e = tid + 1024u * q;
    if (e < E) {
      const u32 a = e / k, j = e - a * k, b = lists[a * 2u * words + j];
      bool keep = true;
      if (a > b) {  // does b list a?
        const u32* lb = reinterpret_cast<const u32*>(lists) + b * words;
        for (u32 t = 0; t < words; ++t) {
          const u32 w = lb[t];
          keep = keep && (w & 0xFFFFu) != a && (w >> 16) != a;
        }
      }
      const u32 u = a < b ? a : b, v = a < b ? b : a;
      const u32 d = (u32)(key[q] >> 32);
      key[q] = keep ? ((u64)d << 32) | (u << 16) | v : KEY_INF;
      if (keep) {
        lo = d < lo ? d : lo;
        hi = d > hi ? d : hi;
      }
    }
  }
#pragma unroll
  for (int step = 32; step >= 1; step >>= 1) {
    const u32 olo = (u32)__shfl_xor((int)lo, step, 64), ohi = (u32)__shfl_xor((int)hi, step, 64);
    lo = olo < lo ? olo : lo;
    hi = ohi > hi ? ohi : hi;
  }
  __syncthreads();
  if (lane == 0) {
    atomicMin(&least, lo);
    atomicMax(&greatest, hi);
  }
  __syncthreads();
  const u32 from = least;
  const float scale = (float)PAIR_SPANS / ((float)(greatest - from) + 1.0f);
  auto span_at = [&](u64 x) { return (float)((u32)(x >> 32) - from) * scale; };
  auto span_of = [&](float f) { return (u32)f < PAIR_SPANS - 1u ? (u32)f : PAIR_SPANS - 1u; };
#pragma unroll
  for (int q = 0; q < NK; ++q)
    if (key[q] != KEY_INF) atomicAdd(&below[span_of(span_at(key[q]))], 1u);
  __syncthreads();
  // inclusive sum of one number per thread over the workgroup
  auto scan = [&](u32 x) {
#pragma unroll
    for (int step = 1; step < 64; step <<= 1) {
      const u32 o = (u32)__shfl_up((int)x, step, 64);
      if (lane >= step) x += o;
    }
    if (lane == 63) wave_total[tid >> 6] = x;
    __syncthreads();
    for (u32 w = 0; w < (tid >> 6); ++w) x += wave_total[w];
    __syncthreads();
    return x;
  };
  const u32 upto = scan(below[tid]);
  below[tid + 1u] = upto;
  if (tid == 0) below[0] = 0;
  __syncthreads();
  const u32 M = below[PAIR_SPANS];
  // a key's bucket, by the keys below its span and its way through it, in [0, 1]: conversions, products, sums and
  // truncations are monotone, so buckets are in the order of the distances.  (The way is one fused operation: where the
  // span's number came from a product that was rounded up, it is less than 0, and the bucket might be one that
  // keys of the span before come after.)
  const float spread = (float)PAIR_BUCKETS / (float)(M ? M : 1u);
  u32 at[NK];  // bucket << 16 | number in it
#pragma unroll
  for (int q = 0; q < NK; ++q) {
    at[q] = 0;
    if (key[q] != KEY_INF) {
      const float f = span_at(key[q]);
      const u32 sp = span_of(f), b0 = below[sp], b1 = below[sp + 1u];
      float way = f - (float)sp;
      way = __builtin_fminf(__builtin_fmaxf(way, 0.0f), 1.0f);
      u32 b = (u32)(((float)b0 + way * (float)(b1 - b0)) * spread);
      b = b < PAIR_BUCKETS - 1u ? b : PAIR_BUCKETS - 1u;
      at[q] = (b << 16) | atomicAdd(&first[b], 1u);
    }
  }
  __syncthreads();
  // exclusive scan of the counts, two per thread
  const u32 c0 = first[2u * tid], c1 = first[2u * tid + 1u];
  if (c0 > PAIR_CROWD || c1 > PAIR_CROWD) crowd = 1;
  const u32 run = scan(c0 + c1) - c0 - c1;
  first[2u * tid] = run;
  first[2u * tid + 1u] = run + c0;
  if (tid == 1023u) first[PAIR_BUCKETS] = M;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NK; ++q)
    if (key[q] != KEY_INF) ek[first[at[q] >> 16] + (at[q] & 0xFFFFu)] = key[q];
  __syncthreads();
  u32* out = reinterpret_cast<u32*>(knn_d) + (u64)off * l;
  if (tid == 0) pair_cnt[leaf] = M;
  if (crowd == 0) {
#pragma unroll
    for (int q = 0; q < NK; ++q) {
      if (key[q] != KEY_INF) {
        const u32 b = at[q] >> 16, s0 = first[b], s1 = first[b + 1u], me = s0 + (at[q] & 0xFFFFu);
        u32 place = s0;
        for (u32 t = s0; t < s1; ++t) {
          const u64 other = ek[t];
          place += other < key[q] || (other == key[q] && t < me) ? 1u : 0u;
        }
        at[q] = place;
      }
    }
    __syncthreads();
    u32* sorted = reinterpret_cast<u32*>(hc_smem);
#pragma unroll
    for (int q = 0; q < NK; ++q)
      if (key[q] != KEY_INF) sorted[at[q]] = (u32)key[q];
    __syncthreads();
    for (u32 e = tid; e < M; e += 1024) out[e] = sorted[e];
    return;
  }
  u32 P = 64;
  while (P < M) P <<= 1;  // at most 1024 * NK, a power of two
  for (u32 e = M + tid; e < P; e += 1024) ek[e] = KEY_INF;
  __syncthreads();
  // bitonic sort; the steps whose partners lie within 64 consecutive keys (more than half of all
  // steps) run in registers, one wavefront per 64 keys, with lane exchanges instead of LDS trips
  // and workgroup barriers
  for (u32 k2 = 2; k2 <= P; k2 <<= 1) {
    u32 j = k2 >> 1;
    // the steps across 64 keys or more, up to three in one trip through LDS: a thread takes the 2,
    // 4 or 8 keys that those steps exchange among themselves
    while (j >= 64) {
      if (j >= 256) {
        lds_steps<3>(ek, P, k2, j, tid);
        j >>= 3;
      } else if (j >= 128) {
        lds_steps<2>(ek, P, k2, j, tid);
        j >>= 2;
      } else {
        lds_steps<1>(ek, P, k2, j, tid);
        j >>= 1;
      }
      __syncthreads();
    }
    // four keys of a thread at a time, so that the lane exchanges of one do not wait for another's
    for (u32 i0 = tid; i0 < P; i0 += 4096) {
      u64 v[4];
      bool keep_low[4];  // this position keeps the smaller key of an exchange across bit jj ...
#pragma unroll
      for (u32 q = 0; q < 4; ++q) {
        const u32 i = i0 + 1024u * q;
        v[q] = i < P ? ek[i] : KEY_INF;
        keep_low[q] = (i & k2) == 0;  // ... when its own bit jj is clear; the other way round otherwise
      }
      // keeps its own key if that is the one wanted here: the smaller on the low side of an
      // ascending run and on the high side of a descending one (equal keys: either)
      auto settle = [&](u32 q, u32 jj, u32 olo, u32 ohi) {
        const u64 o = ((u64)ohi << 32) | olo;
        const bool want_low = (((u32)lane & jj) == 0) == keep_low[q];
        v[q] = ((v[q] < o) == want_low) ? v[q] : o;
      };
      for (u32 jj = j; jj >= 16; jj >>= 1) {  // partners 16 or 32 lanes away: through the LDS crossbar
        const int src = (int)(((u32)lane ^ jj) << 2);
#pragma unroll
        for (u32 q = 0; q < 4; ++q)
          settle(q, jj, (u32)__builtin_amdgcn_ds_bpermute(src, (int)(u32)v[q]),
                 (u32)__builtin_amdgcn_ds_bpermute(src, (int)(u32)(v[q] >> 32)));
      }
      // partners inside a row of 16 lanes: data-parallel-primitive moves.  8 away: the row turned
      // by 8.  4 away: the row turned by 12 for the lanes whose partner is above (banks 0 and 2),
      // by 4 for those whose partner is below (banks 1 and 3).
      if (j >= 8) {
#pragma unroll
        for (u32 q = 0; q < 4; ++q)
          settle(q, 8u, (u32)__builtin_amdgcn_update_dpp(0, (int)(u32)v[q], 0x128, 0xF, 0xF, true),
                 (u32)__builtin_amdgcn_update_dpp(0, (int)(u32)(v[q] >> 32), 0x128, 0xF, 0xF, true));
      }
      if (j >= 4) {
#pragma unroll
        for (u32 q = 0; q < 4; ++q) {
          const int lo = (int)(u32)v[q], hi = (int)(u32)(v[q] >> 32);
          const int olo = __builtin_amdgcn_update_dpp(__builtin_amdgcn_update_dpp(0, lo, 0x12C, 0xF, 0x5, false), lo,
                                                      0x124, 0xF, 0xA, false);
          const int ohi = __builtin_amdgcn_update_dpp(__builtin_amdgcn_update_dpp(0, hi, 0x12C, 0xF, 0x5, false), hi,
                                                      0x124, 0xF, 0xA, false);
          settle(q, 4u, (u32)olo, (u32)ohi);
        }
      }
      if (j >= 2) {  // partners inside a group of four lanes: quad_perm [2,3,0,1], then [1,0,3,2]
#pragma unroll
        for (u32 q = 0; q < 4; ++q)
          settle(q, 2u, (u32)__builtin_amdgcn_update_dpp(0, (int)(u32)v[q], 0x4E, 0xF, 0xF, true),
                 (u32)__builtin_amdgcn_update_dpp(0, (int)(u32)(v[q] >> 32), 0x4E, 0xF, 0xF, true));
      }
#pragma unroll
      for (u32 q = 0; q < 4; ++q)
        settle(q, 1u, (u32)__builtin_amdgcn_update_dpp(0, (int)(u32)v[q], 0xB1, 0xF, 0xF, true),
               (u32)__builtin_amdgcn_update_dpp(0, (int)(u32)(v[q] >> 32), 0xB1, 0xF, 0xF, true));
#pragma unroll
      for (u32 q = 0; q < 4; ++q) {
        const u32 i = i0 + 1024u * q;
        if (i < P) ek[i] = v[q];
      }
    }
    __syncthreads();
  }
  for (u32 e = tid; e < M; e += 1024) out[e] = (u32)ek[e];
}

// Second half, one wavefront per leaf: Kruskal's scan over the sorted pairs with the degree bound
// s, 64 pairs at a time.  A pair whose ends are connected, or one of whose ends is full, stays so.  Of the pairs
// that are left, all those are accepted at once that no earlier one can change: no earlier one shares
// a point with it (the degrees), and one of its two trees is touched by no earlier one (that tree
// stays apart from the other, whatever becomes of those); nor can it change an earlier one, for the same reason.
// Which is the first of a chunk to touch a tree or a point is found by a minimum over lane numbers in LDS,
// in tables so small that strangers share entries: that only sends a pair into another round.  The first pair that is
// left always passes.  A tree that no earlier pair touches goes under the other's root, the smaller under the
// larger where there is a choice (as far as the sizes are known: a root's word holds what it had when it last
// took part in such a choice).
// SLOTS false: accepted pairs go, as two arcs (point << 32 | neighbour), to arcs[2 * (off - leaf) ...] (a leaf of cnt
// points accepts at most cnt - 1; unused entries keep what they hold).  SLOTS true: to the ends' own places, slots[(tree
// * n + point) * s + k] for a point's k-th neighbour in that tree.
//
// What bounds it is the chain of LDS trips.  One pair after another, and every point put under its root
// before each chunk, took 5.6 ms for 30 trees of a million points; so 1.8.
constexpr u32 ROOT = 0x8000u;  // parent words: a root's has this bit and the size of its tree
constexpr u32 MARKS = 256;
template <bool SLOTS>
__global__ __launch_bounds__(64) void hc_kruskal_kernel(const u64* keys, const u32* leaf_off, u32 l, u32 s,
                                                        const i32* knn_d, const u32* pair_cnt, u64* arcs, u32* slots, u32 n) {
  __shared__ unsigned short parent_lds[HC_MAX_LS];
  __shared__ unsigned char deg_lds[HC_MAX_LS];
  __shared__ u32 tree_mark[MARKS], point_mark[MARKS], ring_lds[128];
  __shared__ unsigned short place_lds[SLOTS ? 128 : 1];  // which neighbours the ends are of each other
  volatile unsigned short* parent = parent_lds;
  volatile unsigned char* deg = deg_lds;
  volatile u32* ring = ring_lds;
  volatile unsigned short* place = place_lds;
  const u32 leaf = blockIdx.x;
  const u32 off = leaf_off[leaf];
  const u32 cnt = leaf_off[leaf + 1] - off;
  if (cnt < 2) return;
  const int lane = threadIdx.x;
  const u32 E = pair_cnt[leaf];
  const u32* pairs = reinterpret_cast<const u32*>(knn_d) + (u64)off * l;
  for (u32 i = (u32)lane; i < cnt; i += 64) {
    parent[i] = (unsigned short)(ROOT | 1u);
    deg[i] = 0;
  }
  for (u32 i = (u32)lane; i < MARKS; i += 64) tree_mark[i] = point_mark[i] = 0xFFFFFFFFu;
  auto order_lds = [] {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  order_lds();
  u64* out = arcs + 2ull * (off - leaf);
  u32 accepted = 0, written = 0;
  // The accepted pairs leave 64 at a time, so that the ids' loads overlap and stay out of the chain of
  // dependent steps.
  auto write_out = [&](u32 count) {
    if ((u32)lane < count) {
      const u32 mine = ring[(written + (u32)lane) & 127u];
      const u64 gu = keys[off + (mine >> 16)] & 0xFFFFFFFFull, gv = keys[off + (mine & 0xFFFFu)] & 0xFFFFFFFFull;
      if constexpr (SLOTS) {
        const u32 k = place[(written + (u32)lane) & 127u];
        u32* tree = slots + (u64)(off / n) * n * s;
        tree[gu * s + (k >> 8)] = (u32)gv;
        tree[gv * s + (k & 0xFFu)] = (u32)gu;
      } else {
        out[2 * (written + (u32)lane)] = (gu << 32) | gv;
        out[2 * (written + (u32)lane) + 1] = (gv << 32) | gu;
      }
    }
    written += count;
  };
  u32 turn = 0x3FFFFFFu;  // falls with every round, so that a round's marks lie below all earlier ones
  u32 ahead = (u32)lane < E ? pairs[lane] : 0u, last = 0xFFFFFFFFu;  // (no pair: its ends are one point)
  for (u32 c = 0; c < E && accepted < cnt - 1u; c += 64) {
    const u32 e = c + (u32)lane, pr = ahead;
    ahead = e + 64u < E ? pairs[e + 64u] : 0u;  // the next chunk's, requested early
    const u32 left = (u32)__shfl_up((int)pr, 1, 64);
    const bool dup = pr == (lane == 0 ? last : left);
    last = readlane_u32(pr, 63);
    const u32 u = pr >> 16, v = pr & 0xFFFFu;
    bool act = e < E && !dup;
    u32 ru = u, rv = v;
    u64 taken = 0;  // the chunk's accepted pairs
    u32 du = 0, dv = 0;
    bool entered = false;
    for (;;) {
      u32 pu = 0, pv = 0;
      if (act) {
        pu = parent[ru];
        pv = parent[rv];
        du = deg[u];
        dv = deg[v];
        while (!(pu & ROOT)) {
          ru = pu;
          pu = parent[ru];
        }
        while (!(pv & ROOT)) {
          rv = pv;
          pv = parent[rv];
        }
        act = ru != rv && du < s && dv < s;
      }
      order_lds();
      if (!entered && act) {  // the way is as short for whoever asks next
        if (ru != u) parent[u] = (unsigned short)ru;
        if (rv != v) parent[v] = (unsigned short)rv;
      }
      entered = true;
      if (ballot(act) == 0ull) break;
      const u32 sign = (turn << 6) | (u32)lane;
      --turn;
      if (act) {
        atomicMin(&tree_mark[ru % MARKS], sign);
        atomicMin(&tree_mark[rv % MARKS], sign);
        atomicMin(&point_mark[u % MARKS], sign);
        atomicMin(&point_mark[v % MARKS], sign);
      }
      order_lds();
      bool take = false, own_u = false, own_v = false;
      if (act) {
        own_u = *(volatile u32*)&tree_mark[ru % MARKS] == sign;
        own_v = *(volatile u32*)&tree_mark[rv % MARKS] == sign;
        take = (own_u || own_v) && *(volatile u32*)&point_mark[u % MARKS] == sign &&
               *(volatile u32*)&point_mark[v % MARKS] == sign;
      }
      order_lds();
      if (take) {
        const bool under_v = own_u && (!own_v || (pu & ~ROOT) <= (pv & ~ROOT));
        parent[under_v ? ru : rv] = (unsigned short)(under_v ? rv : ru);
        if (own_u && own_v) parent[under_v ? rv : ru] = (unsigned short)(ROOT | ((pu & ~ROOT) + (pv & ~ROOT)));
        deg[u] = (unsigned char)(du + 1u);
        deg[v] = (unsigned char)(dv + 1u);
        act = false;
      }
      taken |= ballot(take);
      order_lds();
    }
    if ((taken >> lane) & 1ull) {
      const u32 at = (accepted + (u32)__builtin_popcountll(taken & lanemask_lt(lane))) & 127u;
      ring[at] = pr;
      if constexpr (SLOTS) place[at] = (unsigned short)(du << 8 | dv);
    }
    accepted += (u32)__builtin_popcountll(taken);
    order_lds();
    if (accepted - written >= 64u) write_out(64u);
  }
  write_out(accepted - written);
}

// ---- repeated keys out of a sorted array --------------------------------------------------
constexpr u32 UQ_TILE = 2048;  // keys per workgroup of 256 threads

__device__ __forceinline__ bool uq_keep(const u64* keys, u64 i, u64 n) {
  return i < n && keys[i] != KEY_INF && (i == 0 || keys[i] != keys[i - 1]);
}

// The neighbours that up to COLLECT_MAX slots (trees times s) name for each point, each once, as the keys and work list items
// of the final prune: in place of sorting all arcs by point and neighbour, eight passes over 480 MB for 30
// trees of a million points.  A workgroup stages the slots of 64 points, which lie together tree by tree, in LDS; a wave
// takes a point, and an id's first appearance is found in a small hash table in LDS.  Which place a point's keys
// get among the others' depends on timing and has no influence on any result.  30 trees of a million points: sort, removal of
// repeated arcs and planning 6.6 ms, this 0.56 (and 0.6 more in the scan of the trees, whose writes go to the
// points' own places).
constexpr u32 COLLECT_MAX = 96, COLLECT_POINTS = 64, COLLECT_WAVES = 4, COLLECT_HASH = 256;
__global__ __launch_bounds__(64 * COLLECT_WAVES) void hc_collect_kernel(MergeArgs a, const u32* slots, u32 n, u32 T, u32 s, u64* keys,
                                                                        u32* key_count) {
  __shared__ u32 ids[COLLECT_POINTS][COLLECT_MAX + 1];
  __shared__ u32 table_lds[COLLECT_WAVES][COLLECT_HASH];
  __shared__ u32 found[COLLECT_POINTS], before[COLLECT_POINTS], cnt_lds[4], base_lds[4], stat_lds[2], key_base;
  const u32 t = threadIdx.x, lane = t & 63u, w = t >> 6;
  const u32 p0 = blockIdx.x * COLLECT_POINTS, np = n - p0 < COLLECT_POINTS ? n - p0 : COLLECT_POINTS;
  if (t < 4) cnt_lds[t] = 0;
  if (t < 2) stat_lds[t] = 0;
  for (u32 tree = w; tree < T; tree += COLLECT_WAVES) {
    const u32* in = slots + ((u64)tree * n + p0) * s;
    for (u32 i = lane; i < np * s; i += 64) ids[i / s][tree * s + i % s] = in[i];
  }
  __syncthreads();
  u32* table = table_lds[w];
  const u32 m = T * s;  // at most COLLECT_MAX
  for (u32 p = w; p < np; p += COLLECT_WAVES) {
    for (u32 i = lane; i < COLLECT_HASH; i += 64) table[i] = NONE_ID;
    const u32 x[2] = {lane < m ? ids[p][lane] : NONE_ID, lane + 64u < m ? ids[p][lane + 64u] : NONE_ID};
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    u32 c = 0;
#pragma unroll
    for (u32 q = 0; q < 2; ++q) {
      bool fresh = false;
      if (x[q] != NONE_ID) {
        // (at most 96 of 256 places are taken, so there is an end)
        for (u32 h = (x[q] * 0x9E3779B1u) >> 24;; h = (h + 1u) & (COLLECT_HASH - 1u)) {
          const u32 was = atomicCAS(&table[h], NONE_ID, x[q]);
          fresh = was == NONE_ID;
          if (fresh || was == x[q]) break;
        }
      }
      const u64 fm = ballot(fresh);
      if (fresh) ids[p][c + (u32)__builtin_popcountll(fm & lanemask_lt((int)lane))] = x[q];
      c += (u32)__builtin_popcountll(fm);
    }
    if (lane == 0) found[p] = c;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  if (w == 0) {
    const u32 c = lane < np ? found[lane] : 0u;
    u32 incl = c;
#pragma unroll
    for (u32 off = 1; off < 64; off <<= 1) {
      const u32 o = (u32)__shfl_up((int)incl, off, 64);
      if (lane >= off) incl += o;
    }
    before[lane] = incl - c;
    if (lane == 63) key_base = atomicAdd(key_count, incl);
  }
  int kind = -1;
  u32 slot = 0;
  __syncthreads();
  if (t < np && found[t] != 0) {
    kind = plan_segment(a, p0 + t, 0u, found[t], stat_lds, [](u32) { return 0u; });  // (force_prune: nothing is appended)
    slot = atomicAdd(&cnt_lds[kind], 1u);
  }
  for (u32 p = w; p < np; p += COLLECT_WAVES)
    for (u32 i = lane; i < found[p]; i += 64) keys[key_base + before[p] + i] = ((u64)(p0 + p) << 32) | ids[p][i];
  __syncthreads();
  plan_reserve(a, cnt_lds, base_lds, stat_lds);
  __syncthreads();
  if (kind >= 0) plan_file(a, kind, base_lds[kind] + slot, key_base + before[t], found[t], p0 + t, 0u);
}


__global__ __launch_bounds__(256) void uq_count_kernel(const u64* keys, u64 n, u32* counts) {
  __shared__ u32 total;
  if (threadIdx.x == 0) total = 0;
  __syncthreads();
  const u64 base = (u64)blockIdx.x * UQ_TILE + threadIdx.x * 8u;
  u32 c = 0;
  for (u32 k = 0; k < 8; ++k) c += uq_keep(keys, base + k, n) ? 1u : 0u;
  atomicAdd(&total, c);
  __syncthreads();
  if (threadIdx.x == 0) counts[blockIdx.x] = total;
}

// counts[0..m) -> exclusive prefix sums in place, the grand total in counts[m]
__global__ __launch_bounds__(1024) void uq_scan_kernel(u32* counts, u32 m) {
  __shared__ unsigned long long part[1024];
  const u32 t = threadIdx.x;
  const u32 per = (m + 1023u) / 1024u;
  const u32 lo = t * per < m ? t * per : m, hi = lo + per < m ? lo + per : m;
  unsigned long long s = 0;
  for (u32 i = lo; i < hi; ++i) s += counts[i];
  part[t] = s;
  __syncthreads();
  for (u32 o = 1; o < 1024; o <<= 1) {
    const unsigned long long v = t >= o ? part[t - o] : 0ull;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  unsigned long long run = t ? part[t - 1] : 0ull;
  for (u32 i = lo; i < hi; ++i) {
    const u32 v = counts[i];
    counts[i] = (u32)run;
    run += v;
  }
  if (t == 1023) counts[m] = (u32)part[1023];
}

__global__ __launch_bounds__(256) void uq_scatter_kernel(const u64* keys, u64 n, const u32* offsets, u64* out) {
  __shared__ u32 pre[256];
  const u32 t = threadIdx.x;
  const u64 base = (u64)blockIdx.x * UQ_TILE + t * 8u;
  bool keep[8];
  u32 c = 0;
  for (u32 k = 0; k < 8; ++k) {
    keep[k] = uq_keep(keys, base + k, n);
    c += keep[k] ? 1u : 0u;
  }
  pre[t] = c;
  __syncthreads();
  for (u32 o = 1; o < 256; o <<= 1) {
    const u32 v = t >= o ? pre[t - o] : 0u;
    __syncthreads();
    pre[t] += v;
    __syncthreads();
  }
  u64 w = (u64)offsets[blockIdx.x] + (t ? pre[t - 1] : 0u);
  for (u32 k = 0; k < 8; ++k)
    if (keep[k]) out[w++] = keys[base + k];
}

// ---- a stable two-way split of every node, without a sort -------------------------------------
// With L(i) = number of left points before position i, a point of the node [a, b) with nl = L(b) - L(a)
// left points goes to a + (L(i) - L(a)) if it is a left point and to a + nl + (i - a) - (L(i) - L(a))
// otherwise.  The side kernels leave one bit per position.
constexpr u32 SP_TILE = 2048;  // positions per workgroup of 256 threads

// the left points among the positions 64 w .. 64 w + 63 that lie below `end`, as a mask
__device__ __forceinline__ u64 left_mask(const u32* right, u64 w, u64 end) {
  const u64 first = 64u * w;
  if (first >= end) return 0ull;
  u64 r = right[2u * w];
  if (first + 32u < end) r |= (u64)right[2u * w + 1u] << 32;
  const u64 live = end - first >= 64u ? ~0ull : (1ull << (end - first)) - 1ull;
  return ~r & live;
}

__device__ __forceinline__ u32 wave_sum(u32 c) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) c += (u32)__shfl_xor((int)c, o, 64);
  return c;
}

// left points per tile; one wavefront each
__global__ __launch_bounds__(64) void hc_count_left_kernel(const u32* right, u64 m, u32* tile_cnt) {
  u32 c = 0;
  if (threadIdx.x < SP_TILE / 64u)
    c = (u32)__builtin_popcountll(left_mask(right, (u64)blockIdx.x * (SP_TILE / 64u) + threadIdx.x, m));
  c = wave_sum(c);
  if (threadIdx.x == 0) tile_cnt[blockIdx.x] = c;
}

// Lb[j] = L(woff[j]) for the nact + 1 node boundaries; one wavefront each
__global__ __launch_bounds__(64) void hc_seg_left_kernel(const u32* right, const u32* woff, const u32* tile_off, u32* Lb) {
  const u64 a = woff[blockIdx.x];
  const u64 t = a / SP_TILE;
  u32 c = 0;
  if (threadIdx.x < SP_TILE / 64u) c = (u32)__builtin_popcountll(left_mask(right, t * (SP_TILE / 64u) + threadIdx.x, a));
  c = wave_sum(c);
  if (threadIdx.x == 0) Lb[blockIdx.x] = tile_off[t] + c;
}

// Every point to its place: the split position sp inside its node as above, then the child that
// covers sp (children 2 seg and 2 seg + 1 start at cstart[..]) and from there either the final
// order (a finished child, dest = its first final position) or the next level's work array (top
// bit of dest set).
__global__ __launch_bounds__(256) void hc_split_route_kernel(const u32* ids, const u32* right, u64 m, const u32* woff,
                                                             u32 nact, const u32* Lb, const u32* tile_off,
                                                             const u32* cstart, const u32* dest, u64* final_keys,
                                                             u32* next_work) {
  // The tile's 2,048 positions in eight rows of 256: a wavefront reads 64 neighbouring ids at a
  // time and writes the left ones (and the right ones) of a node to neighbouring places.
  __shared__ u32 before[32];  // left points of the tile before row k's quarter w, at [4 k + w]
  const u32 t = threadIdx.x, w = (u32)__builtin_amdgcn_readfirstlane((int)(t >> 6));
  const int lane = (int)(t & 63u);
  const u64 tile0 = (u64)blockIdx.x * SP_TILE;
  u32 id[8];
  u64 lefts[8];
#pragma unroll
  for (u32 k = 0; k < 8; ++k) {
    const u64 i = tile0 + 256u * k + t;
    id[k] = i < m ? ids[i] : 0u;
    lefts[k] = left_mask(right, tile0 / 64u + 4u * k + w, m);
    if (lane == 0) before[4 * k + w] = (u32)__builtin_popcountll(lefts[k]);
  }
  __syncthreads();
  if (t < 32) {  // exclusive running sums of the 32 counts
    const u32 own = before[t];
    u32 v = own;
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) {
      const u32 up = (u32)__shfl_up((int)v, o, 64);
      if ((int)t >= o) v += up;
    }
    before[t] = v - own;
  }
  __syncthreads();
  const u64 first = tile0 + 64u * w;  // the wavefront's first position: its node by a uniform search
  if (first >= m) return;
  u32 lo = side_first_node(woff, nact, first);
  const u32 tile_left = tile_off[blockIdx.x];
#pragma unroll
  for (u32 k = 0; k < 8; ++k) {
    const u64 i = tile0 + 256u * k + t;
    if (i >= m) break;
    const bool left = (lefts[k] >> lane) & 1ull;
    const u32 L = tile_left + before[4 * k + w] + (u32)__builtin_popcountll(lefts[k] & lanemask_lt(lane));
    while ((u64)woff[lo + 1] <= i) ++lo;
    const u32 a = woff[lo], La = Lb[lo], nl = Lb[lo + 1] - La;
    const u32 lr = L - La;  // left points of the node before this one
    const u32 sp = left ? a + lr : a + nl + ((u32)i - a - lr);
    const u32 r = sp >= cstart[2 * lo + 1] ? 2 * lo + 1 : 2 * lo;
    const u32 d = dest[r];
    const u64 kk = sp - cstart[r];
    if (d & 0x80000000u)
      next_work[(u64)(d & 0x7FFFFFFFu) + kk] = id[k];
    else
      final_keys[(u64)d + kk] = id[k];
  }
}

template <class Id>
__global__ __launch_bounds__(256) void hc_iota_mod_kernel(Id* ids, u64 n, u64 total) {
  const u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < total) ids[i] = (Id)(i % n);
}

struct Seg {
  u64 goff, cnt, node, woff;  // place in the final order, size, heap number, place in the work array
  u32 depth, tree;
};
struct Leaf {
  u64 goff, cnt;
};

// Everything one group of trees needs on the device.  The trees of a group are cut side by side:
// tree g of the group owns the positions g*n .. (g+1)*n of every array.
struct HcCtx {
  u64 n = 0, N = 0;  // points; positions of a full group
  u32 G = 1;
  u32 row_bytes = 0, lv_stride = 0;
  bool is_signed = false;
  bool is_f32 = false, is_mips = false;
  const unsigned char* pts = nullptr;
  u32 Ls = 0, s = 0, l = 0;
  u64 seed = 0;
  DevBuf final_keys, work[2], right, segbuf, routebuf, tilebuf, first, leafvec, leafnorm, leaf_off, knn_pos, knn_d, pair_cnt, leaf_list;
  u64 pair_cnt_cap = 0;
  u64 leaf_tiles = 0;  // tiles of 32 rows that leafvec holds
  u64 seg_words = 0;
  HostBuf h_up, h_route, h_first;  // a level's node table, its routing table, the left counts read back
  // test hook (ann_hcnng_leaf_knn): host arrays that receive every point's neighbour positions
  // and distance keys as the nearest-neighbour kernel leaves them
  unsigned short* dump_pos = nullptr;
  i32* dump_d = nullptr;
  int alloc() {
    HIP_TRY(final_keys.alloc(N * 8));
    for (auto& k : work) HIP_TRY(k.alloc(N * 4));
    HIP_TRY(right.alloc((N / 32 + 2) * 4));
    // nodes that split at one level: each holds more than Ls points
    const u64 nact = N / ((u64)Ls + 1) + G + 1;
    seg_words = 8 * nact + 16;
    HIP_TRY(segbuf.alloc(seg_words * 4));
    HIP_TRY(routebuf.alloc(seg_words * 4));
    HIP_TRY(h_up.alloc(seg_words * 4));
    HIP_TRY(h_route.alloc(seg_words * 4));
    HIP_TRY(h_first.alloc((2 * nact + 2) * 4));
    HIP_TRY(tilebuf.alloc((N / SP_TILE + 4) * 4));
    HIP_TRY(first.alloc((2 * nact + 2) * 4));
    // every leaf but a tree's smallest few is well above 32 points: room for one partly used tile
    // per Ls / 4 positions (hc_leaves allocates again if a group needs more)
    leaf_tiles = N / 32 + 4 * (N / Ls) + G + 64;
    // test-only option of ann_hcnng_build (see ann.h): start with one tile, so that hc_leaves
    // takes the path that allocates the buffer again
    if (getenv("ANN_HCNNG_FEW_TILES") != nullptr) leaf_tiles = 1;
    HIP_TRY(leafvec.alloc(leaf_tiles * 32 * lv_stride));
    HIP_TRY(leafnorm.alloc((N + 64) * 4));
    HIP_TRY(leafnorm.al.zero(leafnorm.p, (N + 64) * 4));
    HIP_TRY(leaf_off.alloc(2 * (N + 1) * 4));
    HIP_TRY(knn_pos.alloc(N * l * 2));
    HIP_TRY(knn_d.alloc(N * l * 4));
    return ANN_OK;
  }
};

// The cluster trees tree0 .. tree0+G-1, level by level, all of them in the same launches.  Only
// the points of nodes that still split are worked on: a node's place in the final order is known
// when it is made (children share their parent's range), so finished nodes are copied there and
// the rest is packed for the next level.  On return final_keys holds the point ids (low words),
// tree after tree, leaf after leaf, and `leaves` the leaves in that order.
int hc_partition(HcCtx& X, u32 tree0, u32 G, std::vector<Leaf>& leaves, hipStream_t st) {
  const u64 n = X.n, N = (u64)G * n;
  leaves.clear();
  if (n <= X.Ls) {
    hipLaunchKernelGGL(hc_iota_mod_kernel<u64>, dim3((u32)((N + 255) / 256)), dim3(256), 0, st, X.final_keys.as<u64>(), n, N);
    HIP_TRY(hipGetLastError());
    for (u32 g = 0; g < G; ++g) leaves.push_back(Leaf{(u64)g * n, n});
    return ANN_OK;
  }
  hipLaunchKernelGGL(hc_iota_mod_kernel<u32>, dim3((u32)((N + 255) / 256)), dim3(256), 0, st, X.work[0].as<u32>(), n, N);
  HIP_TRY(hipGetLastError());
  std::vector<Seg> act, next;
  for (u32 g = 0; g < G; ++g) act.push_back(Seg{(u64)g * n, n, 1, (u64)g * n, 0, tree0 + g});
  u64 m = N;
  u32 in = 0;  // which of the two work arrays holds this level's points
  while (!act.empty()) {
    const u32 nact = (u32)act.size();
    if (8ull * nact + 16 > X.seg_words) return fail(ANN_EINTERNAL, "more splitting nodes than planned for");
    // woff[nact+1] | pos1[nact] | pos2[nact]
    // (the host tables are free again: the wait in the middle of the previous level came after
    // this table's copy, and the routing table is not written before this level's wait)
    u32* woff = X.h_up.as<u32>();
    std::fill(woff, woff + (size_t)3 * nact + 1, HC_NONE);
    u32* pos1 = woff + nact + 1;
    u32* pos2 = pos1 + nact;
    for (u32 j = 0; j < nact; ++j) {
      const Seg& sg = act[j];
      woff[j] = (u32)sg.woff;
      if (sg.depth < HC_MAX_DEPTH) {
        const u64 k = 2 * (((u64)sg.tree << 40) + sg.node);
        const u64 i1 = mulhi64(stream_output(X.seed, k), sg.cnt);
        u64 i2 = mulhi64(stream_output(X.seed, k + 1), sg.cnt - 1);
        if (i2 >= i1) ++i2;
        pos1[j] = (u32)(sg.woff + i1);
        pos2[j] = (u32)(sg.woff + i2);
      }
    }
    woff[nact] = (u32)m;
    u32* d_seg = X.segbuf.as<u32>();
    HIP_TRY(hipMemcpyAsync(d_seg, woff, ((size_t)3 * nact + 1) * 4, hipMemcpyHostToDevice, st));
    const u32* ids = X.work[in].as<u32>();
    const u32* right = X.right.as<u32>();
    const u32 per_block = 4 * (X.is_f32 ? SIDE_PER_WAVE_F32 : SIDE_PER_WAVE);
    const u32 grid_side = (u32)((m + per_block - 1) / per_block);
#define HC_SIDE(KERNEL)                                                                                       \
  hipLaunchKernelGGL(KERNEL, dim3(grid_side), dim3(256), 0, st, X.pts, X.row_bytes, ids, m, d_seg, nact,      \
                     d_seg + nact + 1, d_seg + 2 * nact + 1, X.right.as<u32>())
    if (X.is_f32 && X.is_mips)
      HC_SIDE(hc_side_f32_kernel<true>);
    else if (X.is_f32)
      HC_SIDE(hc_side_f32_kernel<false>);
    else if (X.is_signed)
      HC_SIDE(hc_side_kernel<true>);
    else
      HC_SIDE(hc_side_kernel<false>);
#undef HC_SIDE
    HIP_TRY(hipGetLastError());
    // left points per tile, their running sums, and L at every node boundary
    const u32 ntiles = (u32)((m + SP_TILE - 1) / SP_TILE);
    u32* d_tile = X.tilebuf.as<u32>();
    u32* d_Lb = X.first.as<u32>();
    hipLaunchKernelGGL(hc_count_left_kernel, dim3(ntiles), dim3(64), 0, st, right, m, d_tile);
    hipLaunchKernelGGL(uq_scan_kernel, dim3(1), dim3(1024), 0, st, d_tile, ntiles);
    hipLaunchKernelGGL(hc_seg_left_kernel, dim3(nact + 1), dim3(64), 0, st, right, d_seg, d_tile, d_Lb);
    HIP_TRY(hipGetLastError());
    const u32* h_first = X.h_first.as<u32>();
    HIP_TRY(hipMemcpyAsync(X.h_first.p, d_Lb, ((size_t)nact + 1) * 4, hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    // the children: the split leaves every node in its range of the work array
    next.clear();
    u32* cstart = X.h_route.as<u32>();  // cstart[2 nact + 1] | dest[2 nact]
    u32* dest = cstart + 2 * nact + 1;
    u64 nm = 0;
    for (u32 j = 0; j < nact; ++j) {
      const Seg& sg = act[j];
      u64 cl;
      const u64 nl = h_first[j + 1] - h_first[j];
      if (pos1[j] == HC_NONE || nl == 0 || nl == sg.cnt)
        cl = (sg.cnt + 1) / 2;  // too deep, or nothing separated: the order is cut in the middle
      else
        cl = nl;
      const u64 ccnt[2] = {cl, sg.cnt - cl};
      const u64 cgo[2] = {sg.goff, sg.goff + cl};
      const u64 cws[2] = {sg.woff, sg.woff + cl};
      for (int c = 0; c < 2; ++c) {
        cstart[2 * j + c] = (u32)cws[c];
        if (ccnt[c] <= X.Ls) {
          dest[2 * j + c] = (u32)cgo[c];
          leaves.push_back(Leaf{cgo[c], ccnt[c]});
        } else {
          dest[2 * j + c] = 0x80000000u | (u32)nm;
          next.push_back(Seg{cgo[c], ccnt[c], 2 * sg.node + (u64)c, nm, sg.depth + 1, sg.tree});
          nm += ccnt[c];
        }
      }
    }
    cstart[2 * nact] = (u32)m;
    u32* d_route = X.routebuf.as<u32>();
    HIP_TRY(hipMemcpyAsync(d_route, cstart, ((size_t)4 * nact + 1) * 4, hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(hc_split_route_kernel, dim3(ntiles), dim3(256), 0, st, ids, right, m, d_seg, nact, d_Lb, d_tile,
                       d_route, d_route + 2 * nact + 1, X.final_keys.as<u64>(), X.work[1 - in].as<u32>());
    HIP_TRY(hipGetLastError());
    in = 1 - in;
    act.swap(next);
    m = nm;
  }
  HIP_TRY(hipStreamSynchronize(st));  // the host tables may be written again
  std::sort(leaves.begin(), leaves.end(), [](const Leaf& a, const Leaf& b) { return a.goff < b.goff; });
  return ANN_OK;
}

// Leaves -> nearest neighbours -> degree-bounded trees, for a whole group; the accepted pairs of
// the group's j-th leaf land, as arcs, at arcs[2 * (goff_j - j) ...], or, where `slots` is given, there.
int hc_leaves(HcCtx& X, u32 G, const std::vector<Leaf>& leaves, u64* arcs, u32* slots, hipStream_t st) {
  const u64 N = (u64)G * X.n;
  const u32 nleaves = (u32)leaves.size();
  // leaf_off[nleaves + 1] | tile_of_leaf[nleaves + 1]: where a leaf's points and its tiles of 32 begin
  std::vector<u32> lo(2 * ((size_t)nleaves + 1));
  u32* lt = lo.data() + nleaves + 1;
  u64 maxc = 0, ntile = 0;
  for (u32 j = 0; j < nleaves; ++j) {
    lo[j] = (u32)leaves[j].goff;
    lt[j] = (u32)ntile;
    ntile += (leaves[j].cnt + 31) / 32;
    maxc = std::max(maxc, leaves[j].cnt);
  }
  lo[nleaves] = (u32)N;
  lt[nleaves] = (u32)ntile;
  if (ntile > X.leaf_tiles) {  // many small leaves: more partly used tiles than planned for
    HIP_TRY(hipStreamSynchronize(st));
    HIP_TRY(X.leafvec.alloc(ntile * 32 * X.lv_stride));
    X.leaf_tiles = ntile;
  }
  HIP_TRY(hipMemcpyAsync(X.leaf_off.p, lo.data(), lo.size() * 4, hipMemcpyHostToDevice, st));
  HIP_TRY(hipStreamSynchronize(st));  // lo goes out of scope
  const u32* d_leaf_off = X.leaf_off.as<u32>();
  const u32* d_tile_of_leaf = d_leaf_off + nleaves + 1;
  if (X.is_f32)
    hipLaunchKernelGGL(hc_gather_f32_kernel, dim3((u32)ntile), dim3(256), 0, st, X.pts, X.row_bytes, X.final_keys.as<u64>(),
                       d_leaf_off, d_tile_of_leaf, nleaves, X.lv_stride, X.leafvec.as<unsigned char>(),
                       X.leafnorm.as<float>());
  else if (X.is_signed)
    hipLaunchKernelGGL(hc_gather_kernel<true>, dim3((u32)ntile), dim3(256), 0, st, X.pts, X.row_bytes,
                       X.final_keys.as<u64>(), d_leaf_off, d_tile_of_leaf, nleaves, X.lv_stride,
                       X.leafvec.as<unsigned char>(), X.leafnorm.as<i32>());
  else
    hipLaunchKernelGGL(hc_gather_kernel<false>, dim3((u32)ntile), dim3(256), 0, st, X.pts, X.row_bytes,
                       X.final_keys.as<u64>(), d_leaf_off, d_tile_of_leaf, nleaves, X.lv_stride,
                       X.leafvec.as<unsigned char>(), X.leafnorm.as<i32>());
  HIP_TRY(hipGetLastError());
  const u32 kny = (u32)((maxc + 31) / 32);
  const dim3 kgrid((u32)(((u64)nleaves + 7) / 8 * 8 * kny));
#define HC_KNN(KERNEL, NORMT)                                                                                       \
  hipLaunchKernelGGL(KERNEL, kgrid, dim3(64), 0, st, X.leafvec.as<unsigned char>(), X.leafnorm.as<NORMT>(), X.lv_stride, \
                     d_leaf_off, d_tile_of_leaf, X.l, X.knn_pos.as<unsigned short>(), X.knn_d.as<i32>(), (u32)nleaves, kny)
  if (X.is_f32 && X.is_mips) {
    if (X.l <= 10)
      HC_KNN((hc_knn_f32_kernel<10, true>), float);
    else
      HC_KNN((hc_knn_f32_kernel<16, true>), float);
  } else if (X.is_f32) {
    // squared L2: a few more candidates than l are kept, see the end of the kernel
    if (X.l <= 10)
      HC_KNN((hc_knn_f32_kernel<16, false>), float);
    else
      HC_KNN((hc_knn_f32_kernel<24, false>), float);
  } else if (X.l <= 4) {
    HC_KNN(hc_knn_kernel<4>, i32);
  } else if (X.l <= 8) {
    HC_KNN(hc_knn_kernel<8>, i32);
  } else if (X.l <= 10) {
    HC_KNN(hc_knn_kernel<10>, i32);
  } else {
    HC_KNN(hc_knn_kernel<16>, i32);
  }
#undef HC_KNN
  HIP_TRY(hipGetLastError());
  if (X.dump_pos != nullptr) {
    HIP_TRY(hipMemcpyAsync(X.dump_pos, X.knn_pos.p, N * X.l * 2, hipMemcpyDeviceToHost, st));
    HIP_TRY(hipMemcpyAsync(X.dump_d, X.knn_d.p, N * X.l * 4, hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
  }
  if (X.pair_cnt_cap < nleaves) {
    HIP_TRY(hipStreamSynchronize(st));
    HIP_TRY(X.pair_cnt.alloc(((size_t)nleaves + 1) * 4));
    HIP_TRY(X.leaf_list.alloc(((size_t)nleaves + 1) * 4));
    X.pair_cnt_cap = nleaves;
  }
  // the pair sort by size class: a leaf's LDS follows from its size, and the smaller the
  // allocation the more leaves a compute unit sorts at a time
  {
    std::vector<u32> order;
    order.reserve(nleaves);
    u32 first_of[4] = {0, 0, 0, 0};
    const u32 limit[3] = {4096, 8192, HC_MAX_PAIRS};
    for (int c = 0; c < 3; ++c) {
      first_of[c] = (u32)order.size();
      for (u32 j = 0; j < nleaves; ++j) {
        const u64 cj = leaves[j].cnt;
        const u64 e = cj * (X.l < cj - 1 ? X.l : (cj > 1 ? cj - 1 : 1));
        if (e <= limit[c] && (c == 0 || e > limit[c - 1])) order.push_back(j);
      }
    }
    first_of[3] = (u32)order.size();
    HIP_TRY(hipMemcpyAsync(X.leaf_list.p, order.data(), order.size() * 4, hipMemcpyHostToDevice, st));
    HIP_TRY(hipStreamSynchronize(st));  // `order` goes out of scope
    for (int c = 0; c < 3; ++c) {
      const u32 cntc = first_of[c + 1] - first_of[c];
      if (!cntc) continue;
      const u32 lds = limit[c] * 8;
      const auto kernel = c == 0 ? hc_pairs_kernel<4> : c == 1 ? hc_pairs_kernel<8> : hc_pairs_kernel<16>;
      HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
      hipLaunchKernelGGL(kernel, dim3(cntc), dim3(1024), lds, st, X.leaf_list.as<u32>() + first_of[c], X.leaf_off.as<u32>(),
                         X.l, X.knn_pos.as<unsigned short>(), X.knn_d.as<i32>(), X.pair_cnt.as<u32>());
    }
  }
  if (slots != nullptr)
    hipLaunchKernelGGL(hc_kruskal_kernel<true>, dim3(nleaves), dim3(64), 0, st, X.final_keys.as<u64>(), X.leaf_off.as<u32>(), X.l,
                       X.s, X.knn_d.as<i32>(), X.pair_cnt.as<u32>(), nullptr, slots, (u32)X.n);
  else
    hipLaunchKernelGGL(hc_kruskal_kernel<false>, dim3(nleaves), dim3(64), 0, st, X.final_keys.as<u64>(), X.leaf_off.as<u32>(), X.l,
                       X.s, X.knn_d.as<i32>(), X.pair_cnt.as<u32>(), arcs, nullptr, (u32)X.n);
  HIP_TRY(hipGetLastError());
  return ANN_OK;
}

int hc_check(uint64_t n, uint32_t d, ann_dtype dtype, ann_metric metric, uint32_t Ls, uint32_t s, uint32_t l) {
  if (dtype != ANN_U8 && dtype != ANN_I8 && dtype != ANN_F32) return fail(ANN_EINVAL, "unknown dtype");
  if (metric != ANN_L2SQ && !(metric == ANN_MIPS && dtype == ANN_F32))
    return fail(ANN_EINVAL, "ANN_MIPS is supported for ANN_F32 only");
  if (n < 1 || n >= (1ull << 31)) return fail(ANN_EINVAL, "n must be in [1, 2^31)");
  if (dtype == ANN_F32 ? (d < 4 || d > 256) : (d < 1 || d > 128))
    return fail(ANN_EINVAL, "the clustering-based builder takes rows of at most 128 bytes (1024 for ANN_F32)");
  if (Ls < 2 || Ls > HC_MAX_LS) return fail(ANN_EINVAL, "leaf size must be in [2, 1024]");
  if (l < 1 || l > HC_MAX_L) return fail(ANN_EINVAL, "l must be in [1, 16]");
  if ((u64)Ls * l > HC_MAX_PAIRS) return fail(ANN_EINVAL, "leaf size times l must be at most 16384");
  if (s < 1 || s > 255) return fail(ANN_EINVAL, "s must be in [1, 255]");
  return ANN_OK;
}

int hc_setup(HcCtx& X, const ann_graph* g, const void* pts, uint32_t Ls, uint32_t s, uint32_t l, uint64_t seed,
             u32 G) {
  X.n = g->n;
  X.G = G;
  X.N = (u64)G * g->n;
  X.row_bytes = (u32)g->cfg.row_bytes;
  X.lv_stride = (X.row_bytes + 31u) / 32u * 32u;
  X.is_signed = g->dtype == ANN_I8;
  X.is_f32 = g->dtype == ANN_F32;
  X.is_mips = g->metric == ANN_MIPS;
  X.pts = static_cast<const unsigned char*>(pts);
  X.Ls = Ls;
  X.s = s;
  X.l = l;
  X.seed = seed;
  return X.alloc();
}

}  // namespace hcnng
}  // namespace annmi
using namespace annmi::hcnng;

extern "C" {

}  // extern "C"

// One tree: the order of its leaves, their accepted pairs and (when knn_ids is given) every
// point's nearest neighbours inside its leaf with their distances, as the kernels left them.
static int hc_one_tree(const void* points_dev, uint64_t n, uint32_t d, ann_dtype dtype, ann_metric metric,
                       uint32_t Ls, uint32_t s, uint32_t l, uint64_t seed, uint32_t tree, void* stream, uint32_t* perm_host,
                       uint64_t* leaf_off_host, uint64_t* nleaves, uint32_t* pairs_host, uint64_t* npairs,
                       uint32_t* knn_ids, void* knn_dists) {
  if (!points_dev || !perm_host || !leaf_off_host || !nleaves || (!pairs_host && !knn_ids) || (pairs_host && !npairs) ||
      (knn_ids && !knn_dists))
    return fail(ANN_EINVAL, "null argument");
  int rc = hc_check(n, d, dtype, metric, Ls, s, l);
  if (rc) return rc;
  if (tree >= (1u << 20)) return fail(ANN_EINVAL, "tree index must be below 2^20");
  hipStream_t st = static_cast<hipStream_t>(stream);
  ann_graph* g = nullptr;
  rc = new_graph(n, d, dtype, metric, 1, &g);
  if (rc) return rc;
  struct Guard {
    ann_graph* g;
    ~Guard() { ann_graph_free(g); }
  } guard{g};
  const void* pts = nullptr;
  rc = resolve_points(g, points_dev, st, &pts);
  if (rc) return rc;
  HcCtx X;
  rc = hc_setup(X, g, pts, Ls, s, l, seed, 1);
  if (rc) return rc;
  DevBuf arcs;
  HIP_TRY(arcs.alloc(2 * n * 8));
  HIP_TRY(hipMemsetAsync(arcs.p, 0xFF, 2 * n * 8, st));
  std::vector<unsigned short> kpos;
  std::vector<i32> kd;
  if (knn_ids) {
    kpos.resize(n * l);
    kd.resize(n * l);
    X.dump_pos = kpos.data();
    X.dump_d = kd.data();
  }
  std::vector<Leaf> leaves;
  rc = hc_partition(X, tree, 1, leaves, st);
  if (rc) return rc;
  rc = hc_leaves(X, 1, leaves, arcs.as<u64>(), nullptr, st);
  if (rc) return rc;
  std::vector<u64> hk(n), ha(2 * n);
  HIP_TRY(hipMemcpyAsync(hk.data(), X.final_keys.p, n * 8, hipMemcpyDeviceToHost, st));
  HIP_TRY(hipMemcpyAsync(ha.data(), arcs.p, 2 * n * 8, hipMemcpyDeviceToHost, st));
  HIP_TRY(hipStreamSynchronize(st));
  for (u64 i = 0; i < n; ++i) perm_host[i] = (u32)hk[i];
  for (size_t j = 0; j < leaves.size(); ++j) leaf_off_host[j] = leaves[j].goff;
  leaf_off_host[leaves.size()] = n;
  *nleaves = leaves.size();
  if (pairs_host) {
    u64 np = 0;
    for (u64 i = 0; i + 1 < 2 * n; i += 2)
      if (ha[i] != ~0ull) {
        pairs_host[2 * np] = (u32)(ha[i] >> 32);
        pairs_host[2 * np + 1] = (u32)ha[i];
        ++np;
      }
    *npairs = np;
  }
  if (knn_ids) {
    // positions inside the leaf -> point ids; distance keys -> distances
    for (size_t j = 0; j < leaves.size(); ++j) {
      const u64 lo = leaves[j].goff;
      for (u64 i = lo; i < lo + leaves[j].cnt; ++i)
        for (u32 t = 0; t < l; ++t) {
          const u64 o = i * l + t;
          const bool none = kpos[o] == 0xFFFFu;
          knn_ids[o] = none ? ANN_NONE : perm_host[lo + kpos[o]];
          const u32 key = (u32)kd[o];
          if (dtype == ANN_F32) {
            const u32 bits = (key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key;  // inverse of the order-preserving image
            float f;
            memcpy(&f, &bits, 4);
            static_cast<float*>(knn_dists)[o] = none ? INFINITY : f;
          } else {
            static_cast<int32_t*>(knn_dists)[o] = none ? INT32_MAX : (int32_t)key;
          }
        }
    }
  }
  return ANN_OK;
}

extern "C" {

int ann_hcnng_tree_edges(const void* points_dev, uint64_t n, uint32_t d, ann_dtype dtype, ann_metric metric,
                         uint32_t Ls, uint32_t s, uint32_t l, uint64_t seed, uint32_t tree, void* stream, uint32_t* perm_host,
                         uint64_t* leaf_off_host, uint64_t* nleaves, uint32_t* pairs_host, uint64_t* npairs) try {
  if (!pairs_host || !npairs) return fail(ANN_EINVAL, "null argument");
  return hc_one_tree(points_dev, n, d, dtype, metric, Ls, s, l, seed, tree, stream, perm_host, leaf_off_host, nleaves,
                     pairs_host, npairs, nullptr, nullptr);
} catch (...) {
  return annmi::on_exception();
}

int ann_hcnng_leaf_knn(const void* points_dev, uint64_t n, uint32_t d, ann_dtype dtype, ann_metric metric, uint32_t Ls,
                       uint32_t l, uint64_t seed, uint32_t tree, void* stream, uint32_t* perm_host,
                       uint64_t* leaf_off_host, uint64_t* nleaves, uint32_t* knn_ids_host, void* knn_dists_host) try {
  if (!knn_ids_host || !knn_dists_host) return fail(ANN_EINVAL, "null argument");
  return hc_one_tree(points_dev, n, d, dtype, metric, Ls, 1, l, seed, tree, stream, perm_host, leaf_off_host, nleaves,
                     nullptr, nullptr, knn_ids_host, knn_dists_host);
} catch (...) {
  return annmi::on_exception();
}

int ann_hcnng_build(const void* points_dev, uint64_t n, uint32_t d, ann_dtype dtype, ann_metric metric, uint32_t T,
                    uint32_t Ls, uint32_t s, uint32_t l, uint32_t R, float alpha, uint64_t seed, void* stream,
                    ann_graph** out) {
  return ann_hcnng_build_with(points_dev, n, d, dtype, metric, T, Ls, s, l, R, alpha, seed, nullptr, stream, out);
}

int ann_hcnng_build_with(const void* points_dev, uint64_t n, uint32_t d, ann_dtype dtype, ann_metric metric, uint32_t T,
                         uint32_t Ls, uint32_t s, uint32_t l, uint32_t R, float alpha, uint64_t seed,
                         const ann_hcnng_opts* opts, void* stream, ann_graph** out) try {
  if (out) *out = nullptr;
  if (!points_dev || !out) return fail(ANN_EINVAL, "null argument");
  int rc = hc_check(n, d, dtype, metric, Ls, s, l);
  if (rc) return rc;
  if (T < 1 || T >= (1u << 20)) return fail(ANN_EINVAL, "the number of trees must be in [1, 2^20)");
  if ((u64)T * 2 * n >= (1ull << 32)) return fail(ANN_EINVAL, "trees times points must stay below 2^31");
  hipStream_t st = static_cast<hipStream_t>(stream);
  Allocator al;
  if (opts && !allocator_from(opts->alloc, opts->free, opts->alloc_user, stream, &al))
    return fail(ANN_EINVAL, "alloc and free must be given together");
  AllocScope scope(al);
  const bool trace = getenv("ANN_TRACE_BUILD") != nullptr;  // wall-clock breakdown on stderr
  auto t_last = std::chrono::steady_clock::now();
  auto mark = [&](const char* what) {
    if (!trace) return;
    (void)hipStreamSynchronize(st);
    const auto now = std::chrono::steady_clock::now();
    fprintf(stderr, "[hcnng] %-28s %8.3f ms\n", what, std::chrono::duration<double, std::milli>(now - t_last).count());
    t_last = now;
  };
  ann_graph* g = nullptr;
  rc = new_graph(n, d, dtype, metric, R, &g);
  if (rc) return rc;
  struct Guard {
    ann_graph* g;
    ~Guard() {
      if (g) ann_graph_free(g);
    }
  } guard{g};
  HcCtx X;
  DevBuf arcs, arcs_tmp, big_hist, uq_counts, lists, small, arena;
  FailureWait wait;
  rc = check_insert_params(g, 1, alpha);
  if (rc) return rc;
  HIP_TRY(hipMemsetAsync(g->rows, 0xFF, (size_t)n * R * sizeof(u32), st));
  const void* pts = nullptr;
  rc = resolve_points(g, points_dev, st, &pts);
  if (rc) return rc;
  {
    u32 sv = 0;
    HIP_TRY(start_vertex_device(points_dev, n, d, dtype, st, &sv));
    g->start = sv;
  }
  // trees are cut in groups, as many at a time as keep a group within 32 million positions
  u32 G = (u32)std::max<u64>(1, (32ull << 20) / n);
  if (G > T) G = T;
  mark("graph, points, start vertex");
  rc = hc_setup(X, g, pts, Ls, s, l, seed, G);
  if (rc) return rc;
  mark("buffers of a tree group");
  const u64 total = (u64)T * 2 * n;
  // s neighbours per tree and point at most: with few of them every point has a place for each (4 T s n bytes, no more
  // than the arcs), and nothing is sorted
  const bool by_slots = s <= 4u && (u64)T * s <= COLLECT_MAX;
  if (by_slots) {
    HIP_TRY(arcs.alloc((u64)T * s * n * 4));
    HIP_TRY(hipMemsetAsync(arcs.p, 0xFF, (u64)T * s * n * 4, st));
  } else {
    HIP_TRY(arcs.alloc(total * 8));
    HIP_TRY(hipMemsetAsync(arcs.p, 0xFF, total * 8, st));
  }
  HIP_TRY(arcs_tmp.alloc(total * 8));
  mark("arc buffers");
  std::vector<Leaf> leaves;
  for (u32 t = 0; t < T; t += G) {
    const u32 Gc = T - t < G ? T - t : G;
    rc = hc_partition(X, t, Gc, leaves, st);
    if (rc) return rc;
    mark("cluster trees");
    rc = by_slots ? hc_leaves(X, Gc, leaves, nullptr, arcs.as<u32>() + (u64)t * s * n, st)
                  : hc_leaves(X, Gc, leaves, arcs.as<u64>() + (u64)t * 2 * n, nullptr, st);
    if (rc) return rc;
    mark("leaves");
    g->stats.rounds += Gc;
  }
  u32 nuniq = 0;
  if (!by_slots) {
    // all arcs by (point, neighbour): the neighbour bits first, then, stably, the point bits; the
    // unused entries (all ones) end up behind every point
    const u64 he = radix_hist_entries(total);
    HIP_TRY(big_hist.alloc(he * 4));
    const u32 idb = bits_to_hold(n);
    HIP_TRY(radix_sort_edges(arcs.as<u64>(), arcs_tmp.as<u64>(), big_hist.as<u32>(), he, total, idb, st, 0));
    HIP_TRY(radix_sort_edges(arcs.as<u64>(), arcs_tmp.as<u64>(), big_hist.as<u32>(), he, total, idb, st, 32));
    // each (point, neighbour) once
    const u32 ntiles = (u32)((total + UQ_TILE - 1) / UQ_TILE);
    HIP_TRY(uq_counts.alloc(((size_t)ntiles + 1) * 4));
    hipLaunchKernelGGL(uq_count_kernel, dim3(ntiles), dim3(256), 0, st, arcs.as<u64>(), total, uq_counts.as<u32>());
    hipLaunchKernelGGL(uq_scan_kernel, dim3(1), dim3(1024), 0, st, uq_counts.as<u32>(), ntiles);
    hipLaunchKernelGGL(uq_scatter_kernel, dim3(ntiles), dim3(256), 0, st, arcs.as<u64>(), total, uq_counts.as<u32>(),
                       arcs_tmp.as<u64>());
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipMemcpyAsync(&nuniq, uq_counts.as<u32>() + ntiles, 4, hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    mark("arcs sorted, each once");
  }
  // prune(p, neighbours, R) for every point: the re-prune kernel of BatchInsert on empty rows
  HIP_TRY(hipMemsetAsync(g->meta, 0, (size_t)n * sizeof(u32), st));
  HIP_TRY(lists.alloc(3 * n * sizeof(MergeItem)));
  HIP_TRY(small.alloc(64));
  HIP_TRY(hipMemsetAsync(small.p, 0, 64, st));
  const u64 longest = (u64)s * T;  // neighbours of one point, at most
  const u64 arena_cap = longest > MERGE_SPILL_MIN ? (u64)nuniq : 16;
  HIP_TRY(arena.alloc(arena_cap * 8));
  MergeArgs ma{};
  ma.points = static_cast<const char*>(pts);
  ma.graph = g->rows;
  ma.meta = g->meta;
  ma.R = R;
  ma.keys = arcs_tmp.as<u64>();
  ma.nkeys = nuniq;
  u32* sm = small.as<u32>();
  ma.list_count = sm + 8;
  for (int c = 0; c < 3; ++c) ma.list_items[c] = lists.as<MergeItem>() + (u64)c * n;
  ma.list_items[3] = ma.list_items[2] + (n - 1);
  ma.medium_max = gram_path_ok(g->cfg) ? 0u : MERGE_MEDIUM_MAX;
  ma.fast_amax = fast_path_amax(g->cfg);
  ma.gram_ok = gram_path_ok(g->cfg) ? 1u : 0u;
  ma.gram_tmax = gram_path_tmax();
  ma.stage_bytes = prune_stage_bytes(R, g->cfg);
  ma.use_mfma = mfma_prune_ok(R, g->cfg) ? 1u : 0u;
  ma.arena = arena.as<u64>();
  ma.arena_cap = arena_cap;
  ma.arena_top = reinterpret_cast<unsigned long long*>(sm + 4);
  ma.error_flag = sm + 2;
  ma.a16 = llround((double)alpha * 65536.0);
  ma.af = alpha;
  ma.counters = nullptr;
  ma.force_prune = 1;
  g->clean_alpha = alpha;
  if (by_slots) {
    u32* key_count = sm + 12;
    hipLaunchKernelGGL(hc_collect_kernel, dim3((u32)((n + COLLECT_POINTS - 1) / COLLECT_POINTS)), dim3(64 * COLLECT_WAVES), 0, st, ma,
                       arcs.as<u32>(), (u32)n, T, s, arcs_tmp.as<u64>(), key_count);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipMemcpyAsync(&nuniq, key_count, 4, hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    mark("neighbours, each once");
  } else {
    HIP_TRY(launch_plan(ma, st));
  }
  const u64 want = nuniq < 8192 ? nuniq : 8192;
  HIP_TRY(launch_merge(g->cfg, ma, (u32)(want ? want : 1), st, st, st, st));
  u32 flags[4] = {0, 0, 0, 0};
  HIP_TRY(hipMemcpyAsync(flags, small.p, 16, hipMemcpyDeviceToHost, st));
  HIP_TRY(hipStreamSynchronize(st));
  wait.done = true;
  if (flags[2] != 0) return fail(ANN_EINTERNAL, "merge spill arena exhausted");
  mark("prune");
  g->stats.edges = nuniq;
  guard.g = nullptr;
  *out = g;
  return ANN_OK;
} catch (...) {
  return annmi::on_exception();
}

}  // extern "C"
