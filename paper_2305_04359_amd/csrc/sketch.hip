// Sketches of float rows (sketch.hpp): the kernel that makes them, the search instances that read them, and
// the rule that says when they pay.
#include "ann_dispatch.hpp"
#include "search_kernel.hpp"

namespace annmi {

__device__ __forceinline__ u32 bf16_up(float f) {  // upper half of a float, not below f (f >= 0)
  const u32 u = __float_as_uint(f);
  return (u >> 16) + ((u & 0xFFFFu) ? 1u : 0u);
}

// Eight lanes per row; every row is read once and its sketch written once, both in whole pieces.
template <int KIND, int SK>
__global__ __launch_bounds__(256) void sketch_rows_kernel(const char* rows, u64 first, u64 count, u32 row_bytes, u32 npieces,
                                                          char* out) {
  const u64 r = ((u64)blockIdx.x * blockDim.x + threadIdx.x) >> 3;
  const int sub = threadIdx.x & (LPC - 1);
  const bool in = r < count;
  const char* row = rows + (first + (in ? r : 0)) * row_bytes;
  Piece<16> x[4 * SK];
  float most = 0.0f, sum = 0.0f;
#pragma unroll
  for (int j = 0; j < 4 * SK; ++j) {
    const u32 p = (u32)sub + LPC * j;
    x[j] = p < npieces ? load_piece<16>(row + (u64)p * 16) : zero_piece<16>();
  }
#pragma unroll
  for (int j = 0; j < 4 * SK; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float v = __uint_as_float(x[j].w[i]);
      most = __builtin_fmaxf(most, __builtin_fabsf(v));
      sum = __builtin_fmaf(v, v, sum);
    }
  most = group_max(most);
  sum = group_sum(sum);
  const bool ok = most >= SKETCH_LEAST && most <= SKETCH_MOST && sum < __builtin_inff();  // (a NaN shows in the sum)
  const u32 sbits = ok ? bf16_up(most * (1.0f / 126.5f)) : 0u;
  const float s = __uint_as_float(sbits << 16);
  const float inv = ok ? 1.0f / s : 0.0f;
  float err = 0.0f;
  u32 w[4 * SK];
#pragma unroll
  for (int j = 0; j < 4 * SK; ++j) {
    w[j] = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float v = ok ? __uint_as_float(x[j].w[i]) : 0.0f;
      const float k = __builtin_rintf(v * inv);  // at most 127: most * inv <= 126.5
      const float e = __builtin_fmaf(-s, k, v);
      err = __builtin_fmaf(e, e, err);
      w[j] |= ((u32)(int)k & 0xFFu) << (8 * i);
    }
  }
  err = __builtin_sqrtf(group_sum(err)) * 1.001f;
  if constexpr (KIND == K_F32_IP) err = __builtin_fmaf(4e-4f, __builtin_sqrtf(sum), err);
  if (sub == LPC - 1) w[4 * SK - 1] = (sbits << 16) | (ok ? bf16_up(err) : 0x7F80u);
  if (in) {
    char* o = out + (first + r) * (128u * SK) + sub * 16;
#pragma unroll
    for (int c = 0; c < SK; ++c)
      *reinterpret_cast<uint4*>(o + c * 128) = make_uint4(w[4 * c], w[4 * c + 1], w[4 * c + 2], w[4 * c + 3]);
  }
}

// Rows of at least two and a half sketches: 80 to 124 floats and 160 to 252.  (128 bytes of 256, or 256 of 512, save too
// little of what a search reads to pay for the second trip of the rows that it does read: 10,000 queries on a million
// points of 64 floats 583 -> 658 us, 5,000 on 500,000 points of 128 764 -> 994.)
u32 sketch_bytes(const DistCfg& cfg) {
  if (cfg.kind != K_F32_L2 && cfg.kind != K_F32_IP) return 0;
  if (cfg.npieces >= SKETCH_PIECES<1> && cfg.npieces < 32u) return 128;
  return cfg.npieces >= SKETCH_PIECES<2> && cfg.npieces < 64u ? 256 : 0;
}

// Sketches pay where the rows lie beyond the 256 MB of the last-level cache.  A million points of 200 floats under the
// inner product: build at R = 64, L = 128 251 -> 188 ms, 10,000 queries at L = 50 1,930 -> 1,310 us, of which
// making the sketches 175 (1.06 GB moved at 6 TB/s); the searches fetch 6.7 GB where they fetched 12.
//  - Builds gain before their rows fill that cache, which the graph and the visited lists share: 300,000 points of
//    200 floats (240 MB) 74.7 -> 62.4 ms, 150,000 in an insertion (120 MB) 62.2 -> 54.8; 200,000 of 160 at L = 64 (128
//    MB) about 1 %, 110,000 of 100 at L = 64 (44 MB) 24.7 -> 25.7.  Queries on rows that fit do not (200,000 points of
//    160 floats, sketches apart, 229 and 228 us).
//  - What searches save has to repay the sketches of all n rows.  A search takes about 24 L + 400 distances, a third
//    of which need the row after all: queries whose bytes saved are 1.9 times those spent lose 2 % (4,000 on
//    500,000 points of 160 floats, L = 40), 2.8 times gain a third (10,000 on a million of 100, L = 30: 1,031 ->
//    773 us), 14 times 1.7 (50,000 on 700,000 of 180, L = 20: 5,203 -> 3,049 us).
//  - Beams above 128: more entries, so more of a row's candidates may enter, and four waves per SIMD (20,000 queries, 500,000
//    points of 160 floats, L = 200: 3,793 -> 4,100 us).
//  - Below a beam of 16 a search is over soon after its beam has filled.
bool search_sketch_pays(const DistCfg& cfg, u64 n, u64 searches, u32 L, bool query) {
  const u64 sk = sketch_bytes(cfg), row = cfg.row_bytes;
  if (sk == 0 || L > SEARCH_SKETCH_BEAM || L < 16u) return false;
  if (n * row < (query ? 256ull << 20 : 100ull << 20)) return false;
  return searches * (24u * L + 400u) * (13u * row / 20u - sk) >= n * (row + sk) * 5u / 2u;
}

hipError_t launch_sketch_rows(const DistCfg& cfg, const void* rows, u64 first, u64 count, void* out, hipStream_t s) {
  if (count == 0) return hipSuccess;
  const dim3 grid((u32)((count + 31) / 32)), block(256);
  const char* in = static_cast<const char*>(rows);
  char* o = static_cast<char*>(out);
  const u32 rb = (u32)cfg.row_bytes;
  const bool one = sketch_bytes(cfg) == 128u;
  if (cfg.kind == K_F32_IP) {
    if (one)
      hipLaunchKernelGGL((sketch_rows_kernel<K_F32_IP, 1>), grid, block, 0, s, in, first, count, rb, cfg.npieces, o);
    else
      hipLaunchKernelGGL((sketch_rows_kernel<K_F32_IP, 2>), grid, block, 0, s, in, first, count, rb, cfg.npieces, o);
  } else {
    if (one)
      hipLaunchKernelGGL((sketch_rows_kernel<K_F32_L2, 1>), grid, block, 0, s, in, first, count, rb, cfg.npieces, o);
    else
      hipLaunchKernelGGL((sketch_rows_kernel<K_F32_L2, 2>), grid, block, 0, s, in, first, count, rb, cfg.npieces, o);
  }
  return hipGetLastError();
}

template <int KIND, int NCH, int SK>
static hipError_t launch_plain(const SearchArgs& a, const VecTable& T, hipStream_t s) {
  return launch_search_sketched<KIND, NCH, SK, false, false>(a, T, s);
}

hipError_t launch_search_sketch(const DistCfg& cfg, const SearchArgs& a, const VecTable& T, hipStream_t s) {
  ANN_DISPATCH_SKETCH(launch_plain, a, T, s);
}

}  // namespace annmi
