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
//  - Queries and insertions make them anew for every call, and what its searches save has to repay that.  A search takes
//    about 24 L + 400 distances, of which 30 % + L / 500 need the row after all; the first 2,000 + 32 L of a launch save
//    nothing (they wait for their own chains, which the sketches make longer); and what is saved counts by the
//    share of the rows that the cache can't hold, a tenth if all but fits.  Where that makes half of the bytes that
//    the making moves, 1,112 calls (100 to 252 floats, 300 to 800 MB, L = 24 to 128, 1,500 to 40,000 queries, R = 40
//    and 56) are at most 2 % slower than without and up to 45 % faster; below it calls lose up to 27 % (2,000 queries on
//    700,000 points of 124 floats, L = 128: 524 -> 665 us).  Of 596 other calls (drawn from 80 to 252 floats, 260
//    to 1,300 MB, with and without the (1 + eps) rule) three lose more than 3 %, up to 17: two that the rule ends early, one at
//    L = 17; all gain 23 % in the mean.  Insertions of 1,200 to 60,000 points: at most 4 % slower and up to 22 % faster;
//    below 256 MB of rows nearly all lose (2,500 on 128 MB 5 to 13 %).
//  - Builds search over them in dozens of launches.  On 256 MB of rows and more: 1 % slower (160 floats, L = 128, 320 MB)
//    to 26 % faster.  Below, what counts is that the query lies in LDS and leaves registers to waves.  Rows of 256-byte
//    sketches gain from 100 MB on (200 floats, R = 56, L = 128: 38.9 -> 36.9 ms at 128 MB, 55.6 -> 45.9 at 200), but those
//    of less than three sketches at beams of up to 64 lose 2 to 3 % below 150 MB.  Rows of 128-byte sketches have
//    six waves per SIMD for five: they gain where that spares a batch's searches a generation of waves (285,000 points of 112
//    floats, batches of 5,669: 42.7 -> 37.1 ms) and lose 1 to 6 % where it doesn't (335,000, 6,696: 30.8 -> 31.6).
//  - Beams above 128: more entries, so more of a row's candidates may enter, and four waves per SIMD (20,000 queries, 500,000
//    points of 160 floats, L = 200: 3,793 -> 4,100 us).
//  - Below a beam of 16 a search is over soon after its beam has filled.
void SketchUse::launch(u64 searches, u32 L) {
  const u64 idle = 2000u + 32u * L;
  largest = searches > largest ? searches : largest;
  gaining += searches > idle ? searches - idle : 0;
}
bool search_sketch_pays(const DistCfg& cfg, u64 n, u32 L, const SketchUse& use, bool build) {
  constexpr u64 cache = 256ull << 20, simds = 1024;
  const u64 sk = sketch_bytes(cfg), row = cfg.row_bytes, bytes = n * row;
  if (sk == 0 || L > SEARCH_SKETCH_BEAM || L < 16u || use.largest <= SEARCH_SKETCH_MIN) return false;
  if (build && bytes < cache) {
    if (sk == 128u) return bytes >= 100ull << 20 && (use.largest - 1u) / (5u * simds) != (use.largest - 1u) / (sketch_waves(4) * simds);
    return bytes >= (L > 64u || row >= 3u * sk ? 100ull << 20 : 150ull << 20);
  }
  if (build) return true;
  if (bytes < cache) return false;
  const double saved = (double)row * (0.7 - L / 500.0) - (double)sk;
  const double beyond = 1.1 - (double)cache / (double)bytes;
  return (double)use.gaining * (24.0 * L + 400.0) * saved * beyond >= 0.5 * (double)n * (double)(row + sk);
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
