// Host side of the beam search: sizes of the per-wave LDS, the filter layout, and the launch of
// the kernel variants without the (1 + eps) rule (the graph build and plain queries).  The
// variants with the rule, and those of the layered index, are compiled in translation units of
// their own, in parallel.
#include "ann_dispatch.hpp"
#include "search_kernel.hpp"

namespace annmi {

u32 search_lds_bytes(u32 L, u32 hash_buckets) { return search_nslot_for(L) * 64 * 8 + 64 * 8 + hash_buckets * 16; }

// Size of the visited filter.  An explicit hash_bits (log2 of the size in 32-bit words) is taken
// as it is (search_set_filter).  Otherwise, for beams of up to 256: all of the LDS that the waves a SIMD can hold
// by their registers leave to each, up to 2,048 words: one wave less costs more than a larger table
// saves, and LDS below that step is free.  A compute unit hands out its 160 KB in units of 1,280 bytes.
// `waves`: what the registers of the instance that is launched allow (search_instance_waves).
// 10,000 queries, a million 128-d uint8 points (eight waves), R = 64, L = 50: 512 words 364 us, 1,024 (that
// step) 340, 2,048 405; L = 128: 512 words 734, 896 (that step) 656, 1,216 672, 2,048 822.  Five million
// points, L = 50: 672 -> 586.  A million points of 200 floats (four waves): build 262 ms by 1,024 words, 250 by
// 2,048 (that step), 266 by 4,096; 10,000 queries at L = 50 2,055, 1,935 and 2,004 us, and by 1,664, what five waves
// would get, 0.4 % more than by 2,048; at L = 200 1,280 words 3,786, 1,920 (that step) 3,634.  Byte rows of 200 (six waves), 20,000 queries at L =
// 128: 896 words 1,498 us (uint8) and 2,128 (int8), 1,216 (that step) 1,467 and 2,098, 1,344 1,538 and 2,183.
//
// Four slots (beams of 129 to 256): some instances hold seven waves, whose 640 words cost more in repeats than the
// seventh wave brings: 20,000 queries, a million uint8 points, L = 200, eps = 0.25: seven waves 1,994 us, six (960
// words) 1,768, five (1,280) 1,850; 500,000 points of 48 floats 1,601, 1,562, 1,649.  Instances whose registers
// leave five are best at five: without the rule 1,925 us by 960 words, 1,845 by 1,280, 2,110 by 1,920.
//
// More than 2^22 points: a table of 224 buckets (beams of 65 to 128) would need 21-bit tags, one of 304,
// at six waves, still takes 16-bit tags up to 2^23 points: 20,000 queries on five million, L = 100, 1,776 -> 1,558
// us (two million, where 16 bits suffice either way, 1,226 -> 1,237); beyond, the repeats saved are worth
// the waves (10^8 points: search phase of a build 15.1 -> 14.7 s).
//
// Wider beams: 8 words per beam entry, rounded up to a power of two, but at most 1,024 words (512
// above 512 entries), then adjusted to an occupancy step: measured at beams of 200 to 2,048 on a
// hundred million points, where tables of 1,024 and 512 words answer 1.7 to 2.3 times the queries
// per second of tables of 4,096 and 8,192.  The table is never cut below 3/4 of the power of two.
constexpr u32 LDS_UNIT = 1280;
static u32 search_hash_buckets(u64 n, u32 L, u32 waves, u32 lds_more) {
  const u32 nslot = search_nslot_for(L);
  if (L < 8u) return 128;  // (over after a few hops: not worth clearing more)
  if (nslot <= 4u) {
    if ((nslot == 4u || (nslot == 2u && n > (1ull << 22))) && waves > 6u) waves = 6u;
    const u32 share = 163840u / (4u * waves) / LDS_UNIT * LDS_UNIT;
    const u32 nb = (share - search_lds_bytes(L, 0) - lds_more) / 16u;
    return nb < 512u ? nb : 512u;
  }
  u32 want = 8u * L, bits = 9;
  while ((1u << bits) < want && bits < (L > 512u ? 9u : 10u)) ++bits;
  const u32 full = 1u << (bits - 2u);
  const u32 base = search_lds_bytes(L, 0);
  const u32 lds_full = (search_lds_bytes(L, full) + 511u) & ~511u;
  u32 resident = 163840u / lds_full;
  resident = (resident + 3u) & ~3u;
  if (resident > 32u) resident = 32u;
  const u32 budget = (163840u / resident) & ~511u;
  if (budget <= base) return full;
  u32 nb = (budget - base) / 16u;
  if (nb < full - full / 4u) return full;
  if (nb > full) nb = full;
  return nb;
}

// Tags identify a vertex exactly when ids fit id_bits bits and the tag keeps the id_bits -
// floor(log2 buckets) low bits of the mixed id: 16-bit tags carry up to 15 of them (0xFFFF marks
// an empty slot), 21-bit tags up to 20.
void search_filter_mode(u64 n, u32 hash_buckets, u32* id_bits, u32* tag_width) {
  u32 bits = 1;
  while ((1ull << bits) < n) ++bits;  // ids < n <= 2^bits
  u32 q = 0;
  while ((2u << q) <= hash_buckets) ++q;  // floor(log2(buckets))
  if (bits < q + 1u) bits = q + 1u;
  *id_bits = 0;
  *tag_width = 0;
  if (bits <= 24u && bits - q <= 15u) {
    *id_bits = bits;
    *tag_width = 16;
  } else if (bits <= 31u && bits - q <= 20u) {
    *id_bits = bits;
    *tag_width = 21;
  }
}

void search_set_filter(SearchArgs& a, u32 waves, u32 lds_more) {
  a.hash_buckets = a.filter_given ? 1u << (a.filter_given - 2u) : search_hash_buckets(a.n, a.L, waves, lds_more);
  search_filter_mode(a.n, a.hash_buckets, &a.id_bits, &a.tag_width);
}

template <int KIND, int VEC, int NCH>
static hipError_t launch_plain(const SearchArgs& a, const VecTable& T, hipStream_t s, SearchPlan* plan) {
  return launch_search_variant<KIND, VEC, NCH, false, false>(a, T, s, plan);
}

static hipError_t launch_search_plain(const DistCfg& cfg, const SearchArgs& a, const VecTable& T, hipStream_t s,
                                      SearchPlan* plan) {
  ANN_DISPATCH_CFG(launch_plain, a, T, s, plan);
}

// How many waves share a search.  Up to 1,024 searches leave most of the chip idle, and each waits for
// its own chain of hops: four to eight waves take a search of a million 128-d uint8 points, R = 64,
// from 125 to 97 us at L = 64 and from 170 to 135 at L = 100 (one query), 512 of them from 242 to 168
// and 338 to 281, 1,000 of them (four waves) from 245 to 193 and 342 to 291.  2,000 searches of four
// waves do not fit the chip at once (422 -> 439 us at L = 128), and 513 to 1,024 of four waves gain
// nothing on a graph that the last-level cache holds (800 at L = 128, 40,000 to 90,000 points: 232 us
// by one wave each, 242 by four).
//
// Work ahead pays by the trips to memory it hides, and costs the first wave a longer chain per hop
// (lists, hand-over, a sorting network over all of the beam per insertion).  Measured over 5,000 to
// 1.5 million points, speed against one wave each:
//  - beams below 32 are over before it pays (L = 16: 37.4 and 37.7 us for one query), rows of 16 ids
//    bring too little work (uint8: 0.66 to 1.08, nearly all below 1);
//  - beams above 128, four slots: rows of 48 ids and more, for byte rows on graphs beyond the last-level
//    cache (float 1.06 to 1.6, uint8 there 1.0 to 1.3; with R = 32 0.7 to 1.2, byte rows on 50,000
//    points 0.8 to 1.2);
//  - rows below 48 ids, beams above 64: byte rows of up to 128 bytes on graphs beyond 16 MB (0.92 to
//    1.21; 0.87 to 1.0 for rows of 256 bytes, 0.8 to 1.1 on 5,000 points), float rows of up to 7
//    pieces per lane (1.0 to 1.4; 8 pieces 0.87 to 1.04);
//  - rows below 48 ids, beams below 48: byte rows gain for a few searches only (one to 16: 0.95 to 1.2;
//    more: 0.91 to 1.1);
//  - byte rows on graphs that one L2 holds: up to 256 searches (beyond: 0.8 to 1.05), beams above 64
//    with rows of 64 ids (0.97 to 1.4; R = 48 0.9 to 1.04).
// Up to eight searches of byte rows gain on both sides of these lines (1.02 to 1.27), but for four slots
// on short rows.
// Build searches run on a graph that is still smaller and write visited lists; the last line does not
// hold for them (2,000 points, R = 48, L = 128: build 9.5 ms, 10.9 with one wave each), the one on short
// rows from 128 searches on (R = 32, L = 128: 2,000 points 9.9 and 11.0 ms, 20,000 points 16.1 and 15.4).
constexpr u64 LAST_LEVEL_CACHE = 256ull << 20, ONE_L2 = 4ull << 20;
static u32 search_waves(const DistCfg& cfg, const SearchArgs& a) {
  const bool fits = a.R <= 64u && a.L <= 256u && a.n <= WIDE_MAX_POINTS && !a.filter_given;
  if (!fits || a.L < 32u || a.R < 32u || a.nq > 1024u) return 1;
  const u64 graph = a.n * (cfg.row_bytes + 4ull * a.R);
  const bool byte_rows = cfg.kind == K_U8 || cfg.kind == K_I8, short_rows = a.R < 48u;
  const bool build = a.vis != nullptr, lone = a.nq <= 8u;
  if (a.L > 128u && (short_rows || (byte_rows && graph <= LAST_LEVEL_CACHE && !lone))) return 1;
  if (short_rows && a.L > 64u && (byte_rows ? !lone && (cfg.nch > 1 || graph <= 4u * ONE_L2) : cfg.nch > 7) &&
      !(build && a.nq <= 128u))
    return 1;
  if (short_rows && a.L < 48u && byte_rows && a.nq > 16u) return 1;
  if (!build && !lone && byte_rows && graph <= ONE_L2 && (a.nq > 256u || (a.L > 64u && a.R < 64u))) return 1;
  if (a.nq <= 512u) return 8;
  return graph > LAST_LEVEL_CACHE ? 4 : 1;
}

// Whether the next hops' memory is requested ahead.  It costs registers and LDS (88 to 116 registers leave four or
// five waves per SIMD, the filter of 480 buckets 18 waves on a compute unit, instead of 32) and instructions (three entries of the beam looked up per hop, one in thirteen expansions undone), and
// hides one of a hop's two trips to memory: it pays while the chip is half empty.  Speed against one wave
// each without it, uint8 and int8 rows, 5,000 to 500,000 points, R = 32 to 64:
//  - 513 to 3,000 searches: 0.98 to 1.28 (2,000 uint8 searches at L = 128, R = 64: 233 -> 203 us on 100,000
//    points, 374 -> 325 on a million); 4,000: 0.95 to 1.23, 6,000: 0.70 to 1.2, most below 0.9;
//  - on graphs that one L2 holds a trip is short: 2,000 searches 0.99 to 1.09, 3,000 0.95 to 1.05;
//  - beams below 32: 0.90 to 1.08; up to 512 searches, which several waves share where that pays, 0.71 to 1.1.
// Searches that run beside others (parts of a batch) are not alone on the chip, however few.
static bool search_ahead(const DistCfg& cfg, const SearchArgs& a) {
  if (a.nq <= 512u || a.R < 32u || a.R > 64u || a.L < 32u || a.L > 128u || a.n > AHEAD_MAX_POINTS || a.filter_given || a.shares_chip) return false;
  if (cfg.kind != K_U8 && cfg.kind != K_I8) return false;
  const u64 graph = a.n * (cfg.row_bytes + 4ull * a.R);
  return a.nq <= (graph > ONE_L2 ? 3072u : 2048u);
}

// one wave per search
static hipError_t launch_search_alone(const DistCfg& cfg, const SearchArgs& a, const VecTable& T, hipStream_t s,
                                      SearchPlan* plan) {
  const bool own = a.starts != nullptr || a.next_start != nullptr;
  if (own) return a.eps16 >= 0 ? launch_search_own_eps(cfg, a, T, s, plan) : launch_search_own(cfg, a, T, s, plan);
  return a.eps16 >= 0 ? launch_search_eps(cfg, a, T, s, plan) : launch_search_plain(cfg, a, T, s, plan);
}

hipError_t launch_search(const DistCfg& cfg, const SearchArgs& a, hipStream_t s) {
  if (a.nq == 0) return hipSuccess;
  VecTable T{a.points, (u32)cfg.row_bytes, cfg.npieces};
  const u32 waves = search_waves(cfg, a);
  if (waves > 1u) return launch_search_wide(cfg, a, T, waves, s);
  if (search_ahead(cfg, a)) return launch_search_ahead(cfg, a, T, s);
  if (a.sketch != nullptr && a.L <= SEARCH_SKETCH_BEAM) {
    const bool own = a.starts != nullptr || a.next_start != nullptr;
    if (!own) return a.eps16 >= 0 ? launch_search_sketch_eps(cfg, a, T, s) : launch_search_sketch(cfg, a, T, s);
    if (a.eps16 < 0) return launch_search_sketch_own(cfg, a, T, s);
  }
  return launch_search_alone(cfg, a, T, s, nullptr);
}

hipError_t plan_search(const DistCfg& cfg, const SearchArgs& a, SearchPlan* plan) {
  return launch_search_alone(cfg, a, VecTable{a.points, (u32)cfg.row_bytes, cfg.npieces}, nullptr, plan);
}

}  // namespace annmi
