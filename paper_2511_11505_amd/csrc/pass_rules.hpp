// Which kernel runs a pass of the grouped GEMM.  Plain C++, so that the rules
// can be built and checked without a GPU; cus is the number of compute units.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace fs {
namespace {

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

constexpr int kStreamMaxRows = 4096;   // larger batches use the LDS-ring kernels

// The streaming kernel takes a pass when its groups average at most 64 rows
// and the LDS-ring kernel's 128 x 256 tiles would not give every CU one.
inline bool use_stream(int dtype, int64_t max_rows, int G, int ffn, int d) {
  if (dtype != 1 || max_rows > kStreamMaxRows || max_rows > (int64_t)64 * G || ffn % 64 != 0 ||
      d % 64 != 0)
    return false;
  const int64_t ring_tiles =
      (int64_t)G * std::max<int64_t>(1, cdiv(max_rows, (int64_t)128 * G)) * std::max(1, ffn / 128);
  return ring_tiles < 256;
}

// Relative time of one dense group on tiles of up to h rows: rounds of tiles over
// the CUs, each costing its rows and a fixed part worth about 32.
inline int64_t r192_cost(int64_t rows, int n_tiles, int cus, int h, int unit) {
  const int64_t t = cdiv(rows, h), height = cdiv(cdiv(rows, t), unit) * unit;
  return cdiv(t * n_tiles, cus) * (height + 32);
}

// Largest tile height of a pass on the 192-row tiles.  Of one dense group,
// whose rows the host knows: the one of least cost.
// Of routed groups, whose sizes are known on the device only, 0: the kernel
// chooses (tall_tiles.hpp), in about 0.5 us; but 192 where the rows make four
// rounds of 128-row tiles and more, since the height then matters little: of 57
// such passes in bf16, 192 rows never took more than 1.012 times the ring's time.
inline int r192_height(int64_t max_rows, int G, int n_tiles, int cus, int unit = 32) {
  if (G > 1) return max_rows * n_tiles >= (int64_t)4 * 128 * cus ? 192 : 0;
  int best = 192;
  for (int h = 192 - unit; h >= 128; h -= unit)
    if (r192_cost(max_rows, n_tiles, cus, h, unit) < r192_cost(max_rows, n_tiles, cus, best, unit)) best = h;
  return best;
}

// Whether the 192-row tiles pay on one dense group.  Yes where a height above
// 128 saves rounds: 68 bf16 passes of 700 to 4096 rows took 0.61 to 0.92 of the
// ring's time.  At 128 rows both kernels run the same tiles, and the ring's
// eight waves are the better ones on few m-tiles (d 5120, F 8192, gate/up of 1000
// rows: 149 us, 155 here; 2048 rows 285 and 284) and where the last round leaves
// more than a fifth of the CUs idle (d 3072, F 1536, 4096 rows, 384 tiles: 79 +
// 47 us, 84 + 51 here).
inline bool r192_pays(int64_t rows, int n_tiles, int cus, int unit = 32) {
  const int64_t ring = cdiv(rows, 128) * n_tiles, rounds = cdiv(ring, cus);
  const int h = r192_height(rows, 1, n_tiles, cus, unit);
  if (r192_cost(rows, n_tiles, cus, h, unit) < rounds * (128 + 32)) return true;
  return rows > 1024 && ring * 5 >= rounds * cus * 4;
}

// The 192-row tiles take the passes whose groups average at least 112 rows and
// whose 128-row ring tiles would give every CU one (below that the ring splits
// K).  64 groups, d 2048, F 1408, gate/up + down: 96 rows a group 169 + 79 us
// on the ring, 168 + 81 us on these tiles; 128 rows 216 + 114 and 180 + 87;
// 384 rows 367 + 209 and 330 + 197.  32 groups of 1024 rows, d 7168, F 2048:
// 1755 + 978 and 1690 + 829 (FP8 916 + 565 and 860 + 470).  One group of 8192
// rows, gate/up of d 5120, F 8192: 1228 -> 998 us (1.38 PFLOP/s).
// rows are the likely ones (likely_rows) where the bound is loose: replicated
// tokens, 160 experts top-6, 20 of them here, d 5120, the whole layer (us, ring |
// so): 1300 tokens (a bound of 390 rows a group, 49 of them real; the ring both
// times) 458 | 458, 2000 tokens 523 | 521, 4096 tokens (154 real rows, these
// tiles) 711 | 665.  Deciding by the bound took 3 us more at 1300 tokens.
inline bool r192_ok(int64_t rows, int G, int k_blocks, int64_t ring_tiles, int cus) {
  return rows >= (int64_t)112 * G && ring_tiles >= cus && k_blocks >= 4;
}

// Kernel of one pass (gate/up: NOUT = F, K = d; down: NOUT = d, K = F).
// RING128: the ring's 128 x 128 tiles, for down passes and linears.
enum PassKind { PASS_R64, PASS_STREAM, PASS_RING, PASS_R192, PASS_SKINNY, PASS_STAGED, PASS_RING128 };

// One dense group whose 128 x 256 ring tiles leave CUs idle, K below 4096: the
// 64-row tiles while they make one round (two of 64 x 128 fit a CU), from there
// the ring, in one round and without a K split.  (us, 64-row tiles | ring | ring
// with K split and the reduction) gate/up of d 2048, F 2816 (K 2048): 333 rows
// 20 | 30 | 40, 700 rows (484 tiles) 28 | 29 | 49, 1000 rows (704) 40 | 30 | 44,
// 1400 rows 52 | 32 | 59; down of d 7168, F 2048: 333 rows 28 | 31 | 45, 700
// rows (616) 43 | 31 | 51; linear, n 5120: K 640, 640 rows (400) 10.5 | 13.2,
// 1300 rows (840) 17.5 | 15.0; K 384, 1300 rows 14.1 | 12.6.  A longer K needs
// the split: gate/up of d 7168, F 2048, 64 rows 35 | 91 | 24.  Columns that the
// 256-wide tiles do not divide have 128 x 128 ring tiles, twice as many: to one
// 64-row tile per CU (linear, n 1152, K 1024: 1700 rows, 243 tiles 12.0 | 12.7,
// 2000 rows, 288 tiles 13.7 | 12.9).
inline bool r64_one_round(int64_t rows, int n_wide, int K, int cus, bool ring256 = true) {
  return K < 4096 && cdiv(rows, 64) * n_wide <= (ring256 ? 2 : 1) * cus;
}
// The ring splits K where its tiles leave CUs idle, but not as above.
inline bool ring_may_split(int G, int K) { return G > 1 || K >= 4096; }

// One dense group of at most 64 rows.  Whole K per workgroup, no reduction:
// - down passes of very few rows: 32 output columns per workgroup, K cut over
//   its waves (the skinny kernel; K % 512 == 0).  us, skinny and 64-row tiles: d
//   7168, F 2048, 1 row 8.7 and 10.2, 20 rows 10.8 and 11.2, 33 rows 12.0 and
//   11.9; d 1024, F 512, 48 rows 5.2 and 5.7; d 5120, F 8192, 8 rows 28.1 and
//   29.2, 20 rows 33.0 and 31.2;
// - the 64-row tiles while their narrow weight tiles occupy enough CUs for the
//   length of K.  us, 64-row tiles and streaming: gate/up of d 2048, F 2816, 1
//   row 10.2 and 12.8; d 5120, F 8192, 64 rows 34 and 53 (256 tiles); but d
//   3072, F 1536, 1 row 12.8 and 12.1, 20 rows 15.7 and 14.2, 33 rows 15.7 and
//   16.3 (48 tiles), and d 7168, F 2048, 1 row 24.8 and 18.0, 64 rows 35 and 25;
// else weight streaming.
inline PassKind few_rows_kind(bool gateup, int64_t rows, int NOUT, int K) {
  const int64_t narrow = NOUT / (gateup ? 32 : 64);
  if (!gateup && K % 512 == 0 && (rows <= 8 || rows * K <= 40960)) return PASS_SKINNY;
  return K < 2560 || narrow * 50 >= K || (rows > 32 && K < 4096) ? PASS_R64 : PASS_STREAM;
}

// A pass whose columns the ring's 256-wide tiles do not divide (gate/up F % 128 =
// 64, down d % 256 = 128).  All of them can run on 64-row tiles; long passes are
// faster on 128-row ones: gate/up on the register-staged 128 x 128 tiles, whose
// rounds (two workgroups per CU, as of the 64-row tiles) take about 1.35 times
// as long, down on the ring's 128 x 128 tiles (one per CU).
// us, 64-row | staged | ring 128 x 128 tiles: gate/up of 64 groups of 110 rows, d
// 1664, F 2496: 294 | 252 | 268; of 16 groups of 180 rows, d 640, F 1472: 28 | 32 |
// 32; down of the first 166 | 133 | 131, of the second 18 | 32 | 22; down of 3000
// rows in one group, d 4480, F 1536: 65 | 66 | 62, 1500 rows 38 | 33 | 37 (420 ring
// tiles: two rounds on the ring, one staged), 700 rows 23 | 28 | 18.
// Group sizes are known on the device only: a group of r rows is taken to make
// r / 128 + 0.4 tiles, at least one.
inline PassKind odd_kind(bool gateup, int64_t rows, int G, int NOUT, int cus) {
  const int64_t n = NOUT / (gateup ? 64 : 128), slots = 2 * cus;
  if (gateup) {
    auto rounds = [&](int64_t bm) {
      const int64_t tiles = G == 1 ? cdiv(rows, bm) * n
                                   : std::max<int64_t>(G, (rows * 10 + 4 * G * bm) / (10 * bm)) * n;
      return cdiv(tiles, slots);
    };
    return rounds(64) * 100 > rounds(128) * 135 ? PASS_STAGED : PASS_R64;
  }
  if (G == 1) {
    const int64_t t = cdiv(rows, 128) * n;
    if (cdiv(rows, 64) * n <= cus) return PASS_R64;
    return t > cus && t <= slots ? PASS_STAGED : PASS_RING128;
  }
  const int64_t t64 = G * cdiv(rows, (int64_t)64 * G) * n;
  return rows <= (int64_t)16 * G || t64 * 4 < (int64_t)11 * cus ? PASS_R64 : PASS_RING128;
}

// Grouped passes of short groups (hidden size below 4096) on the 64-row tiles, since
// a 128-row tile is mostly padding: gate/up up to 40 rows a group and K of 2048,
// down up to 32 rows and K of 1024, or where the ring would split a K below 4096.  us,
// weights from HBM, ring and 64-row tiles: gate/up of 64 groups, d 2048, F 1408: 12
// rows a group 142 and 136, 44 rows 150 and 144, but of 24, d 1280, F 2560, 44 rows 65
// and 71; of 60, d 2560, F 1408: 163 and 166, 171 and 175; of 128, d 512, F 384: 28 and
// 21, 28 and 25; down of the first 68 and 71, 71 and 80, of the last 15.2 and 13.5, 16.8
// and 18.4; of 24, d 1280, F 2560 (120 ring tiles): 4 rows 42 and 44, 24 rows 50 and 44,
// 44 rows 59 and 49; 32 groups of 12 rows, d 1024, F 4096 (128 ring tiles), both passes
// 159 with the ring's down, 167 with 64-row tiles.
inline bool short_groups(bool gateup, int64_t max_rows, int G, int K, int d, int64_t ring_tiles, int cus) {
  if (max_rows > (int64_t)48 * G || d >= 4096) return false;
  if (gateup) return max_rows <= (int64_t)40 * G && K <= 2048;
  return (max_rows <= (int64_t)32 * G && K <= 1024) ||
         (ring_tiles < cus && max_rows >= (int64_t)12 * G && K < 4096);
}

inline PassKind pass_kind(int dtype, bool gateup, int64_t max_rows, int64_t likely_rows, int G,
                          int ffn, int d, int cus) {
  if (dtype != 1) return PASS_R64;   // every fp32 pass
  const int NOUT = gateup ? ffn : d, K = gateup ? d : ffn, n_tiles = NOUT / (gateup ? 128 : 256);
  const bool stream = use_stream(dtype, max_rows, G, ffn, d);
  if (stream) return G == 1 ? few_rows_kind(gateup, max_rows, NOUT, K) : PASS_STREAM;
  const bool own = NOUT % (gateup ? 128 : 256) == 0, both = ffn % 128 == 0 && d % 256 == 0;
  const int64_t ring_tiles = G * cdiv(max_rows, (int64_t)128 * G) * n_tiles;
  // (where only the other pass's columns do not divide, short groups and passes
  // that would split K do as if both did not)
  if (!own || (!both && G > 1 && (ring_tiles < cus || max_rows <= (int64_t)48 * G)))
    return odd_kind(gateup, likely_rows, G, NOUT, cus);
  if (G == 1) {
    // (K limits it only where both widths divide, and the split ring is the choice)
    if (r64_one_round(max_rows, NOUT / (gateup ? 64 : 128), both ? K : 64, cus)) return PASS_R64;
  } else if (both && short_groups(gateup, max_rows, G, K, d, ring_tiles, cus)) {
    return PASS_R64;
  }
  if (!r192_ok(likely_rows, G, K / 64, ring_tiles, cus)) return PASS_RING;
  return G > 1 || r192_pays(max_rows, n_tiles, cus) ? PASS_R192 : PASS_RING;
}

// An FP8 pass: the ring or the 192-row tiles, whose line in bf16 holds in FP8 too.
// The FFN of groups of 112, 128, 160 and 390 rows (us, ring | 192-row tiles): 64
// groups, d 2048, F 1408: 169 | 155, 170 | 165, 196 | 192, 337 | 317; 32 groups,
// d 7168, F 2048: 350 | 317, 349 | 343, 413 | 393, 716 | 627; 16 groups, d 5120, F
// 8192: 485 | 464, 580 | 480, 580 | 534, 986 | 893.  Shorter ones were not tried.
inline PassKind pass_kind_fp8(bool gateup, int64_t max_rows, int G, int ffn, int d, int cus) {
  const int NOUT = gateup ? ffn : d, K = gateup ? d : ffn, n_tiles = NOUT / (gateup ? 128 : 256);
  const int64_t ring_tiles = G * cdiv(max_rows, (int64_t)128 * G) * n_tiles;
  if (!r192_ok(max_rows, G, K / 128, ring_tiles, cus)) return PASS_RING;
  return G > 1 || r192_pays(max_rows, n_tiles, cus, 64) ? PASS_R192 : PASS_RING;
}

// A dense linear, one group of m rows: 64-row tiles where the ring's would
// leave CUs idle (as above), else the 192-row tiles, else the ring (128 x 128
// tiles when n is not a multiple of 256; never split).
inline PassKind dense_kind(int dtype, int m, int n, int kdim, int cus) {
  if (dtype != 1 || r64_one_round(m, n / 128, kdim, cus, n % 256 == 0)) return PASS_R64;
  const int64_t ring_tiles = cdiv(m, 128) * (n / 256);
  if (n % 256 != 0) return PASS_RING128;
  return r192_ok(m, 1, kdim / 64, ring_tiles, cus) && r192_pays(m, n / 256, cus) ? PASS_R192 : PASS_RING;
}

}  // namespace
}  // namespace fs
