// How the 192-row kernel (gemm_r192.hpp) cuts a pass into tiles.  Plain C++ for
// the kernel, the host's rules and host tests.
#pragma once

#include <math.h>
#include <stdint.h>

#ifdef __HIPCC__
#define FS_HD __host__ __device__ __forceinline__
#else
#define FS_HD inline
#endif
// a value that is the same in every lane, held in a scalar register
#ifdef __HIP_DEVICE_COMPILE__
#define FS_UNI(x) __builtin_amdgcn_readfirstlane(x)
#else
#define FS_UNI(x) (x)
#endif

namespace fs {
namespace {

// Relative time of a pass whose groups hold `rows` rows in `m_tiles` m-tiles,
// times nn n-tiles, on wgs workgroups (a multiple of 8, one per CU): each runs
// its share of its XCD's range tile by tile, and a tile costs its rows and a
// fixed part worth about 96 of them.
FS_HD float tall_cost(int rows, int m_tiles, int nn, int wgs) {
  // (the quotient of whole numbers below 2^24 rounds to a whole one only where
  // it is one)
  const float rounds = ceilf((float)((m_tiles * nn + 7) / 8) / (float)(wgs / 8));
  return rounds * ((float)rows / (float)m_tiles + 96.0f);
}

// Largest tile height of a pass, from the number of m-tiles that its groups
// make at 192, 160 (0: not a choice) and 128 rows.  The tallest tiles make the
// fewest L2 requests, but where a few tiles more than the CUs make a whole
// further round, lower ones that need the same number of rounds or one more
// take less time; a gain below 2% is within the estimate's error.  Routed
// passes of 13 shapes at 80 to 600 rows a group (230 passes in bf16, 250 in
// FP8), time of the 128-row ring over this kernel's: always 192 rows 1.087 and
// 1.077 (lowest 0.85 and 0.84; 44 and 35 passes below 0.97), by this rule 1.128
// and 1.096 (0.95 and 0.95; 1 and 3 below 0.97).
FS_HD int tall_height(int rows, int t192, int t160, int t128, int nn, int wgs) {
  if (t192 <= 0) return 192;
  int h = 192;
  float best = 0.98f * tall_cost(rows, t192, nn, wgs);
  if (t160 > 0) {
    const float c = tall_cost(rows, t160, nn, wgs);
    if (c < best) best = 0.98f * c, h = 160;
  }
  if (tall_cost(rows, t128, nn, wgs) < best) h = 128;
  return h;
}

// Height of a group's tiles: `tiles` of them cover its rows, all of this height
// (a multiple of unit) but the last.
FS_HD int tall_rows(int rows, int tiles, int unit) {
  return FS_UNI((rows + tiles - 1) / tiles + unit - 1) & ~(unit - 1);
}

// Tile `local` (the same in every lane) of a group of `tiles` m-tiles and nn n-tiles: m-tiles in bands of
// at most 8, a band's m-tiles fastest, then the n-tiles, so that the tiles an
// XCD runs together share both operands.
FS_HD void tall_order(int local, int tiles, int nn, int& mt, int& nt) {
  const int bands = FS_UNI((tiles + 7) / 8), bh = FS_UNI((tiles + bands - 1) / bands);
  const int band = FS_UNI(local / (nn * bh));
  local -= band * nn * bh;
  const int left = tiles - band * bh, bw = bh < left ? bh : left;
  nt = FS_UNI(local / bw);
  mt = band * bh + local - nt * bw;
}

}  // namespace
}  // namespace fs
