// fp32 passes of the grouped SwiGLU expert FFN (Section 2.1) and the fp32
// dense linear, on the fp32 matrix cores.
//
// v_mfma_f32_16x16x4_f32 multiplies and accumulates in fp32 (no reduced
// format), at twice the rate of unpacked vector FMAs.  A workgroup of four
// waves owns 64 rows x BN weight rows (128, or 64 where 128 would give too
// few tiles) and walks K in blocks of 32 floats through a three-slot LDS
// ring filled by direct global->LDS copies two blocks ahead; two workgroups
// fit a CU, so one computes while the other waits for its tile's first
// blocks.  A staged row is 128 bytes; 16-byte chunk c of row r sits at
// position c ^ ((r / 2) % 8), so a 16-byte LDS read by sixteen consecutive
// rows covers every bank once.  Lane l reads row l % 16, floats 4 (l / 16)
// .. + 3 of a 16-wide K step and feeds them to four MFMAs (A and B use the
// same K order); accumulator element v of lane l is row 4 (l / 16) + v,
// column l % 16.
//
// Routed groups are short (tens of rows), so padded rows would be most of
// the MFMA work: a tile's waves run only the 16-row fragments that hold
// rows (one K loop per count, so the loop itself has no branch).
//
// Measured against 64 x 64 tiles on the vector ALUs (4 x 4 outputs per
// thread): 64 groups of about 48 rows, d 2048, F 1408: gate/up 734 -> 415
// us, down 322 -> 216 us (MFMA busy 80% of the cycles a CU has work; 8% of
// the rest is the last round of tiles); 512 dense rows, F 2816: gate/up 226
// -> 124 us, down 152 -> 65 us.  The block of those shapes 1491 -> 840 us.
#include <algorithm>

#include "gemm_common.hpp"
#include "internal.hpp"

namespace fs {
namespace {

template <int MODE, int WM>
__global__ __launch_bounds__(256, 2) void gemm_f32_kernel(
    const float* __restrict__ A, const int32_t* __restrict__ rows,
    const int32_t* __restrict__ goff, int G, int64_t m_total, const float* __restrict__ B, int K,
    int NOUT, float* __restrict__ C, int ldc) {
  constexpr int NT = 256, WN = 4 / WM;             // waves: WM row blocks x WN column blocks
  constexpr int BM = 64, BN = 32 * WN, BK = 32, NST = 3;
  constexpr int TMX = BM / WM / 16;                // 16-row fragments per wave
  constexpr int STAGE = (BM + BN) * 128;
  constexpr int A_LD = BM / 8 / 4, B_LD = BN / 8 / 4, NLD = A_LD + B_LD;   // DMAs per wave
  constexpr int NCOL = MODE == MODE_GATEUP ? BN / 2 : BN;
  __shared__ int s_goff[kMaxGroups + 1];
  __shared__ int s_tpre[kMaxGroups + 1];
  __shared__ int s_wtot[NT / 64];
  __shared__ __align__(1024) unsigned char ring[NST * STAGE];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int l16 = lane & 15, quad = lane >> 4;
  sched_setup<NT, BM>(goff, G, m_total, s_goff, s_tpre, s_wtot);
  const int nn = NOUT / NCOL;
  const int64_t total = (int64_t)nn * s_tpre[G];
  const int64_t per_xcd = (total + kXcd - 1) / kXcd;
  const int64_t xcd_base = (int64_t)(blockIdx.x % kXcd) * per_xcd;
  const int64_t stride = gridDim.x / kXcd;
  const size_t bstride = (size_t)(MODE == MODE_GATEUP ? 2 * NOUT : NOUT) * K;
  const int KT = K / BK;
  const int drow = lane / 8, dpos = lane % 8;
  const unsigned ring_lds = lds_addr(ring);
  const unsigned wave_u = __builtin_amdgcn_readfirstlane(wave);

  // fragment rows of this wave inside a slot
  int arow[TMX], brow[2];
#pragma unroll
  for (int i = 0; i < TMX; ++i) arow[i] = wm * (BM / WM) + i * 16 + l16;
#pragma unroll
  for (int t = 0; t < 2; ++t) brow[t] = wn * 32 + t * 16 + l16;
  int ghint = 0;

  for (int64_t j = blockIdx.x / kXcd; j < per_xcd; j += stride) {
    const int64_t L = xcd_base + j;
    if (L >= total) break;
    const int g = find_group_from(s_tpre, G, nn, L, ghint);
    ghint = g;
    const int Tg = s_tpre[g + 1] - s_tpre[g];
    const int local = (int)(L - (int64_t)nn * s_tpre[g]);
    const int nt = local / Tg;
    const int m0 = (local - nt * Tg) * BM, n0 = nt * NCOL;
    const int row_base = s_goff[g], rows_g = s_goff[g + 1] - row_base;
    const float* Bg = B + (size_t)g * bstride;

    // sources of this wave's DMAs (8 rows of 128 bytes each); rows past the
    // group's end load its last row and are never stored
    const float *pa[A_LD], *pb[B_LD];
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
      const int r = (wave * A_LD + i) * 8 + drow;
      const int grow = row_base + min(m0 + r, rows_g - 1);
      const int64_t sr = (MODE == MODE_GATEUP && rows) ? (int64_t)rows[grow] : (int64_t)grow;
      pa[i] = A + sr * K + (dpos ^ ((r >> 1) & 7)) * 4;
    }
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
      // a wave's 32 weight rows: 16 gate rows and the matching 16 up rows,
      // or 32 output columns
      const int r = (wave * B_LD + i) * 8 + drow;
      const int wrow = MODE == MODE_GATEUP ? ((r >> 4) & 1) * NOUT + n0 + (r >> 5) * 16 + (r & 15)
                                           : n0 + r;
      pb[i] = Bg + (size_t)wrow * K + (dpos ^ ((r >> 1) & 7)) * 4;
    }
    auto issue = [&](int kt) {
      const unsigned slot = ring_lds + (unsigned)(kt % NST) * STAGE;
#pragma unroll
      for (int i = 0; i < A_LD; ++i) dma16_at(pa[i] + kt * BK, slot + (wave_u * A_LD + i) * 1024u);
#pragma unroll
      for (int i = 0; i < B_LD; ++i)
        dma16_at(pb[i] + kt * BK, slot + BM * 128u + (wave_u * B_LD + i) * 1024u);
    };
    // fragments of this wave that hold rows
    const int live = min(max(rows_g - m0 - wm * (BM / WM), 0), BM / WM);
    const int tma = __builtin_amdgcn_readfirstlane((live + 15) / 16);

    auto tile = [&](auto TMA) {
      constexpr int TM = decltype(TMA)::value;
      constexpr int TMA1 = TM > 0 ? TM : 1;
      floatx4 acc[TMA1][2];
#pragma unroll
      for (int i = 0; i < TMA1; ++i)
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[i][t] = floatx4{0.f, 0.f, 0.f, 0.f};
      issue(0);
      if (KT > 1) issue(1);
      for (int kt = 0; kt < KT; ++kt) {
        // block kt has landed once only block kt + 1's DMAs remain; slot
        // (kt + 2) % 3 was read in the iteration before this barrier
        if (kt + 1 < KT)
          wait_vmcnt<NLD>();
        else
          wait_vmcnt<0>();
        wait_lgkm0();
        barrier_nofence();
        if (kt + 2 < KT) issue(kt + 2);
        if constexpr (TM > 0) {
          const unsigned char* sa = ring + (kt % NST) * STAGE;
          const unsigned char* sb = sa + BM * 128;
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            floatx4 fa[TM], fb[2];
#pragma unroll
            for (int t = 0; t < 2; ++t)
              fb[t] = *reinterpret_cast<const floatx4*>(
                  sb + brow[t] * 128 + (((h * 4 + quad) ^ ((brow[t] >> 1) & 7)) << 4));
#pragma unroll
            for (int i = 0; i < TM; ++i)
              fa[i] = *reinterpret_cast<const floatx4*>(
                  sa + arow[i] * 128 + (((h * 4 + quad) ^ ((arow[i] >> 1) & 7)) << 4));
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
              for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                  acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[i][s], fb[t][s], acc[i][t],
                                                                   0, 0, 0);
          }
        }
      }
      if constexpr (TM > 0) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int m = m0 + wm * (BM / WM) + i * 16 + 4 * quad + v;
            if (m >= rows_g) continue;
            const int grow = row_base + m;
            if (MODE == MODE_GATEUP) {
              const float gt = acc[i][0][v], up = acc[i][1][v];
              C[(size_t)grow * ldc + n0 + wn * 16 + l16] = gt / (1.0f + expf(-gt)) * up;
            } else {
              const int64_t orow = rows ? (int64_t)rows[grow] : (int64_t)grow;
#pragma unroll
              for (int t = 0; t < 2; ++t)
                C[orow * ldc + n0 + wn * 32 + t * 16 + l16] = acc[i][t][v];
            }
          }
      }
    };
    switch (tma) {
      case 0: tile(std::integral_constant<int, 0>{}); break;
      case 1: tile(std::integral_constant<int, 1>{}); break;
      case 2: tile(std::integral_constant<int, 2>{}); break;
      case 3: tile(std::integral_constant<int, TMX < 3 ? TMX : 3>{}); break;
      default: tile(std::integral_constant<int, TMX>{}); break;
    }
    __syncthreads();   // the next tile refills slots that slower waves may still read
  }
}

template <int MODE, int WM>
void run(const float* A, const int32_t* rows, const int32_t* goff, int G, int64_t m_total,
         const float* B, int K, int NOUT, float* C, int ldc, int cus, hipStream_t s) {
  constexpr int NCOL = (MODE == MODE_GATEUP ? 16 : 32) * (4 / WM);
  const int64_t tiles = (cdiv64(m_total, 64) + G) * (NOUT / NCOL);
  // two (128 weight rows) or three (64) workgroups fit a CU's LDS
  const int64_t slots = (int64_t)(WM == 1 ? 2 : 3) * cus;
  const int64_t grid = std::min<int64_t>(cdiv64(tiles, kXcd), cdiv64(slots, kXcd)) * kXcd;
  launch_k(gemm_f32_kernel<MODE, WM>, (unsigned)grid, 256, 0, s, A, rows, goff, G, m_total, B, K,
           NOUT, C, ldc);
}

}  // namespace

void launch_gemm_f32(bool gateup, const float* A, const int32_t* rows, const int32_t* goff, int G,
                     int64_t m_total, const float* B, int K, int NOUT, float* C, int ldc, int cus,
                     hipStream_t s) {
  // 128 weight rows per tile; 64 where the output width does not allow 128
  // or 128 would give fewer than the two tiles per CU that run together
  // (tiles counted from the row bound, one partial tile per group).  512 rows
  // x 2816 x 2048 (352 wide tiles on 256 CUs): 148 us wide, 124 us narrow;
  // 64 groups of about 48 rows, 1408 wide tiles: 415 us wide, 436 us narrow.
  const int wide = gateup ? 64 : 128;
  const bool narrow = NOUT % wide != 0 || (cdiv64(m_total, 64) + G - 1) * (NOUT / wide) < 2 * cus;
  if (gateup && narrow)
    run<MODE_GATEUP, 2>(A, rows, goff, G, m_total, B, K, NOUT, C, ldc, cus, s);
  else if (gateup)
    run<MODE_GATEUP, 1>(A, rows, goff, G, m_total, B, K, NOUT, C, ldc, cus, s);
  else if (narrow)
    run<MODE_DOWN, 2>(A, rows, goff, G, m_total, B, K, NOUT, C, ldc, cus, s);
  else
    run<MODE_DOWN, 1>(A, rows, goff, G, m_total, B, K, NOUT, C, ldc, cus, s);
}

}  // namespace fs
