// Grouped SwiGLU FFN passes and dense linears on 64-row tiles: every fp32
// pass, and the bf16 passes whose groups are short, whose one dense group makes
// few tiles, or whose columns the ring's tiles do not divide (Section 2.1;
// pass_rules.hpp says which).
//
// A workgroup of four waves owns 64 rows x BN weight rows (128, or 64 where
// 128 would give too few tiles) and walks K in blocks of ROWB bytes a row
// through a ring of NST LDS slots filled by direct global->LDS copies NST - 1
// blocks ahead: 128 bytes (32 floats, 64 bf16) in three slots, where two (BN
// 128) or three workgroups fit a CU and one computes while another waits; 256
// bytes in four slots, or 128 in eight, where there is at most one workgroup
// per CU.  16-byte chunk c of staged row r sits at position c ^ ((r / 2) % 8)
// (256-byte rows: c ^ (r % 16)), so a 16-byte LDS read by sixteen consecutive
// rows covers every bank once.  Lane l reads row l % 16, chunk l / 16 of a 64-byte half
// block: one v_mfma_f32_16x16x32_bf16 operand, or the operands of four
// v_mfma_f32_16x16x4_f32 (both operands use the same K order).  fp32
// multiplies and accumulates in fp32, at twice the rate of unpacked vector
// FMAs.
//
// The weights are the MFMA's row operand, so accumulator element v of lane l
// is weight row 4 (l / 16) + v of its fragment and activation row l % 16: a
// lane holds consecutive output columns of one row.  In down passes the two
// fragments of a wave's 32 columns interleave in fours (their weight rows are
// permuted on the way into LDS), so a lane stores eight consecutive columns.
//
// Routed groups are short (tens of rows), so padded rows would be most of
// the MFMA work: a tile's waves run only the 16-row fragments that hold
// rows (one K loop per count, so the loop itself has no branch).
//
// Measured, fp32, against 64 x 64 tiles on the vector ALUs (4 x 4 outputs
// per thread): 64 groups of about 48 rows, d 2048, F 1408: gate/up 734 -> 415
// us, down 322 -> 216 us (MFMA busy 66% and 56% of all cycles, by its counters);
// 512 dense rows, F 2816: gate/up 226 -> 124 us, down 152 -> 65 us.  The block of
// those shapes 1496 -> 847 us.
#include <algorithm>
#include <type_traits>

#include "gemm_common.hpp"
#include "internal.hpp"

namespace fs {
namespace {

__device__ __forceinline__ void store4(float* p, const float (&v)[4]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void store4(bf16_t* p, const float (&v)[4]) {
  *reinterpret_cast<uint2*>(p) = make_uint2(f2bf(v[0]) | ((uint32_t)f2bf(v[1]) << 16),
                                            f2bf(v[2]) | ((uint32_t)f2bf(v[3]) << 16));
}

template <typename T, int MODE, int WM, int ROWB, int NST, int OCC>
__global__ __launch_bounds__(256, OCC) void gemm_r64_kernel(
    const T* __restrict__ A, const int32_t* __restrict__ rows, const int32_t* __restrict__ goff,
    int G, int64_t m_total, const T* __restrict__ B, int K, int NOUT, T* __restrict__ C, int ldc) {
  constexpr bool F32 = sizeof(T) == 4;
  constexpr int CE = 16 / sizeof(T);               // elements per 16-byte chunk
  constexpr int NT = 256, WN = 4 / WM;             // waves: WM row blocks x WN column blocks
  constexpr int BM = 64, BN = 32 * WN, CPR = ROWB / 16, BK = CPR * CE;
  constexpr int RPD = 1024 / ROWB;                 // rows per DMA
  using FragT = typename std::conditional<F32, floatx4, bf16x8>::type;
  constexpr int TMX = BM / WM / 16;                // 16-row fragments per wave
  constexpr int STAGE = (BM + BN) * ROWB;
  constexpr int A_LD = BM / RPD / 4, B_LD = BN / RPD / 4, NLD = A_LD + B_LD;   // DMAs per wave
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
  const int drow = lane / CPR, dpos = lane % CPR;
  auto swz = [](int r) { return ROWB == 128 ? (r >> 1) & 7 : r & 15; };
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
    const T* Bg = B + (size_t)g * bstride;

    // sources of this wave's DMAs (RPD rows of ROWB bytes each); rows past the
    // group's end load its last row and are never stored
    const T *pa[A_LD], *pb[B_LD];
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
      const int r = (wave * A_LD + i) * RPD + drow;
      const int grow = row_base + min(m0 + r, rows_g - 1);
      const int64_t sr = (MODE == MODE_GATEUP && rows) ? (int64_t)rows[grow] : (int64_t)grow;
      pa[i] = A + sr * K + (dpos ^ swz(r)) * CE;
    }
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
      // a wave's 32 weight rows: 16 gate rows and the matching 16 up rows,
      // or 32 output columns, fragment t's row q holding column
      // 8 (q / 4) + 4 t + q % 4
      const int r = (wave * B_LD + i) * RPD + drow;
      const int q = r & 15, t = (r >> 4) & 1;
      const int wrow = MODE == MODE_GATEUP ? t * NOUT + n0 + (r >> 5) * 16 + q
                                           : n0 + (r & ~31) + 8 * (q >> 2) + 4 * t + (q & 3);
      pb[i] = Bg + (size_t)wrow * K + (dpos ^ swz(r)) * CE;
    }
    auto issue = [&](int kt) {
      const unsigned slot = ring_lds + (unsigned)(kt % NST) * STAGE;
#pragma unroll
      for (int i = 0; i < A_LD; ++i) dma16_at(pa[i] + kt * BK, slot + (wave_u * A_LD + i) * 1024u);
#pragma unroll
      for (int i = 0; i < B_LD; ++i)
        dma16_at(pb[i] + kt * BK, slot + BM * (unsigned)ROWB + (wave_u * B_LD + i) * 1024u);
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
#pragma unroll
      for (int b = 0; b < NST - 1; ++b)
        if (b < KT) issue(b);
      for (int kt = 0; kt < KT; ++kt) {
        // block kt has landed once only the DMAs of the NST - 2 blocks after
        // it remain; the slot of block kt + NST - 1 was read in the iteration
        // before this barrier
        if (kt + NST - 2 < KT)
          wait_vmcnt<(NST - 2) * NLD>();
        else
          wait_vmcnt<0>();
        wait_lgkm0();
        barrier_nofence();
        if (kt + NST - 1 < KT) issue(kt + NST - 1);
        if constexpr (TM > 0) {
          const unsigned char* sa = ring + (kt % NST) * STAGE;
          const unsigned char* sb = sa + BM * ROWB;
#pragma unroll
          for (int h = 0; h < CPR / 4; ++h) {
            FragT fa[TM], fb[2];
#pragma unroll
            for (int t = 0; t < 2; ++t)
              fb[t] = *reinterpret_cast<const FragT*>(
                  sb + brow[t] * ROWB + (((h * 4 + quad) ^ swz(brow[t])) << 4));
#pragma unroll
            for (int i = 0; i < TM; ++i)
              fa[i] = *reinterpret_cast<const FragT*>(
                  sa + arow[i] * ROWB + (((h * 4 + quad) ^ swz(arow[i])) << 4));
            if constexpr (F32) {
#pragma unroll
              for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                  for (int t = 0; t < 2; ++t)
                    acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[t][s], fa[i][s], acc[i][t],
                                                                     0, 0, 0);
            } else {
#pragma unroll
              for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                  acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[t], fa[i], acc[i][t], 0, 0,
                                                                      0);
            }
          }
        }
      }
      if constexpr (TM > 0) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const int m = m0 + wm * (BM / WM) + i * 16 + l16;
          if (m >= rows_g) continue;
          const int grow = row_base + m;
          if constexpr (MODE == MODE_GATEUP) {
            float h[4];
#pragma unroll
            for (int v = 0; v < 4; ++v)
              h[v] = F32 ? acc[i][0][v] / (1.0f + expf(-acc[i][0][v])) * acc[i][1][v]
                         : swiglu_bf16_epi(acc[i][0][v], acc[i][1][v]);
            store4(C + (size_t)grow * ldc + n0 + wn * 16 + 4 * quad, h);
          } else {
            const int64_t orow = rows ? (int64_t)rows[grow] : (int64_t)grow;
            T* p = C + orow * ldc + n0 + wn * 32 + 8 * quad;
            if constexpr (F32) {
              float y[4];
#pragma unroll
              for (int t = 0; t < 2; ++t) {
#pragma unroll
                for (int v = 0; v < 4; ++v) y[v] = acc[i][t][v];
                store4(p + 4 * t, y);
              }
            } else {
              Vec16<bf16_t> o;
#pragma unroll
              for (int v = 0; v < 8; ++v) o.set(v, acc[i][v >> 2][v & 3]);
              st16(p, o.raw);
            }
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

template <typename T, int MODE, int WM, int ROWB, int NST, int OCC>
void run(const T* A, const int32_t* rows, const int32_t* goff, int G, int64_t m_total, const T* B,
         int K, int NOUT, T* C, int ldc, int cus, hipStream_t s) {
  constexpr int NCOL = (MODE == MODE_GATEUP ? 16 : 32) * (4 / WM);
  const int64_t tiles = (cdiv64(m_total, 64) + G) * (NOUT / NCOL);
  const int64_t grid = std::min<int64_t>(cdiv64(tiles, kXcd), cdiv64((int64_t)OCC * cus, kXcd)) * kXcd;
  launch_k(gemm_r64_kernel<T, MODE, WM, ROWB, NST, OCC>, (unsigned)grid, 256, 0, s, A, rows, goff, G,
           m_total, B, K, NOUT, C, ldc);
}

template <typename T>
void pass(bool gateup, const T* A, const int32_t* rows, const int32_t* goff, int G,
          int64_t m_total, const T* B, int K, int NOUT, T* C, int ldc, int cus, hipStream_t s) {
  // Tiles counted from the row bound, one partial tile per group.
  const int64_t m_tiles = cdiv64(m_total, 64) + G - 1;
  const int wide = gateup ? 64 : 128;
  const bool only_narrow = NOUT % wide != 0;
#define FS_PASS(WM, ROWB, NST, OCC)                                                            \
  do {                                                                                         \
    if (gateup)                                                                                \
      run<T, MODE_GATEUP, WM, ROWB, NST, OCC>(A, rows, goff, G, m_total, B, K, NOUT, C, ldc,   \
                                              cus, s);                                         \
    else                                                                                       \
      run<T, MODE_DOWN, WM, ROWB, NST, OCC>(A, rows, goff, G, m_total, B, K, NOUT, C, ldc,     \
                                            cus, s);                                           \
  } while (0)
  // At most one narrow tile per CU: one workgroup with a deep ring hides
  // its own load latency (bf16, 333 rows x 2048 x 2816, 192 tiles: three 16
  // KB slots 29 us, eight 18 us, four of 256-byte rows 15.7 us).
  if (m_tiles * (NOUT / (wide / 2)) <= cus) {
    if (K % (256 / (int)sizeof(T)) == 0)
      FS_PASS(2, 256, 4, 1);
    else
      FS_PASS(2, 128, 8, 1);
    return;
  }
  // 128 weight rows per tile, two workgroups per CU; 64 and three where the
  // width does not allow 128 and, in fp32, whose tiles take the matrix cores
  // long enough for the balance to count, where 128 gives fewer than two
  // tiles per CU.  fp32, 512 rows x 2816 x 2048 (352 wide tiles on 256 CUs):
  // 148 us wide, 124 us narrow; 64 groups of about 48 rows (1408 tiles): 415
  // and 436 us.  bf16, 700 rows of the same (484 tiles): 30 and 36 us.
  if (only_narrow || (sizeof(T) == 4 && m_tiles * (NOUT / wide) < 2 * cus))
    FS_PASS(2, 128, 3, 3);
  else
    FS_PASS(1, 128, 3, 2);
#undef FS_PASS
}

}  // namespace

void launch_gemm_r64(int dtype, bool gateup, const void* A, const int32_t* rows,
                     const int32_t* goff, int G, int64_t m_total, const void* B, int K, int NOUT,
                     void* C, int ldc, int cus, hipStream_t s) {
  if (dtype == 0)
    pass(gateup, (const float*)A, rows, goff, G, m_total, (const float*)B, K, NOUT, (float*)C, ldc,
         cus, s);
  else
    pass(gateup, (const bf16_t*)A, rows, goff, G, m_total, (const bf16_t*)B, K, NOUT, (bf16_t*)C,
         ldc, cus, s);
}

}  // namespace fs
