// Grouped SwiGLU FFN passes on tiles of up to 192 rows x 256 weight rows, for
// groups of a hundred rows and more (Section 2.1, prefill).
//
// What bounds the 128 x 256 ring (gemm.hip) is not the matrix cores but the
// stream of L2 requests that fills its LDS: 48 KB per 64-wide K block of a tile
// (one L2 request per 128-byte row), its copies alone taking as long as the
// pass; in a timing variant the same loop without copies ran 1.8 times faster.
// (This kernel's counters: 81 G requests/s and the matrix cores 53% busy on 16
// groups of about 512 rows, d 5120, F 8192, gate/up; 96 G/s and 71% on 8192 dense
// rows.)  (A first version of this kernel with 64-byte
// rows, 256 x 256 x 32 tiles, made as many requests for half the bytes and
// was no faster than the ring.)  So the tile is taller, and the wave tile
// larger: four waves (2 x 2), one per SIMD, each up to 96 x 128 through
// v_mfma_f32_16x16x32_bf16, 192 accumulators; an LDS fragment read feeds six
// or eight MFMAs.
//
//   Heights  The pass's largest height is 192, 160 or 128 rows: of one dense
//            group the host chooses it, of routed groups, whose sizes the host
//            does not know, every workgroup (tall_height; about 0.5 us).  A
//            group's tiles have equal heights, a multiple of 32 up to that, so
//            the last tile is not a stub; the tile's code is one loop per
//            height (no branch inside).  A wave's 16-row fragments alternate
//            between the two wave rows.  (224 and 256 rows make the compiler
//            move accumulators in and out of the AGPRs inside the loop: 32
//            groups of 1024 rows, gate/up 1670 us at 192, 1796 at 224.)
//   Ring     A has two 64-wide LDS slots, B three: activations mostly hit in
//            L2, weights come from HBM and need the longer lead (two slots
//            each: the 16-expert gate/up 1572 us, with three for B 1307 us).
//            Copies and waits run on from tile to tile.
//   Order    m-tiles in bands of at most eight, then the n-tiles, so the tiles
//            an XCD runs together share both operands.
//   Output   Weights are the MFMA's row operand, weight rows are permuted on
//            the way into LDS: a lane holds eight consecutive output columns
//            and stores them as they are, without staging.
//
//   FP8      E4M3 codes on v_mfma_scale_f32_32x32x64_f8f6f4 (unit scales): the
//            same bytes per block, 32-row fragments, heights in steps of 64;
//            the epilogue applies the row and column scales, which copies
//            into LDS bring at the tile's start.
//
// Measured (us, ring -> this): 8192 rows, d 5120, F 8192, dense gate/up 1228
// -> 998 (1.38 PFLOP/s; on another box 1014, the vendor library's dense kernel
// 921), down 590 -> 546; 16 groups of about 512 rows of the same: 1410 -> 1290 and 706
// -> 641; 32 groups of 1024 rows, d 7168, F 2048: 1755 -> 1690 and 978 ->
// 829, FP8 916 -> 860 and 565 -> 470; 64 groups of 384 rows, d 2048, F 1408:
// 347 -> 298 and 199 -> 176.
#pragma once

#include <algorithm>
#include <type_traits>
#include <utility>

#include "gemm_common.hpp"
#include "internal.hpp"
#include "tall_tiles.hpp"

namespace fs {
namespace {

// f(0), f(1), .. f(N - 1) with compile-time indices (the loops below are too
// long for the unroller).
template <typename F, int... I>
__device__ __forceinline__ void static_for_(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_(f, std::make_integer_sequence<int, N>{});
}

// global->LDS copies whose LDS address is a wave-uniform base plus a
// constant: M0 is formed by one scalar add.
template <int OFF>
__device__ __forceinline__ void dma16_o(const void* g, unsigned lds) {
  asm volatile("s_add_u32 m0, %0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               :
               : "s"(__builtin_amdgcn_readfirstlane(lds)), "v"(g), "n"(OFF)
               : "memory", "scc");
}
template <int OFF>
__device__ __forceinline__ void dma16_so(const unsigned char* base, unsigned off, unsigned lds) {
  asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(__builtin_amdgcn_readfirstlane(lds)), "v"(off), "s"(uniform_ptr(base)), "n"(OFF)
               : "memory", "scc");
}
// 4 bytes per lane, lane l's at LDS address lds + 4 l
__device__ __forceinline__ void dma4_at(const void* g, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off"
               :
               : "s"(lds), "v"(g)
               : "memory");
}

typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8_t;
typedef int int32x4 __attribute__((ext_vector_type(4)));
typedef int int32x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) int32x4 lds_int32x4_t;

template <int MODE, bool F8>
__global__ __launch_bounds__(256, 1) void gemm_r192_kernel(
    const typename std::conditional<F8, uint8_t, bf16_t>::type* __restrict__ A,
    const int32_t* __restrict__ rows, const int32_t* __restrict__ goff, int G, int64_t m_total,
    const typename std::conditional<F8, uint8_t, bf16_t>::type* __restrict__ B, int K, int NOUT,
    bf16_t* __restrict__ C, int ldc, int hmax, const float* __restrict__ sA,
    const float* __restrict__ sB) {
  using TE = typename std::conditional<F8, uint8_t, bf16_t>::type;
  using FragT = typename std::conditional<F8, int32x8, bf16x8>::type;
  using AccT = typename std::conditional<F8, floatx16, floatx4>::type;
  constexpr int ES = sizeof(TE), CE = 16 / ES;     // bytes, elements per 16-byte chunk
  constexpr int NT = 256, BM = 192, BN = 256;
  constexpr int ROWB = 128, BK = ROWB / ES;        // staged bytes per row and K block
  constexpr int FR = F8 ? 32 : 16;                 // fragment rows
  constexpr int HU = 2 * FR;                       // tile heights: multiples of this
  constexpr int ASTAGE = BM * ROWB, BSTAGE = BN * ROWB;   // two A slots, three B slots
  constexpr int NCOL = MODE == MODE_GATEUP ? BN / 2 : BN;
  constexpr int TN = 128 / FR, B_LD = 8, A_MAX = BM / 32; // B fragments, DMAs per wave
  constexpr int TMIN = 128 / HU;                   // shorter tiles take this loop
  __shared__ int s_goff[kMaxGroups + 1];
  __shared__ int s_tpre[kMaxGroups + 1];
  __shared__ int s_wtot[NT / 64];
  __shared__ int s_cnt[NT / 64][3];
  __shared__ __align__(16) int s_rows[NT];         // row indices of a tile
  __shared__ __align__(16) float s_sa[F8 ? NT : 4], s_sb[F8 ? NT : 4];   // its scales
  __shared__ __align__(1024) unsigned char ring[2 * ASTAGE + 3 * BSTAGE];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int lr = lane & (FR - 1), lh = lane / FR;  // fragment row, K part (and column part)
  auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
  const int nn = NOUT / NCOL;
  sched_offsets<NT>(goff, G, m_total, s_goff);
  if (hmax == 0) {
    // the pass's largest tile height, from the m-tiles of all groups at each
    int cnt[3] = {0, 0, 0};
    for (int g = tid; g < G; g += NT) {
      const int n = max(s_goff[g + 1] - s_goff[g], 0);
      cnt[0] += (n + 191) / 192;
      if constexpr (!F8) cnt[1] += (n + 159) / 160;
      cnt[2] += (n + 127) / 128;
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const int n = wave_sum_i(cnt[i]);
      if (lane == 0) s_cnt[wave][i] = n;
    }
    __syncthreads();
    int t[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) t[i] = uni(s_cnt[0][i] + s_cnt[1][i] + s_cnt[2][i] + s_cnt[3][i]);
    hmax = uni(tall_height(uni(s_goff[G] - s_goff[0]), t[0], t[1], t[2], nn, (int)gridDim.x));
  }
  sched_tiles<NT>(G, s_goff, s_tpre, s_wtot, hmax);
  const int64_t total = (int64_t)nn * uni(s_tpre[G]);
  const int64_t per_xcd = (total + kXcd - 1) / kXcd;
  const int64_t xcd_base = (int64_t)(blockIdx.x % kXcd) * per_xcd;
  const int64_t stride = gridDim.x / kXcd;
  const size_t bstride = (size_t)(MODE == MODE_GATEUP ? 2 * NOUT : NOUT) * K;
  const int KT = K / BK;                           // at least 4
  // a DMA copies 8 rows of 128 bytes: lane l row l / 8, and the 16-byte chunk
  // that belongs at position l % 8 of that row (chunk c of row r sits at
  // c ^ ((r / 2) % 8), so that the lanes an LDS read serves together cover
  // every bank once)
  const int drow = lane >> 3, dpos = lane & 7;
  const unsigned ring_lds = lds_addr(ring);
  const unsigned ldsA = ring_lds + wave * 1024;
  const unsigned ldsB = ring_lds + 2 * ASTAGE + wave * (B_LD * 1024);

  // LDS address of this lane's bytes of a fragment row in each half block
  // (16 bytes for bf16; for FP8 32, the second 16 at position ^ 1), from the
  // wave's first A and B fragment
  const int sw = (lr >> 1) & 7;
  unsigned ab[2], bb[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int fo = lr * ROWB + (((ks * 4 + (F8 ? 2 * lh : lh)) ^ sw) << 4);
    ab[ks] = ring_lds + wm * FR * ROWB + fo;
    bb[ks] = ring_lds + 2 * ASTAGE + wn * (MODE == MODE_GATEUP ? 64 : 128) * ROWB + fo;
  }
  // B DMA i of this wave fills tile rows 64 wave + 8 i ..; row r of each 32
  // holds the output column that puts consecutive columns into a lane's
  // accumulators: bf16 row 16 t + 4 q + v column 8 q + 4 t + v, FP8 row
  // 8 a + 4 h + b column 16 h + 4 a + b
  unsigned bl[B_LD];
#pragma unroll
  for (int i = 0; i < B_LD; ++i) {
    const int r = (i & 3) * 8 + drow;
    const int col = F8 ? 16 * ((r >> 2) & 1) + 4 * (r >> 3) + (r & 3)
                       : 8 * ((r & 15) >> 2) + 4 * (r >> 4) + (r & 3);
    bl[i] = (unsigned)(((i >> 2) * 32 + col) * K * ES + (dpos ^ ((r >> 1) & 7)) * 16);
  }

  struct Item {
    int g, m0, n0, row_base, rows_t, tma;
  };
  int ghint = 0;
  auto decode = [&](int64_t L, Item& it) {
    it.g = uni(find_group_from(s_tpre, G, nn, L, ghint));
    ghint = it.g;
    const int Tg = uni(s_tpre[it.g + 1]) - uni(s_tpre[it.g]);
    const int local = uni((int)(L - (int64_t)nn * s_tpre[it.g]));
    int mt, nt;
    tall_order(local, Tg, nn, mt, nt);
    it.n0 = nt * NCOL;
    it.row_base = uni(s_goff[it.g]);
    const int rows_g = uni(s_goff[it.g + 1]) - it.row_base;
    const int h = tall_rows(rows_g, Tg, HU);
    it.m0 = mt * h;
    it.rows_t = min(rows_g - it.m0, h);
    it.tma = max(TMIN, (it.rows_t + HU - 1) / HU);
  };
  // row indices of an item's rows into s_rows (rows past its end: the last)
  auto fetch_rows = [&](const Item& it) {
    dma4_at(rows + it.row_base + it.m0 + min(wave * 64 + lane, it.rows_t - 1),
            lds_addr(s_rows) + wave * 256);
  };
  // FP8: the scales of an item's rows and weight rows, the latter in the order
  // of the B tile's columns.  Gate/up: a wave reads only the row indices that
  // it copied itself (past the item's end they repeat the last row), since
  // another wave may already have replaced its own by the next item's.
  auto fetch_scales = [&](const Item& it) {
    const int c = wave * 64 + lane;
    const int r = (MODE == MODE_GATEUP && rows) ? s_rows[c] : it.row_base + it.m0 + min(c, it.rows_t - 1);
    dma4_at(sA + r, lds_addr(s_sa) + wave * 256);
    const float* sg = sB + (size_t)it.g * (MODE == MODE_GATEUP ? 2 * NOUT : NOUT) + it.n0;
    dma4_at(sg + (MODE == MODE_GATEUP && c >= 128 ? NOUT + c - 128 : c), lds_addr(s_sb) + wave * 256);
  };
  // the copies' sources: the next block of this wave's A rows (A DMA i fills
  // tile rows 32 i + 8 wave ..) and B rows
  const TE* pa[A_MAX];
  const unsigned char* pb = nullptr;
  auto sources_a = [&](const Item& it) {
#pragma unroll
    for (int i = 0; i < A_MAX; ++i) {
      const int r = min((4 * i + wave) * 8 + drow, it.rows_t - 1);
      const int v = (MODE == MODE_GATEUP && rows) ? s_rows[r] : it.row_base + it.m0 + r;
      pa[i] = A + (size_t)v * K + (dpos ^ ((wave & 1) * 4 + (drow >> 1))) * CE;
    }
  };
  auto source_b = [&](const Item& it) {
    const int wrow0 = MODE == MODE_GATEUP ? (wave >> 1) * NOUT + it.n0 + (wave & 1) * 64
                                          : it.n0 + wave * 64;
    pb = reinterpret_cast<const unsigned char*>(
        uniform_ptr(B + (size_t)it.g * bstride + (size_t)wrow0 * K));
  };

  Item it, itN;
  int64_t j = blockIdx.x / kXcd;
  if (j >= per_xcd || xcd_base + j >= total) return;   // a whole workgroup
  decode(xcd_base + j, it);
  if (MODE == MODE_GATEUP && rows) {
    fetch_rows(it);
    wait_vmcnt<0>();
    __syncthreads();
  }
  sources_a(it);
  source_b(it);
  // LDS offsets of the slots of the current block, the next (and, B, the one
  // after)
  unsigned oa0 = 0, oa1 = ASTAGE, ob0 = 0, ob1 = BSTAGE, ob2 = 2 * BSTAGE;
  auto copy_a = [&](unsigned oa) __attribute__((always_inline)) {
    static_for<A_MAX>([&](auto I) __attribute__((always_inline)) {
      constexpr int i = decltype(I)::value;
      dma16_o<i * 4096>(pa[i], ldsA + oa);
      pa[i] += BK;
    });
  };
  auto copy_b = [&](unsigned ob) __attribute__((always_inline)) {
    static_for<B_LD>([&](auto I) __attribute__((always_inline)) {
      constexpr int i = decltype(I)::value;
      dma16_so<i * 1024>(pb, bl[i], ldsB + ob);
    });
    pb += ROWB;
  };
  copy_a(oa0);
  copy_b(ob0);
  copy_b(ob1);
  copy_a(oa1);
  copy_b(ob2);

  for (;;) {
    const bool has_next = j + stride < per_xcd && xcd_base + j + stride < total;
    // without a next item the copies past this one's end re-read its own rows
    itN = it;
    if (has_next) decode(xcd_base + j + stride, itN);
    auto tile = [&](auto TMA) __attribute__((always_inline)) {
      constexpr int TM = decltype(TMA)::value;
      constexpr int A_LD = TM * (HU / 32);
      constexpr int MPS = TM * TN, NR = TM + TN;
      AccT acc[TM][TN];
      static_for<TM * TN>([&](auto q) __attribute__((always_inline)) {
        if constexpr (F8)
          acc[q / TN][q % TN] = AccT{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                                     0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        else
          acc[q / TN][q % TN] = AccT{0.f, 0.f, 0.f, 0.f};
      });
      FragT F[2][TM + TN];
      // fragment r of the half block at LDS addresses la (A) and lb (B), in
      // the order the MFMAs use them: A0, all B, A1 ..  (FP8: la2 / lb2 are
      // the addresses of the lane's second 16 bytes)
      auto read1 = [&](FragT (&f)[TM + TN], unsigned la, unsigned lb, unsigned la2, unsigned lb2,
                       auto R) __attribute__((always_inline)) {
        constexpr int r = decltype(R)::value;
        constexpr int x = r == 0 ? 0 : (r <= TN ? TM + r - 1 : r - TN);
        constexpr int n = x - TM;
        constexpr int off = x < TM ? x * HU * ROWB
                            : MODE == MODE_GATEUP
                                ? ((n % (TN / 2)) * FR + (n / (TN / 2)) * 128) * ROWB
                                : n * FR * ROWB;
        const unsigned p = (x < TM ? la : lb) + off;
        if constexpr (F8) {
          const int32x4 lo = *(const lds_int32x4_t*)(uintptr_t)p;
          const int32x4 hi = *(const lds_int32x4_t*)(uintptr_t)((x < TM ? la2 : lb2) + off);
          f[x] = int32x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        } else {
          f[x] = *(const lds_bf16x8_t*)(uintptr_t)p;
        }
      };
      // block 0 has landed in every wave (after it, B 1, A 1, B 2)
      wait_vmcnt<A_MAX + 2 * B_LD>();
      barrier_nofence();
      if constexpr (F8) fetch_scales(it);
      // gate/up: the next tile's row indices; down: this tile's
      if (rows) fetch_rows(MODE == MODE_DOWN ? it : itN);
      {
        const unsigned la = ab[0] + oa0, lb = bb[0] + ob0;
        static_for<NR>([&](auto r) __attribute__((always_inline)) {
          read1(F[0], la, lb, la ^ 16, lb ^ 16, r);
        });
      }
      // Half block KS of a block: its MFMAs on fc, the reads of the next half
      // block into fn between them.  In the second half the workgroup meets
      // after the first MFMA: the next block has landed (only the B copies
      // of the block after it may be in flight), and every wave holds this
      // half in registers, so the block's slots are free.  The A copies of
      // the block two ahead and the B copies of the block three ahead go out
      // there.  WHEN: 0 all of them are this item's, 1 the B copies are the
      // next item's (the item's third last block), 2 all are (its second
      // last), 3 so in its last block.
      auto half = [&](FragT (&fc)[TM + TN], FragT (&fn)[TM + TN], auto KS, auto WHEN)
          __attribute__((always_inline)) {
        constexpr int ks = decltype(KS)::value, when = decltype(WHEN)::value;
        constexpr bool end = when == 3 && ks == 1;
        // the next half block's fragments; opaque, so that their addresses
        // stay a few registers and immediate offsets
        unsigned la = ab[ks ^ 1] + (ks == 0 ? oa0 : oa1);
        unsigned lb = bb[ks ^ 1] + (ks == 0 ? ob0 : ob1);
        asm volatile("" : "+v"(la), "+v"(lb));
        unsigned la2 = la ^ 16, lb2 = lb ^ 16;
        if constexpr (F8) asm volatile("" : "+v"(la2), "+v"(lb2));
        static_for<MPS>([&](auto Q) __attribute__((always_inline)) {
          constexpr int q = decltype(Q)::value;
          constexpr int i = q / TN, n = q % TN;
          if constexpr (F8)
            acc[i][n] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fc[TM + n], fc[i], acc[i][n],
                                                                        0, 0, 0, 127, 0, 127);
          else
            acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fc[TM + n], fc[i], acc[i][n], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (q == 0 && ks == 1) {
            wait_lgkm0();
            if constexpr (!end) wait_vmcnt<B_LD>();
            barrier_nofence();
            __builtin_amdgcn_sched_barrier(0);
          }
          if constexpr (!end)
            static_for<NR>([&](auto R) __attribute__((always_inline)) {
              constexpr int at = F8 ? decltype(R)::value * MPS * 3 / 4 / NR
                                    : 1 + decltype(R)::value * (MPS * 3 / 4) / NR;
              if constexpr (q == at) read1(fn, la, lb, la2, lb2, R);
            });
          if constexpr (ks == 1)
            static_for<A_MAX + B_LD>([&](auto D) __attribute__((always_inline)) {
              constexpr int d = decltype(D)::value;
              constexpr int at = F8 ? d * (MPS - 1) / (A_MAX + B_LD) : 1 + d * (MPS - 2) / (A_MAX + B_LD);
              if constexpr (q == at) {
                if constexpr (d < A_MAX) {
                  if constexpr (when >= 2 || d < A_LD) {
                    dma16_o<d * 4096>(pa[d], ldsA + oa0);
                    pa[d] += BK;
                  }
                } else {
                  dma16_so<(d - A_MAX) * 1024>(pb, bl[d - A_MAX], ldsB + ob0);
                  if constexpr (d == A_MAX + B_LD - 1) pb += ROWB;
                }
              }
            });
          __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (ks == 1) {
          const unsigned o = ob0, p = oa0;
          ob0 = ob1;
          ob1 = ob2;
          ob2 = o;
          oa0 = oa1;
          oa1 = p;
        }
      };
      using I0 = std::integral_constant<int, 0>;
      using I1 = std::integral_constant<int, 1>;
      using I2 = std::integral_constant<int, 2>;
      using I3 = std::integral_constant<int, 3>;
      for (int kt = 0; kt + 3 < KT; ++kt) {
        half(F[0], F[1], I0{}, I0{});
        half(F[1], F[0], I1{}, I0{});
      }
      source_b(itN);
      half(F[0], F[1], I0{}, I1{});
      half(F[1], F[0], I1{}, I1{});
      // (the next item's row indices landed by the meeting in this item's
      // second block; its copies fill every row block, whatever its height)
      sources_a(itN);
      half(F[0], F[1], I0{}, I2{});
      half(F[1], F[0], I1{}, I2{});
      half(F[0], F[1], I0{}, I3{});
      half(F[1], F[0], I1{}, I3{});
      // a use of every accumulator here: else the compiler sinks the FP8 MFMAs
      // of the last blocks into the epilogue's branches, past the copies
      if constexpr (F8)
        static_for<TM * TN>([&](auto q) __attribute__((always_inline)) {
          const AccT& x = acc[q / TN][q % TN];
          asm volatile("" : : "a"(x));
        });
      // (this tile's row indices and scales landed by its second block)
      // epilogue: a lane's columns are consecutive (bf16: element v of
      // fragments 2p, 2p + 1 is column 8 lh + v (+ 4) of the wave's p-th 32;
      // FP8: element v of fragment p column 16 lh + v), of row lr of the
      // fragment
      static_for<TM>([&](auto I) __attribute__((always_inline)) {
        constexpr int i = decltype(I)::value;
        const int m = i * HU + wm * FR + lr;
        if (m < it.rows_t) {
          int64_t orow = it.row_base + it.m0 + m;
          if (MODE == MODE_DOWN && rows) orow = s_rows[m];
          const int wc = wn * (MODE == MODE_GATEUP ? 64 : 128);
          bf16_t* p = C + orow * ldc + it.n0 + wc + (F8 ? 16 : 8) * lh;
          const float sa = F8 ? s_sa[m] : 1.f;
          static_for<(MODE == MODE_GATEUP ? 2 : 4)>([&](auto P) __attribute__((always_inline)) {
            constexpr int n = decltype(P)::value;
            if constexpr (F8) {
              // (opaque, and a scheduling barrier after each store: else every
              // column scale is read at once, into more registers than there are)
              unsigned sbo = wc + 32 * n + 16 * lh;
              asm volatile("" : "+v"(sbo));
              const float* sb = s_sb + sbo;
              static_for<2>([&](auto S) __attribute__((always_inline)) {
                constexpr int s0 = decltype(S)::value * 8;
                Vec16<bf16_t> o;
#pragma unroll
                for (int v = 0; v < 8; ++v) {
                  const float x = acc[i][n][s0 + v] * sa * sb[s0 + v];
                  if constexpr (MODE == MODE_GATEUP)
                    o.set(v, swiglu_bf16_epi(x, acc[i][2 + n][s0 + v] * sa * sb[128 + s0 + v]));
                  else
                    o.set(v, x);
                }
                st16(p + 32 * n + s0, o.raw);
                __builtin_amdgcn_sched_barrier(0);
              });
            } else {
              Vec16<bf16_t> o;
#pragma unroll
              for (int v = 0; v < 8; ++v) {
                const float x = acc[i][2 * n + (v >> 2)][v & 3];
                if constexpr (MODE == MODE_GATEUP)
                  o.set(v, swiglu_bf16_epi(x, acc[i][4 + 2 * n + (v >> 2)][v & 3]));
                else
                  o.set(v, x);
              }
              st16(p + 32 * n, o.raw);
            }
          });
        }
      });
    };
    if constexpr (F8) {
      if (it.tma == 2)
        tile(std::integral_constant<int, 2>{});
      else
        tile(std::integral_constant<int, 3>{});
    } else {
      switch (it.tma) {
        case 4: tile(std::integral_constant<int, 4>{}); break;
        case 5: tile(std::integral_constant<int, 5>{}); break;
        default: tile(std::integral_constant<int, 6>{}); break;
      }
    }
    if (!has_next) break;
    j += stride;
    it = itN;
  }
  wait_vmcnt<0>();   // no copy outlives the workgroup's LDS
}

template <int MODE, bool F8>
void run_r192(const void* A, const int32_t* rows, const int32_t* goff, int G, int64_t m_total,
              const void* B, int K, int NOUT, void* C, int ldc, int cus, int hmax, const float* sA,
              const float* sB, hipStream_t s) {
  using TE = typename std::conditional<F8, uint8_t, bf16_t>::type;
  const int64_t tiles = (cdiv64(m_total, hmax ? hmax : 128) + G) * (NOUT / (MODE == MODE_GATEUP ? 128 : 256));
  const int64_t grid = std::min<int64_t>(cdiv64(tiles, kXcd), cdiv64(cus, kXcd)) * kXcd;
  launch_k(gemm_r192_kernel<MODE, F8>, (unsigned)grid, 256, 0, s, (const TE*)A, rows, goff, G,
           m_total, (const TE*)B, K, NOUT, (bf16_t*)C, ldc, hmax, sA, sB);
}

}  // namespace
}  // namespace fs
