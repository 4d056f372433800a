// Grouped SwiGLU FFN passes on tiles of up to 192 rows x 256 weight rows, for
// groups of a hundred rows and more (Section 2.1, prefill).
//
// What bounds the 128 x 256 ring (gemm.hip) is not the matrix cores but the
// stream of L2 requests that fills its LDS: about 100 G requests/s over the
// chip, 48 KB per 64-wide K block of a tile (one L2 request per 128-byte
// row), its copies alone taking as long as the pass; the same loop without
// copies runs 1.8 times faster.  (A first version of this kernel with 64-byte
// rows, 256 x 256 x 32 tiles, made as many requests for half the bytes and
// was no faster than the ring.)  So the tile is taller, and the wave tile
// larger: four waves (2 x 2), one per SIMD, each up to 96 x 128 through
// v_mfma_f32_16x16x32_bf16, 192 accumulators; an LDS fragment read feeds six
// or eight MFMAs.
//
//   Heights  A group's tiles have equal heights, a multiple of 32 up to 192,
//            so the last tile is not a stub; the tile's code is one loop per
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
// Measured (us, ring -> this): 8192 rows, d 5120, F 8192, dense gate/up 1228
// -> 998 (1.38 PFLOP/s, as fast as the vendor library's dense kernel), down
// 590 -> 546; 16 groups of about 512 rows of the same: 1410 -> 1307 and 706
// -> 673; 32 groups of 1024 rows, d 7168, F 2048: 1755 -> 1670 and 978 ->
// 829; 64 groups of 384 rows, d 2048, F 1408: 347 -> 300 and 199 -> 178.
#pragma once

#include <algorithm>
#include <type_traits>
#include <utility>

#include "gemm_common.hpp"
#include "internal.hpp"

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

typedef __attribute__((address_space(3))) bf16x8 lds_frag_t;

template <int MODE>
__global__ __launch_bounds__(256, 1) void gemm_r192_kernel(
    const bf16_t* __restrict__ A, const int32_t* __restrict__ rows,
    const int32_t* __restrict__ goff, int G, int64_t m_total, const bf16_t* __restrict__ B, int K,
    int NOUT, bf16_t* __restrict__ C, int ldc, int hmax) {
  constexpr int NT = 256, BM = 192, BN = 256;
  constexpr int ROWB = 128;                        // staged bytes per row and K block (64 bf16)
  constexpr int BK = 64;
  constexpr int ASTAGE = BM * ROWB, BSTAGE = BN * ROWB;   // two A slots, three B slots
  constexpr int NCOL = MODE == MODE_GATEUP ? BN / 2 : BN;
  constexpr int TN = 8, TMAX = BM / 32, B_LD = 8;
  __shared__ int s_goff[kMaxGroups + 1];
  __shared__ int s_tpre[kMaxGroups + 1];
  __shared__ int s_wtot[NT / 64];
  __shared__ __align__(16) int s_rows[NT];         // row indices of a tile
  __shared__ __align__(1024) unsigned char ring[2 * ASTAGE + 3 * BSTAGE];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int l16 = lane & 15, quad = lane >> 4;
  auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
  sched_setup<NT>(goff, G, m_total, s_goff, s_tpre, s_wtot, hmax);
  const int nn = NOUT / NCOL;
  const int64_t total = (int64_t)nn * uni(s_tpre[G]);
  const int64_t per_xcd = (total + kXcd - 1) / kXcd;
  const int64_t xcd_base = (int64_t)(blockIdx.x % kXcd) * per_xcd;
  const int64_t stride = gridDim.x / kXcd;
  const size_t bstride = (size_t)(MODE == MODE_GATEUP ? 2 * NOUT : NOUT) * K;
  const int KT = K / BK;                           // even, at least 4
  // a DMA copies 8 rows of 128 bytes: lane l row l / 8, and the 16-byte chunk
  // that belongs at position l % 8 of that row (chunk c of row r sits at
  // c ^ ((r / 2) % 8))
  const int drow = lane >> 3, dpos = lane & 7;
  const unsigned ring_lds = lds_addr(ring);
  const unsigned ldsB = ring_lds + 2 * ASTAGE + wave * (B_LD * 1024);

  // this lane's 16 bytes of a fragment row in each half block, from the
  // wave's first A and B fragment
  const int sw = (l16 >> 1) & 7;
  unsigned ab[2], bb[2];                           // LDS byte addresses
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int fo = l16 * ROWB + (((ks * 4 + quad) ^ sw) << 4);
    ab[ks] = ring_lds + wm * 16 * ROWB + fo;
    bb[ks] = ring_lds + 2 * ASTAGE + wn * (MODE == MODE_GATEUP ? 64 : 128) * ROWB + fo;
  }
  // B DMA i of this wave fills tile rows 64 wave + 8 i ..: of each 32 rows,
  // row 16 t + 4 q + v holds output column 8 q + 4 t + v
  unsigned bl[B_LD];
#pragma unroll
  for (int i = 0; i < B_LD; ++i)
    bl[i] = (unsigned)(((i >> 2) * 32 + (i & 1) * 16 + ((i >> 1) & 1) * 4 + (drow >> 2) * 8 +
                        (drow & 3)) * K * 2 + (dpos ^ ((i & 1) * 4 + (drow >> 1))) * 16);

  struct Item {
    int g, m0, n0, row_base, rows_t, tma;
  };
  int ghint = 0;
  auto decode = [&](int64_t L, Item& it) {
    it.g = uni(find_group_from(s_tpre, G, nn, L, ghint));
    ghint = it.g;
    const int Tg = uni(s_tpre[it.g + 1]) - uni(s_tpre[it.g]);
    int local = uni((int)(L - (int64_t)nn * s_tpre[it.g]));
    // m-tiles in bands of at most 8, a band's m-tiles fastest, then the
    // n-tiles: the tiles an XCD runs together share both operands
    const int bands = uni((Tg + 7) / 8), bh = uni((Tg + bands - 1) / bands);
    const int band = uni(local / (nn * bh));
    local -= band * nn * bh;
    const int bw = min(bh, Tg - band * bh);
    const int nt = uni(local / bw), mt = band * bh + local - nt * bw;
    it.n0 = nt * NCOL;
    it.row_base = uni(s_goff[it.g]);
    const int rows_g = uni(s_goff[it.g + 1]) - it.row_base;
    // the group's tiles have equal heights, a multiple of 32 rows
    const int h = uni(((rows_g + Tg - 1) / Tg + 31) & ~31);
    it.m0 = mt * h;
    it.rows_t = min(rows_g - it.m0, h);
    it.tma = max(4, (it.rows_t + 31) / 32);
  };
  // row indices of an item's rows into s_rows (rows past its end: the last)
  auto fetch_rows = [&](const Item& it) {
    dma4_at(rows + it.row_base + it.m0 + min(wave * 64 + lane, it.rows_t - 1),
            lds_addr(s_rows) + wave * 256);
  };
  // the copies' sources: the next block of this wave's A rows (tma DMAs) and
  // B rows
  const bf16_t* pa[TMAX];
  const unsigned char* pb = nullptr;
  auto sources_a = [&](const Item& it) {
#pragma unroll
    for (int i = 0; i < TMAX; ++i) {
      const int blk = wave * it.tma + i;
      const int r = min(blk * 8 + drow, it.rows_t - 1);
      const int v = (MODE == MODE_GATEUP && rows) ? s_rows[r] : it.row_base + it.m0 + r;
      pa[i] = A + (size_t)v * K + (dpos ^ (((blk & 1) * 4 + (drow >> 1)) & 7)) * 8;
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
  unsigned ldsA = ring_lds + wave * it.tma * 1024;
  // LDS offsets of the B slots of the current block, the next and the one
  // after
  unsigned ob0 = 0, ob1 = BSTAGE, ob2 = 2 * BSTAGE;
  auto copy_a = [&](auto S) __attribute__((always_inline)) {
    static_for<TMAX>([&](auto I) __attribute__((always_inline)) {
      constexpr int i = decltype(I)::value;
      if (i < it.tma) dma16_o<decltype(S)::value * ASTAGE + i * 1024>(pa[i], ldsA);
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
  copy_a(std::integral_constant<int, 0>{});
  copy_b(ob0);
  copy_b(ob1);
  copy_a(std::integral_constant<int, 1>{});
  copy_b(ob2);

  for (;;) {
    const bool has_next = j + stride < per_xcd && xcd_base + j + stride < total;
    if (has_next) decode(xcd_base + j + stride, itN);
    auto tile = [&](auto TMA) __attribute__((always_inline)) {
      constexpr int TM = decltype(TMA)::value;
      constexpr int MPS = TM * TN, NR = TM + TN;
      floatx4 acc[TM][TN];
      static_for<TM * TN>([&](auto q) __attribute__((always_inline)) {
        acc[q / TN][q % TN] = floatx4{0.f, 0.f, 0.f, 0.f};
      });
      bf16x8 F[2][TM + TN];
      // fragment r of the half block at LDS addresses la (A) and lb (B), in
      // the order the MFMAs use them: A0, B0 .. B7, A1 ..
      auto read1 = [&](bf16x8 (&f)[TM + TN], unsigned la, unsigned lb, auto R)
          __attribute__((always_inline)) {
        constexpr int r = decltype(R)::value;
        constexpr int x = r == 0 ? 0 : (r <= TN ? TM + r - 1 : r - TN);
        constexpr int n = x - TM;
        if constexpr (x < TM)
          f[x] = *(const lds_frag_t*)(uintptr_t)(la + x * 32 * ROWB);
        else
          f[x] = *(const lds_frag_t*)(uintptr_t)(
              lb + (MODE == MODE_GATEUP ? (n & 3) * 16 + (n >> 2) * 128 : n * 16) * ROWB);
      };
      using I0 = std::integral_constant<int, 0>;
      using I1 = std::integral_constant<int, 1>;
      // block 0 has landed in every wave (after it, at least 20 copies)
      wait_vmcnt<20>();
      barrier_nofence();
      // gate/up: the next tile's row indices; down: this tile's
      if (rows && (MODE == MODE_DOWN || has_next)) fetch_rows(MODE == MODE_DOWN ? it : itN);
      static_for<NR>([&](auto r) __attribute__((always_inline)) { read1(F[0], ab[0], bb[0] + ob0, r); });
      // Half block KS of a block (A slot S): its MFMAs on fc, the reads of the
      // next half block into fn between them.  In the second half the
      // workgroup meets after the first MFMA: the next block has landed (only
      // the B copies of the block after it may be in flight), and every wave
      // holds this half in registers, so the block's slots are free.  The A
      // copies of the block two ahead and the B copies of the block three
      // ahead go out there.  WHEN: 0 all of them are this item's, 1 the
      // second block's B copies are the next item's (the item's last four
      // blocks begin), 2 all are the next item's.
      auto half = [&](bf16x8 (&fc)[TM + TN], bf16x8 (&fn)[TM + TN], int tmaN, auto S, auto KS,
                      auto WHEN) __attribute__((always_inline)) {
        constexpr int slot = decltype(S)::value, ks = decltype(KS)::value;
        constexpr int when = decltype(WHEN)::value;
        constexpr bool last = when == 2;
        constexpr bool end = last && slot == 1 && ks == 1;
        constexpr bool nextb = last || (when == 1 && slot == 1);
        // the next half block's fragments; opaque, so that their addresses
        // stay two registers and immediate offsets
        unsigned la = ab[ks ^ 1] + (ks == 0 ? slot : slot ^ 1) * ASTAGE;
        unsigned lb = bb[ks ^ 1] + (ks == 0 ? ob0 : ob1);
        asm volatile("" : "+v"(la), "+v"(lb));
        static_for<MPS>([&](auto Q) __attribute__((always_inline)) {
          constexpr int q = decltype(Q)::value;
          constexpr int i = q / TN, n = q % TN;
          acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fc[TM + n], fc[i], acc[i][n], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (q == 0 && ks == 1) {
            wait_lgkm0();
            if constexpr (!end) {
              if (!last || has_next)
                wait_vmcnt<B_LD>();
              else
                wait_vmcnt<0>();
            }
            barrier_nofence();
            __builtin_amdgcn_sched_barrier(0);
          }
          if constexpr (!end)
            static_for<NR>([&](auto R) __attribute__((always_inline)) {
              if constexpr (q == 1 + decltype(R)::value * (MPS * 3 / 4) / NR) read1(fn, la, lb, R);
            });
          if constexpr (ks == 1)
            static_for<TMAX + B_LD>([&](auto D) __attribute__((always_inline)) {
              constexpr int d = decltype(D)::value;
              if constexpr (q == 1 + d * (MPS - 2) / (TMAX + B_LD)) {
                if constexpr (d < TMAX) {
                  if constexpr (!last) {
                    if constexpr (d < TM) dma16_o<slot * ASTAGE + d * 1024>(pa[d], ldsA);
                  } else {
                    if (d < tmaN) dma16_o<slot * ASTAGE + d * 1024>(pa[d], ldsA);
                  }
                  pa[d] += BK;
                } else {
                  if (!nextb || has_next)
                    dma16_so<(d - TMAX) * 1024>(pb, bl[d - TMAX], ldsB + ob0);
                  if constexpr (d == TMAX + B_LD - 1) pb += ROWB;
                }
              }
            });
          __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (ks == 1) {
          const unsigned o = ob0;
          ob0 = ob1;
          ob1 = ob2;
          ob2 = o;
        }
      };
      using W0 = std::integral_constant<int, 0>;
      using W1 = std::integral_constant<int, 1>;
      using W2 = std::integral_constant<int, 2>;
      for (int kt = 0; kt + 4 < KT; kt += 2) {
        half(F[0], F[1], 0, I0{}, I0{}, W0{});
        half(F[1], F[0], 0, I0{}, I1{}, W0{});
        half(F[0], F[1], 0, I1{}, I0{}, W0{});
        half(F[1], F[0], 0, I1{}, I1{}, W0{});
      }
      half(F[0], F[1], 0, I0{}, I0{}, W1{});
      half(F[1], F[0], 0, I0{}, I1{}, W1{});
      if (has_next) source_b(itN);
      half(F[0], F[1], 0, I1{}, I0{}, W1{});
      half(F[1], F[0], 0, I1{}, I1{}, W1{});
      // (none of the A copies without a next item: tmaN 0; its row indices
      // landed by the meeting in this item's second block)
      int tmaN = 0;
      if (has_next) {
        sources_a(itN);
        tmaN = itN.tma;
        ldsA = ring_lds + wave * tmaN * 1024;
      }
      half(F[0], F[1], tmaN, I0{}, I0{}, W2{});
      half(F[1], F[0], tmaN, I0{}, I1{}, W2{});
      half(F[0], F[1], tmaN, I1{}, I0{}, W2{});
      half(F[1], F[0], tmaN, I1{}, I1{}, W2{});
      // (this tile's row indices landed by its second block)
      // epilogue: element v of fragments 2p, 2p + 1 is column 8 quad + v (+ 4)
      // of the wave's p-th 32 columns, row l16 of the fragment
      static_for<TM>([&](auto I) __attribute__((always_inline)) {
        constexpr int i = decltype(I)::value;
        const int m = i * 32 + wm * 16 + l16;
        if (m < it.rows_t) {
          int64_t orow = it.row_base + it.m0 + m;
          if (MODE == MODE_DOWN && rows) orow = s_rows[m];
          bf16_t* p = C + orow * ldc + it.n0 + wn * (MODE == MODE_GATEUP ? 64 : 128) + 8 * quad;
          static_for<(MODE == MODE_GATEUP ? 2 : 4)>([&](auto P) __attribute__((always_inline)) {
            constexpr int n = decltype(P)::value;
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
          });
        }
      });
    };
    switch (it.tma) {
      case 4: tile(std::integral_constant<int, 4>{}); break;
      case 5: tile(std::integral_constant<int, 5>{}); break;
      default: tile(std::integral_constant<int, 6>{}); break;
    }
    if (!has_next) break;
    j += stride;
    it = itN;
  }
}

template <int MODE>
void run_r192(const void* A, const int32_t* rows, const int32_t* goff, int G, int64_t m_total,
              const void* B, int K, int NOUT, void* C, int ldc, int cus, int hmax, hipStream_t s) {
  const int64_t tiles = (cdiv64(m_total, hmax) + G) * (NOUT / (MODE == MODE_GATEUP ? 128 : 256));
  const int64_t grid = std::min<int64_t>(cdiv64(tiles, kXcd), cdiv64(cus, kXcd)) * kXcd;
  launch_k(gemm_r192_kernel<MODE>, (unsigned)grid, 256, 0, s, (const bf16_t*)A, rows, goff, G,
           m_total, (const bf16_t*)B, K, NOUT, (bf16_t*)C, ldc, hmax);
}

}  // namespace
}  // namespace fs
