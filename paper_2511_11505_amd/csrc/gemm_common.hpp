// Shared by the grouped GEMM kernels: the ragged-group tile schedule and the
// direct global->LDS copies with their waits.
#pragma once

#include "common.hpp"

namespace fs {
namespace {

constexpr int kMaxGroups = 512;
constexpr int kXcd = 8;
enum { MODE_GATEUP = 0, MODE_DOWN = 1 };

// SiLU(g) * u for the bf16 epilogues, whose result is rounded to bf16: the
// hardware exponential and reciprocal (about 1 ulp each in fp32) replace the
// IEEE division, which costs ten instructions per element.
__device__ __forceinline__ float swiglu_bf16_epi(float g, float u) {
  return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u;
}

// Group offsets in LDS, clamped to [0, m_total]: rows past the host bound are
// never read or written, so a short bound cannot overrun the H workspace.
template <int NT>
__device__ void sched_offsets(const int32_t* __restrict__ goff, int G, int64_t m_total,
                              int* s_goff) {
  for (int g = threadIdx.x; g <= G; g += NT) {
    int v = goff ? goff[g] : (g == 0 ? 0 : (int)m_total);
    s_goff[g] = v < 0 ? 0 : (v > (int)m_total ? (int)m_total : v);
  }
  __syncthreads();
}

// The exclusive prefix of m-tiles (of BM rows) per group, in LDS, from the
// offsets.
template <int NT>
__device__ void sched_tiles(int G, const int* s_goff, int* s_tpre, int* s_wtot, int BM) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int IPT = (kMaxGroups + 1 + NT - 1) / NT;
  int cnt[IPT];
  int local = 0;
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int g = tid * IPT + i;
    const int c = (g < G && s_goff[g + 1] > s_goff[g]) ? (s_goff[g + 1] - s_goff[g] + BM - 1) / BM : 0;
    cnt[i] = c;
    local += c;
  }
  int incl = local;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(incl, o, FS_WAVE);
    if (lane >= o) incl += v;
  }
  if (lane == 63) s_wtot[wave] = incl;
  __syncthreads();
  int pre = 0;
  for (int w = 0; w < wave; ++w) pre += s_wtot[w];
  int run = pre + incl - local;
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int g = tid * IPT + i;
    if (g <= G) s_tpre[g] = run;
    run += cnt[i];
  }
  __syncthreads();
}

template <int NT, int BM>
__device__ __forceinline__ void sched_setup(const int32_t* __restrict__ goff, int G, int64_t m_total,
                                            int* s_goff, int* s_tpre, int* s_wtot) {
  sched_offsets<NT>(goff, G, m_total, s_goff);
  sched_tiles<NT>(G, s_goff, s_tpre, s_wtot, BM);
}

// Largest g in [0, G) with nn * tpre[g] <= L.
__device__ __forceinline__ int find_group(const int* s_tpre, int G, int nn, int64_t L) {
  int lo = 0, hi = G - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if ((int64_t)nn * s_tpre[mid] <= L)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// find_group for a workgroup's items, which come in increasing order: the
// answer is at least lo (the previous item's group), and most often lo or
// lo + 1, so two LDS reads usually settle it before any binary search.
__device__ __forceinline__ int find_group_from(const int* s_tpre, int G, int nn, int64_t L, int lo) {
  if (lo + 1 < G && (int64_t)nn * s_tpre[lo + 1] <= L) {
    ++lo;
    if (lo + 1 < G && (int64_t)nn * s_tpre[lo + 1] <= L) {
      int hi = G - 1;
      ++lo;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if ((int64_t)nn * s_tpre[mid] <= L)
          lo = mid;
        else
          hi = mid - 1;
      }
    }
  }
  return lo;
}

typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) void glb_void_t;

// One direct global->LDS load of 16 bytes per lane: lane l's bytes land at
// LDS address lds + 16 * l, where lds is the wave's destination as a
// wave-uniform 32-bit LDS address (kept in SGPRs by the caller, so a copy
// needs no address-space conversion or lane broadcast).  Issued as inline
// assembly so that the compiler does not add a conservative wait for every
// outstanding DMA before each LDS read; the kernels order them themselves
// with explicit vmcnt waits and barriers.  M0 carries the LDS address and has
// no other user in these kernels.
__device__ __forceinline__ void dma16_at(const void* g, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               :
               : "s"(lds), "v"(g)
               : "memory");
}

// The same with the global address split into a wave-uniform 64-bit base
// (SGPRs) and a 32-bit per-lane byte offset: the weight rows of a wave's DMAs
// share one base, so they hold two VGPRs of offsets instead of a 64-bit
// pointer per DMA.
__device__ __forceinline__ void dma16_sb(const void* base, unsigned off, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(lds), "v"(off), "s"(base)
               : "memory");
}

// A pointer made wave-uniform (held in SGPRs): lane 0's value.
template <typename T>
__device__ __forceinline__ T* uniform_ptr(T* p) {
  const uint64_t v = (uint64_t)(uintptr_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (T*)(uintptr_t)(((uint64_t)hi << 32) | lo);
}

// A 16-byte load marked non-temporal (the streaming hint), for the expert
// weights that the fragment-ordered decode passes read exactly once.
// DeepSeek-V3-shaped decode, routed gate/up 266 -> 239 us (6.43 TB/s, 0.80
// of HBM), down 142 -> 140 us, step 0.531 -> 0.508 ms (same-box A/B).  The
// 64-row shared expert's weight-streaming kernels were slower with it
// (gate/up 28 -> 30 us, down 17 -> 18 us) and keep ordinary loads.
template <typename V>
__device__ __forceinline__ V ld_stream(const void* p) {
  typedef int v4i __attribute__((ext_vector_type(4)));
  static_assert(sizeof(V) == 16, "16-byte loads");
  const v4i v = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(p));
  return __builtin_bit_cast(V, v);
}

// LDS address of a __shared__ location as a wave-uniform 32-bit value.
__device__ __forceinline__ unsigned lds_addr(const void* p) {
  return __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(const lds_void_t*)p);
}

// s_waitcnt with only vmcnt constrained (gfx9 encoding).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

__device__ __forceinline__ void barrier_nofence() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

__device__ __forceinline__ void wait_lgkm0() {
  // lgkmcnt(0), vmcnt and expcnt unconstrained
  __builtin_amdgcn_s_waitcnt((0xF) | (0x3 << 14) | (0x7 << 4) | (0x0 << 8));
}

}  // namespace
}  // namespace fs
