// Device helpers shared by the attention kernels (seg_attn.hip, mq_attn.hip) and the similarity kernels
// (equiv.hip): direct-to-LDS copies, partial-row stores, explicit waits and barriers.
#pragma once

#include "ga_internal.hpp"

namespace ga {

// Multi-query attention of bf16 plans with many query rows (mq_attn.hip): as many workgroups per CU
// as its registers allow (head_dim 128: 242, two waves per SIMD; 64: 165, three).
__host__ __device__ constexpr int mq_wgs_per_cu(int head_dim) { return head_dim == 64 ? 3 : 2; }
hipError_t launch_mq_attn(const AttnArgs& a, int head_dim, int grid, hipStream_t stream,
                          hipEvent_t t0, hipEvent_t t1);

namespace {

// Direct-to-LDS copy of 16 bytes per lane: LDS[lds_base + 16 * lane] <- global[base + off].
// base (the page block) and lds_base are wave-uniform SGPR values, off a per-lane VGPR.  Issued
// as inline assembly so that the compiler's wait-count pass does not treat every later LDS read
// as a possible alias of the copy (it would drain the whole pipeline before each stage);
// ordering is explicit instead: wait_vmcnt() before the barrier that publishes a stage.  M0
// holds the LDS base; the kernel keeps no other value in M0.  The copies are non-temporal (nt):
// every K/V byte is read once per step, and streaming it through the caches at normal priority
// would evict the partial rows this kernel writes and the merge kernel reads back.
// The multi-query (causal) variant copies with the normal cache policy instead: there the row
// blocks of one chunk read the same pages, and the later ones find them in the caches.
// (tests/test_isa_invariants.py checks in the built assembly that every M0 write is one of these.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma16(unsigned off, const void* base, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1 nt"
               :: "v"(off), "s"(base), "s"(lds_base) : "memory", "m0");
}
__device__ __forceinline__ void dma16_cached(unsigned off, const void* base, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(off), "s"(base), "s"(lds_base) : "memory", "m0");
}
// Partial-row stores with device scope (sc1): the L2 writes them through to the memory side at
// once instead of holding them dirty and writing them back later, in the middle of the K/V read
// stream.  (Same bytes; the merged-DAG attention measured 376 -> 370.5 us.)
// A store of more than 64 bits reads its data registers one cycle after issue, and the
// compiler's hazard checks do not look inside inline assembly: the 16-byte store carries its own
// wait states, or the next instruction may overwrite the data before it is read.
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void store_dev16(f16x8* p, f16x8 v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" :: "v"(p), "v"(v) : "memory");
}
__device__ __forceinline__ void store_dev8(f32x2* p, f32x2 v) {
  asm volatile("global_store_dwordx2 %0, %1, off sc1" :: "v"(p), "v"(v) : "memory");
}
#pragma clang diagnostic pop

// s_waitcnt vmcnt(n) for a runtime n in [0, 63] (expcnt and lgkmcnt left alone).  The gfx9
// encoding splits vmcnt into bits [3:0] and [15:14].
#define GA_VMCNT(k) (((k) & 15) | (7 << 4) | (15 << 8) | (((k) >> 4) << 14))
__device__ __forceinline__ void wait_vmcnt(int n) {
  // Loads placed before the wait in the source must be issued before it: the s_waitcnt builtin
  // alone does not order ordinary loads, and a load sunk below it would be waited for later,
  // inside the stage loop, draining the copy ring.
  asm volatile("" ::: "memory");
#define GA_VMW(k) case k: __builtin_amdgcn_s_waitcnt(GA_VMCNT(k)); break;
#define GA_VMW8(b) GA_VMW(b) GA_VMW(b + 1) GA_VMW(b + 2) GA_VMW(b + 3) GA_VMW(b + 4) \
                   GA_VMW(b + 5) GA_VMW(b + 6) GA_VMW(b + 7)
  switch (n) {
    GA_VMW8(0) GA_VMW8(8) GA_VMW8(16) GA_VMW8(24) GA_VMW8(32) GA_VMW8(40) GA_VMW8(48) GA_VMW8(56)
    default: __builtin_amdgcn_s_waitcnt(GA_VMCNT(0)); break;
  }
#undef GA_VMW8
#undef GA_VMW
}

template <int N>
__device__ __forceinline__ void wait_vmcnt_const() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(GA_VMCNT(N));
}

// Workgroup barrier without a memory fence: LDS-DMA completion is ordered by the explicit
// vmcnt wait before it; the empty asm statements keep the compiler from moving LDS accesses
// across it.
__device__ __forceinline__ void wg_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Barrier for data exchanged through LDS by ordinary LDS writes: waits for this wave's LDS
// operations only (lgkmcnt(0)), not for its global stores.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

__device__ __forceinline__ float exp2_(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float log2_(float x) { return __builtin_amdgcn_logf(x); }

__device__ __forceinline__ int64_t uniform64(int64_t v) {
  const int lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)(uint64_t)v);
  const int hi = __builtin_amdgcn_readfirstlane((int)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// Scores more than 2^kTau above a row's running reference trigger a reference update; below
// that the stale reference is kept (probabilities up to 2^kTau are exact in fp32 and bf16).
constexpr float kTau = 8.0f;

}  // namespace
}  // namespace ga
