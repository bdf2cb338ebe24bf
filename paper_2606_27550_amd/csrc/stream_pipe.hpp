// Device helpers of the LM-head kernels that stream W through LDS rings:
// vocabulary slicing, explicit load-count waits, direct global->LDS copies
// and a fence-free workgroup barrier.
#pragma once

#include "common.hpp"

namespace entmtp {

// First vocabulary row of slice b of G (multiples of 4; V past the last).
__device__ __forceinline__ int slice_begin(int b, int G, int V) {
  if (b >= G) return V;
  return static_cast<int>((static_cast<long long>(V) * b / G) & ~3ll);
}

// s_waitcnt vmcnt(N) lgkmcnt(0) (gfx9 encoding; expcnt not waited on): this
// wave's direct-to-LDS loads older than the last N have landed and its own
// LDS reads are complete.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (0 << 8));
}

// s_waitcnt lgkmcnt(N) alone (vmcnt and expcnt left at their maxima).
template <int N>
__device__ __forceinline__ void wait_lds_but() {
  static_assert(N >= 0 && N < 16, "lgkmcnt range");
  __builtin_amdgcn_s_waitcnt(0xC07F | (N << 8));
}
__device__ __forceinline__ void wait_lds() { wait_lds_but<0>(); }

// One direct global->LDS copy of 16 bytes per lane: lane l's bytes land at
// lds + 16 * l (lds is wave-uniform).  Kept in a device-only function: in a
// kernel's (host+device) lambda this gfx950 builtin would keep the compiler
// from emitting the kernel's host launch stub.
__device__ __forceinline__ void lds_dma16(const void* src, void* lds) {
  __builtin_amdgcn_global_load_lds(src, lds, 16, 0, 0);
}

// The same copy through a buffer descriptor (lane l from byte voff(l) + soff of
// the buffer; lanes whose voff lies past its end receive zeros, and a caller
// keeps voff + soff below it for the others).  global_load_lds counts as a flat access, beside which the
// compiler makes every wait for an ordinary load a full drain; beside buffer
// copies its counted waits stay exact, and the address is one 32-bit offset.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t dma_buffer(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}
__device__ __forceinline__ void buf_dma16_at(__amdgpu_buffer_rsrc_t buf, uint32_t voff, int soff, void* lds) {
  typedef __attribute__((address_space(3))) void lds_void;
  __builtin_amdgcn_raw_ptr_buffer_load_lds(buf, (lds_void*)lds, 16, voff, soff, 0, 0);
}
__device__ __forceinline__ void buf_dma16(__amdgpu_buffer_rsrc_t buf, uint32_t voff, void* lds) {
  buf_dma16_at(buf, voff, 0, lds);
}

// Four bytes at byte voff of the buffer (zero past its end).  The range check
// is relied on for the per-lane offset alone: the scalar offset, which it need
// not cover, stays zero.
__device__ __forceinline__ float buf_load(__amdgpu_buffer_rsrc_t buf, uint32_t voff) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(buf, static_cast<int>(voff), 0, 0));
}

// Workgroup barrier without a memory-model fence.  __syncthreads() would add
// a release fence, which waits for every outstanding load (the LDS-DMA
// stages count as LDS writes) and so drains the pipeline; here the waits are
// explicit (wait_vmcnt) and the empty asm statements only stop the compiler
// from moving LDS accesses across the barrier.
__device__ __forceinline__ void stage_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

}  // namespace entmtp
