// Loads from global memory straight into LDS, issued and awaited by hand (the compiler does not know of them).
#pragma once
#include "common.h"

#define LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

// 16 bytes per lane: lane l lands at M0 + OFF + 16 l, and reads global address (scalar base) + (32-bit lane offset) + OFF.
__device__ __forceinline__ void set_m0_rt(uint32_t lds_addr) { asm volatile("s_mov_b32 m0, %0" :: "s"(lds_addr) : "memory"); }
template <int OFF> __device__ __forceinline__ void dma16_imm(uint32_t voff, const char* sbase) {
  asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" :: "v"(voff), "s"(sbase), "n"(OFF) : "memory");
}
// A scalar base that the compiler may just have brought back from a vector register (it keeps what it has no scalar registers for
// there): five wait states lie between that and a load that uses it, which the compiler sees to for its own loads only.  Here the scalar
// unit writes the base once more, in place, and no wait is needed behind that.  It stands in front of every group of loads above.
// (Five wait states in front of each load instead: 2-4 % of a large training step.)
template <typename T> __device__ __forceinline__ void settle(T*& sbase) { asm volatile("s_mov_b64 %0, %0" : "+s"(sbase)::"memory"); }
template <int N> __device__ __forceinline__ void lds_wait() { asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory"); }
template <int N> __device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
