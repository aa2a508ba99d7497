// Shared device/host helpers of the MoE hot-path library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "moe_hotpath.h"

#define MOE_WAVE 64

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

// fp32 -> bf16 bits, round to nearest even (hardware conversion on gfx950).
__device__ __forceinline__ uint16_t f32_to_bf16(float v) {
  __bf16 b = static_cast<__bf16>(v);
  return __builtin_bit_cast(uint16_t, b);
}
__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}
// two packed bf16 (low half = element 0) <-> two floats
__device__ __forceinline__ float bf16lo(uint32_t p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float bf16hi(uint32_t p) { return __uint_as_float(p & 0xFFFF0000u); }
// one v_cvt_pk_bf16_f32 (round to nearest even, as the scalar conversion)
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// Inclusive prefix sum over the 64 lanes of a wave, all of them active.  Six vector instructions that take their partner
// through the lane permutation of the operand (rows of 16 lanes first, then lane 15 of a row for the row behind it, then lane 31
// for the upper half), some 50 cycles; six ds_bpermute, each waiting for the one before, were some 800, and the tile lookup
// of a grouped product scans up to eight times before its first load.
__device__ __forceinline__ int wave_incl_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);   // row_shr:1 (nothing comes in from outside the row)
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);   // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2 and 3
  return v;
}
// The value of a lane whose number is the same in the whole wave.
__device__ __forceinline__ int wave_lane(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }

static inline bool moe_aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// ---- launch bookkeeping (prof.hip) ----------------------------------------
// When profiling is on, brackets the launch with two events on `stream`.
struct MoeLaunchScope {
  MoeLaunchScope(const char* name, hipStream_t stream);
  ~MoeLaunchScope();
  int slot;
  hipStream_t stream;
};
int moe_check_launch();  // MOE_OK or MOE_ERR_LAUNCH from hipGetLastError()

#define MOE_LAUNCH(name, kernel, grid, block, shmem, stream, ...)              \
  do {                                                                         \
    MoeLaunchScope _scope(name, stream);                                       \
    hipLaunchKernelGGL(kernel, grid, block, shmem, stream, __VA_ARGS__);       \
  } while (0)
