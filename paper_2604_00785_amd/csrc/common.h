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

// Reduction of v by op over a group of G lanes, in every lane of the group.  Partners inside a row of 16 lanes come through DPP lane
// permutations (neighbour, other pair of the quad, then the mirrored lane of the 8- and 16-lane halves: by then all lanes of the
// smaller unit agree, so the mirror is as good as the XOR partner), beyond a row through the exchange of rows or halves.
template <int CTRL> __device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, 0xF, 0xF, false));
}
template <int G, typename Op> __device__ __forceinline__ uint32_t group_reduce(uint32_t v, Op op) {
  if constexpr (G >= 2) v = op(v, dpp_u32<0xB1>(v));     // quad_perm [1,0,3,2]
  if constexpr (G >= 4) v = op(v, dpp_u32<0x4E>(v));     // quad_perm [2,3,0,1]
  if constexpr (G >= 8) v = op(v, dpp_u32<0x141>(v));    // row_half_mirror
  if constexpr (G >= 16) v = op(v, dpp_u32<0x140>(v));   // row_mirror
  if constexpr (G >= 32) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = op(r[0], r[1]);
  }
  if constexpr (G >= 64) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    v = op(r[0], r[1]);
  }
  return v;
}
template <int G> __device__ __forceinline__ float group_sum(float v) {   // the sums of a butterfly with partners lane ^ 1, ^ 2, ^ 4, ..
  return __uint_as_float(group_reduce<G>(__float_as_uint(v), [](uint32_t a, uint32_t b) __attribute__((always_inline)) {
    return __float_as_uint(__uint_as_float(a) + __uint_as_float(b));
  }));
}
template <int G> __device__ __forceinline__ float group_max(float v) {
  return __uint_as_float(group_reduce<G>(__float_as_uint(v), [](uint32_t a, uint32_t b) __attribute__((always_inline)) {
    return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b)));
  }));
}

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
