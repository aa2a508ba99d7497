// The selection of one token, which the routing kernels (route.hip) and the first kernel of a decoding step (small_gemm.hip) share.
#pragma once
#include "perm_common.h"

__device__ __forceinline__ uint32_t ordered_bits(float v) {
  v += 0.0f;  // -0.0 -> +0.0 so the two zeros tie
  uint32_t u = __float_as_uint(v);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float from_ordered_bits(uint32_t u) {
  return __uint_as_float((u & 0x80000000u) ? u & 0x7FFFFFFFu : ~u);
}

// Selection and gates of one token by a group of G lanes (gl: lane inside the group): val[j] is the logit of expert
// gl + j G.  Winner i ends up in lane i % G, slot i / G: my_idx its expert, my_w its gate.
template <int G, int VPL>
__device__ __forceinline__ void route_token(const float (&val)[VPL], int gl, int E, int k, int renormalize, int (&my_idx)[VPL],
                                            float (&my_w)[VPL]) {
  const auto larger = [](uint32_t a, uint32_t b) __attribute__((always_inline)) { return a > b ? a : b; };
  const auto smaller = [](uint32_t a, uint32_t b) __attribute__((always_inline)) { return a < b ? a : b; };
  uint32_t key[VPL];
#pragma unroll
  for (int j = 0; j < VPL; ++j) {
    // 0 is for padding and retired keys; the lowest bit pattern, a negative NaN, goes one up
    key[j] = gl + j * G < E ? larger(ordered_bits(val[j]), 1u) : 0u;
  }
  float my_val[VPL];
#pragma unroll
  for (int j = 0; j < VPL; ++j) { my_idx[j] = 0; my_val[j] = 0.f; }
  // full-softmax denominator pieces need the row maximum, which is winner 0
  float row_max = 0.f;
  for (int i = 0; i < k; ++i) {
    uint32_t best = key[0];
#pragma unroll
    for (int j = 1; j < VPL; ++j) best = larger(best, key[j]);
    best = group_reduce<G>(best, larger);
    uint32_t id = 0xFFFFFFFFu;            // the lane's lowest expert with that key
#pragma unroll
    for (int j = VPL - 1; j >= 0; --j) id = key[j] == best ? static_cast<uint32_t>(gl + j * G) : id;
    const int e = static_cast<int>(group_reduce<G>(id, smaller));
#pragma unroll
    for (int j = 0; j < VPL; ++j) key[j] = gl + j * G == e ? 0u : key[j];
    const float v = from_ordered_bits(best);
    if (i == 0) row_max = v;
    if (k <= G) {
      if (gl == i) { my_idx[0] = e; my_val[0] = v; }
    } else if (gl == i % G) {
#pragma unroll
      for (int j = 0; j < VPL; ++j)
        if (j == i / G) { my_idx[j] = e; my_val[j] = v; }
    }
  }
  // denominator
  float part = 0.f;
  if (renormalize) {
#pragma unroll
    for (int j = 0; j < VPL; ++j)
      if (gl + j * G < k) part += expf(my_val[j] - row_max);
  } else {
#pragma unroll
    for (int j = 0; j < VPL; ++j)
      if (gl + j * G < E) part += expf(val[j] - row_max);
  }
  part = group_sum<G>(part);
  const float inv = 1.0f / part;
#pragma unroll
  for (int j = 0; j < VPL; ++j) my_w[j] = expf(my_val[j] - row_max) * inv;
}
