// The streaming products (small_gemm.hip): the grouped products of a layer whose experts have few rows each.
#pragma once
#include "common.h"

// Rows per expert, on average, up to which the forward products take the streaming kernels.  Measured at d 2048, f 1024,
// 64 experts: 12 rows 114 + 63 us against 137 + 64 us in the tiled kernel, 19 rows 119 + 66 against 116-128 + 64, 25 rows
// 126 + 71 against 118-139 + 64.
constexpr int STREAM_ROWS = 20;
// One grouped product out[r] = act[r] . W[e]^T (weights [N][K], K contiguous), or the pair gate/up with the
// SwiGLU epilogue.  E, K, N as in GemmArgs; row_token / row_weight may be null.
struct StreamFwdArgs {
  const uint16_t* A;            // activations, [R_cap][K], or [T][K] with row_token
  const int32_t* row_token;
  const float* row_weight;
  const int32_t* offsets;
  const uint16_t* B0;           // Wg | Wd
  const uint16_t* B1;           // Wu
  uint16_t* O0;                 // g | yp
  uint16_t* O1;                 // u
  uint16_t* O2;                 // h
  int E, K, N;
};

// R_cap: row capacity, rows: rows to expect (both only shape the launch)
int moe_stream_gate_up(const StreamFwdArgs& a, int R_cap, long long rows, hipStream_t s);
int moe_stream_down(const StreamFwdArgs& a, int R_cap, long long rows, hipStream_t s);
