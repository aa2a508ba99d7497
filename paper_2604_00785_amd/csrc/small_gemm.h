// The streaming products (small_gemm.hip): the grouped products of a layer whose experts have few rows each.
#pragma once
#include "common.h"

// The forward products take the streaming kernels where a load of any skew leaves few 16-row tiles per expert, so that its
// weights are not fetched again and again: at most STREAM_ROWS rows per expert, or no expert with more than STREAM_TOKENS
// rows (a token's experts are distinct, so no expert has more rows than there are tokens).  A rank's share may hold the
// large experts: where R_cap allows more rows and only the expected number is small, both kernels are launched and look
// at the number of rows on the device; the one that it is not for ends at once.
// Forward pass in us, tiled / streaming, other weights in every pass (the tiled side picks its tile size; both sides' results
// have the same bits):
//                                             rows per expert  even load    zipf loads
//   d 2048, f 1024, 64 experts, 8 per token           2        159 / 150    112 / 99, 108 / 93
//                                                     4        171 / 161    143 / 125, 143 / 120
//                                                     6        173 / 164    149 / 135, 150 / 135
//                                                     8        174 / 166    152 / 142, 153 / 142
//                                                    12        176 / 168    159 / 170, 163 / 172
//                                                    16        178 / 184    169 / 183, 173 / 188
//   d 2048, f 1024, 64 experts, 1 per token           7        175 / 167     92 / 95, 93 / 96
//   d 2048, f 512, 128 experts, 8 per token           8        186 / 177    153 / 139, 156 / 139
//   d 1088, f 576, 96 experts, 4 per token            4         87 / 84      55 / 50, 54 / 46
//                                                     8         89 / 88      69 / 69, 64 / 70
//   d 1024, f 512, 128 experts, 2 per token           8         95 / 94      54 / 57, 55 / 59
//   d 1024, f 1024, 32 experts, 4 per token           8         58 / 47      54 / 47, 54 / 47
//   d 512, f 256, 128 experts, 8 per token            8         46 / 44      45 / 41, 45 / 40
//   d 2048, f 1024, 240 experts, 8 per token          4        554 / 513    239 / 244, 241 / 243
//                                                     8        576 / 544    292 / 325, 295 / 329
// On 10000 calls of 33 to 1024 tokens with 0.7 to 28 rows per expert streaming is 10 % faster on average with an even load at every
// number of rows up to 10, and 30 % (one row) to 9 % (8 rows) with a zipf load.  Where all experts together are 3000 tiles or more, it is 6 % ahead
// with an even and 6 % behind with a zipf load at 6 to 8 rows, and nothing known on the host tells them apart.  With fewer than 1600 tiles it stays ahead
// on average up to 16 rows, with fewer than 512 up to 28; the line is not moved there.
constexpr int STREAM_ROWS = 8, STREAM_TOKENS = 32;

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
  int max_rows;                 // nothing is done where there are more rows
};

// rows: rows to expect (only shapes the launch, not the results)
int moe_stream_gate_up(const StreamFwdArgs& a, long long rows, hipStream_t s);
int moe_stream_down(const StreamFwdArgs& a, long long rows, hipStream_t s);

// A few tokens' forward pass, rows gathered: Stages 1 to 3 with gate_up in one kernel, down with the combine in another, each where it is
// faster than its parts (the rules stand at the kernels).  The caller has checked the arguments; at MOE_JOIN_TOKENS and below the products
// stream.
constexpr int MOE_JOIN_TOKENS = 8;
static_assert(MOE_JOIN_TOKENS <= STREAM_TOKENS);
bool moe_route_gate_up_fits(int T, int E, int k, int e_count, int f);
int moe_route_gate_up(const moe_layer* L, long long rows, hipStream_t s);   // rows: to expect, here and below
bool moe_down_combine_fits(int T, int k, int d, int f, long long rows);
int moe_down_combine(const moe_layer* L, hipStream_t s);
