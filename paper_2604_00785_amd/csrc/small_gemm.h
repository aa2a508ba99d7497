// The streaming products (small_gemm.hip): the grouped products of a layer whose experts have few rows each.
#pragma once
#include "common.h"

// The forward products take the streaming kernels where a load of any skew leaves few 16-row tiles per expert, so that its
// weights are not fetched again and again: at most STREAM_ROWS rows per expert, or no expert with more than STREAM_TOKENS
// rows (a token's experts are distinct, so no expert has more rows than there are tokens).  A rank's share may hold the
// large experts: where R_cap allows more rows and only the expected number is small, both kernels are launched and look
// at the number of rows on the device; the one that it is not for ends at once.
// Both forward products, tiled / streaming, in us, other weights in every pass (the tiled side picks its tile size; both sides' results
// have the same bits):
//                                             rows per expert  even load    zipf loads
//   d 2048, f 1024, 64 experts, 8 per token           2        128 / 121     73 / 69, 114 / 83
//                                                     4        138 / 135    117 / 95, 119 / 106
//                                                     6        139 / 137    122 / 112, 127 / 119
//                                                     8        140 / 138    131 / 155, 128 / 145
//   d 2048, f 1024, 64 experts, 1 per token           7        140 / 137     74 / 73, 81 / 92
//   d 2048, f 512, 128 experts, 8 per token           8        150 / 143    123 / 114
//   d 1088, f 576, 96 experts, 4 per token            4         76 / 66      44 / 36
//                                                     8         76 / 68      48 / 50
//   d 1024, f 512, 128 experts, 2 per token           8         83 / 78      45 / 43
//   d 1024, f 1024, 32 experts, 4 per token           8         50 / 41      46 / 40
//   d 512, f 256, 128 experts, 8 per token            8         26 / 25      27 / 22
// From 12 on they are even (76 / 76, 82 / 82), at 32 the tiles are ahead (147 / 155, 86 / 92; both with streaming tiles of up to 64 activation
// rows, which gave nothing below and were taken back).  The 64 experts of f 1024 are 2048 tiles, as many as the chip holds at a time: one expert
// with more than 16 rows adds a round of waves that each stream alone (64 tokens, one even load in four: 164 us).
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
