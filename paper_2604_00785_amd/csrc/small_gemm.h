// The streaming products (small_gemm.hip): the grouped products of a layer whose experts have few rows each.
#pragma once
#include "common.h"

// The forward products take the streaming kernels where a load of any skew leaves few 16-row tiles per expert, so that its
// weights are not fetched again and again: at most STREAM_ROWS rows per expert, or no expert with more than STREAM_TOKENS
// rows (a token's experts are distinct, so no expert has more rows than there are tokens).  A rank's share may hold the
// large experts: where R_cap allows more rows and only the expected number is small, both kernels are launched and look
// at the number of rows on the device; the one that it is not for ends at once.
// Forward pass, tiled / streaming, in us, other weights in every pass (the tiled side picks its tile size; both sides' results
// have the same bits):
//                                             rows per expert  even load    zipf load
//   d 2048, f 1024, 64 experts, 8 per token           1/8         59 /  33     58 /  32
//                                                     4          173 / 173    141 / 130
//                                                     6          189 / 186    156 / 152
//                                                     8          179 / 179    160 / 170
//                                                    10          160 / 179    150 / 174
//   d 1088, f 576, 96 experts, 4 per token            3           88 /  81     54 /  43
//                                                     8           94 /  90     71 /  78
//                                                    12           95 /  96     84 /  92
//   d 512, f 256, 128 experts, 8 per token            2           34 /  34     32 /  26
//                                                     8           47 /  49     45 /  43
//                                                    12           42 /  47     42 /  44
//   d 1024, f 512, 128 experts, 2 per token           6           97 /  96     59 /  59
//   d 2048, f 1024, 64 experts, 1 per token           6          160 / 164     93 / 108
//   d 2048, f 1024, the 20 of 240 experts that zipf makes the largest, 8 per token: 32 tokens 67 / 52 and 80 / 77
// At 6 to 8 rows per expert the order changes with load and shape (tiles up to 16 %, streaming up to 6 % ahead), by nothing known
// on the host; from 10 on the tiles are ahead.
constexpr int STREAM_ROWS = 8, STREAM_TOKENS = 32;

// The 64-deep step with which expert e begins the reduction of a forward product; it goes on to the end and then takes the steps in front
// of it.  Where a weight row is a multiple of 4096 bytes, workgroups that run in step would otherwise all read the same 128 bytes of
// their rows' 4096 at a time, and those lie in a fraction of the memory channels.  By the expert alone, so that every kernel and
// tile size sums a row in the same order.  Weights read by gate_up (E 64), TB/s, from the beginning -> rotated: K 2048, 64 rows per expert
// 4.25 -> 5.33, 192 rows 3.75 -> 4.49; K 4096 4.32 -> 5.82 and 3.89 -> 4.98; from 264 rows on, where the matrix pipe bounds, no
// difference.  With other K nothing is to be gained (1024, 1536, 1792, 2304, 3072, 3584: 4.8 to 5.3 either way), nor in the products
// with weights stored [K][N], whose steps read whole rows.
__device__ __forceinline__ int first_k_step(int e, int K) { return K % 2048 == 0 ? e * 11 % 32 : 0; }

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

// A layer's forward pass with at most 64 (token, slot) pairs, rows gathered: Stages 1 to 3 with gate_up in one kernel, and, for a few
// tokens, down with the combine in another.  The caller has checked the arguments.
bool moe_small_layer_fits(int T, int E, int k);
int moe_route_gate_up(const moe_layer* L, long long rows, hipStream_t s);   // rows: to expect
bool moe_down_combine_fits(int T, int k);
int moe_down_combine(const moe_layer* L, hipStream_t s);
