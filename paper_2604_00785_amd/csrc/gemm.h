// The grouped products as the library itself calls them.  `most` bounds the rows of one expert and, with R_cap, chooses the
// variant of the forward products; `rows` is the number of routed rows to expect: it chooses tile sizes and shapes launches,
// and no result depends on it.  `edges`, two numbers or null, is for tests: on entry the tile edge of either launch (128 or 256; 0: the
// rule decides, and only then the streaming kernels may be taken), on return the edge that it ran with (0: streamed).  Everything
// else as in moe_hotpath.h.
#pragma once
#include "common.h"

extern "C" int moe_gemm_fwd(const moe_bf16* xp, const int32_t* row_token, const float* row_weight, const int32_t* expert_offsets, const moe_bf16* Wg,
                 const moe_bf16* Wu, const moe_bf16* Wd, int E, int R_cap, long long rows, int most, int d, int f, moe_bf16* g,
                 moe_bf16* u, moe_bf16* h, moe_bf16* yp, void* stream, int* edges = nullptr);
int moe_gemm_fwd_gather(const moe_bf16* x, int T, const int32_t* row_token, const float* row_weight, const int32_t* expert_offsets,
                        const moe_bf16* Wg, const moe_bf16* Wu, const moe_bf16* Wd, int E, int R_cap, long long rows, int d,
                        int f, moe_bf16* g, moe_bf16* u, moe_bf16* h, moe_bf16* yp, void* stream);
extern "C" int moe_gemm_bwd(const moe_bf16* dyp, const moe_bf16* xp, int T, const int32_t* row_token, const moe_bf16* g, const moe_bf16* u,
                 const moe_bf16* h, const int32_t* expert_offsets, const moe_bf16* Wg, const moe_bf16* Wu,
                 const moe_bf16* Wd, int E, int R_cap, long long rows, int d, int f, moe_bf16* dxp, moe_bf16* dWg,
                 moe_bf16* dWu, moe_bf16* dWd, void* ws, size_t ws_bytes, void* stream, int* edges = nullptr);
// dgate null: the sums over the strips of the gate gradient's shares are left to moe_permute_bwd_dgate.
extern "C" int moe_gemm_bwd_folded(const moe_bf16* dout, const moe_bf16* x, int T, int k, const int32_t* row_token, const float* row_weight,
                        const int32_t* slot_row, const moe_bf16* g, const moe_bf16* u, const moe_bf16* hw,
                        const int32_t* expert_offsets, const moe_bf16* Wg, const moe_bf16* Wu, const moe_bf16* Wd, int E,
                        int R_cap, long long rows, int d, int f, moe_bf16* dxp, moe_bf16* dWg, moe_bf16* dWu,
                        moe_bf16* dWd, float* dgate, void* ws, size_t ws_bytes, void* stream, int* edges = nullptr);
// Those shares in the workspace of moe_gemm_bwd_folded: [R_cap][f / 64].
const float* moe_folded_part(const void* ws, int R_cap, int f);

// combine.hip.  moe_unpermute_combine (topk_w given), moe_unpermute_sum or moe_permute_bwd, where few slots have a local row.
int moe_combine_sparse(const moe_bf16* src, const int32_t* slot_row, const float* topk_w, int T, int k, int d, moe_bf16* out,
                       const char* name, void* stream);
// moe_unpermute_combine and moe_unpermute_combine_bwd in one pass over the rows of yp.
int moe_combine_both(const moe_bf16* dout, const moe_bf16* yp, const int32_t* slot_row, const float* topk_w, int T, int k, int d,
                     moe_bf16* out, moe_bf16* dyp, float* dgate, void* stream);
bool moe_permute_bwd_adds_dgate(int T, int k, int d);   // whether the call below is worth taking
// moe_permute_bwd, and dgate[t, i] = sum over c < strips of part[slot_row[t, i] * strips + c] (0 for a slot without a local row).
int moe_permute_bwd_dgate(const moe_bf16* dxp, const int32_t* slot_row, int T, int k, int d, moe_bf16* dx, const float* part,
                          int strips, float* dgate, void* stream);
