// The grouped products as the library itself calls them.  `most` bounds the rows of one expert and, with R_cap, chooses the
// variant of the forward products; `rows` is the number of routed rows to expect: it chooses tile sizes and shapes launches,
// and no result depends on it.  Everything else as in moe_hotpath.h.
#pragma once
#include "common.h"

int moe_gemm_fwd(const moe_bf16* xp, const int32_t* row_token, const float* row_weight, const int32_t* expert_offsets, const moe_bf16* Wg,
                 const moe_bf16* Wu, const moe_bf16* Wd, int E, int R_cap, long long rows, int most, int d, int f, moe_bf16* g,
                 moe_bf16* u, moe_bf16* h, moe_bf16* yp, void* stream);
int moe_gemm_fwd_gather(const moe_bf16* x, int T, const int32_t* row_token, const float* row_weight, const int32_t* expert_offsets,
                        const moe_bf16* Wg, const moe_bf16* Wu, const moe_bf16* Wd, int E, int R_cap, long long rows, int d,
                        int f, moe_bf16* g, moe_bf16* u, moe_bf16* h, moe_bf16* yp, void* stream);
int moe_gemm_bwd(const moe_bf16* dyp, const moe_bf16* xp, int T, const int32_t* row_token, const moe_bf16* g, const moe_bf16* u,
                 const moe_bf16* h, const int32_t* expert_offsets, const moe_bf16* Wg, const moe_bf16* Wu,
                 const moe_bf16* Wd, int E, int R_cap, long long rows, int d, int f, moe_bf16* dxp, moe_bf16* dWg,
                 moe_bf16* dWu, moe_bf16* dWd, void* ws, size_t ws_bytes, void* stream);
int moe_gemm_bwd_folded(const moe_bf16* dout, const moe_bf16* x, int T, int k, const int32_t* row_token, const float* row_weight,
                        const int32_t* slot_row, const moe_bf16* g, const moe_bf16* u, const moe_bf16* hw,
                        const int32_t* expert_offsets, const moe_bf16* Wg, const moe_bf16* Wu, const moe_bf16* Wd, int E,
                        int R_cap, long long rows, int d, int f, moe_bf16* dxp, moe_bf16* dWg, moe_bf16* dWu,
                        moe_bf16* dWd, float* dgate, void* ws, size_t ws_bytes, void* stream);
