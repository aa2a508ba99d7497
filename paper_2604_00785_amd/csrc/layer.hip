// The whole layer in one call: what a program would otherwise enqueue through five to twelve calls of the C ABI.
// Host code only; it adds two things to the calls it makes: one argument check per call instead of one crossing of
// the language boundary per stage, and what the grouped products by themselves do not know: the number of experts of the
// whole layer, from which the expected number of local rows follows, and of tokens, which no expert's rows exceed.
#include "gemm.h"
#include "perm_common.h"
#include "small_gemm.h"

namespace {
bool overlap(const void* a, size_t a_bytes, const void* b, size_t b_bytes) {
  const uintptr_t p = reinterpret_cast<uintptr_t>(a), q = reinterpret_cast<uintptr_t>(b);
  return p < q + b_bytes && q < p + a_bytes;
}
// Whether the combine and its backward may be one kernel: not where the forward pass writes what the backward reads (the gradient of
// half the squared output is the output itself) or writes again, and not where the backward will be refused and the forward pass
// is to be complete nevertheless.
bool combine_in_one(const moe_layer* L) {
  for (const void* p : {static_cast<const void*>(L->dout), static_cast<const void*>(L->dyp), static_cast<const void*>(L->dgate)})
    if (!p || !moe_aligned16(p)) return false;
  const size_t row = static_cast<size_t>(L->d) * sizeof(moe_bf16), out = L->T * row;
  return !overlap(L->out, out, L->dout, out) && !overlap(L->out, out, L->dyp, out * L->k) &&
         !overlap(L->out, out, L->dgate, static_cast<size_t>(L->T) * L->k * sizeof(float));
}
// Whether the forward pass is one that kernels for several of its stages may take: a small call, rows gathered, that none of the stages
// would refuse.
bool few_gathered(const moe_layer* L) {
  if (L->path == MOE_LAYER_PLAIN || L->T > MOE_JOIN_TOKENS) return false;
  if (moe_check_permute_args(nullptr, L->topk_idx, L->T, L->d, L->E, L->k, L->e_begin, L->e_count, L->expert_offsets, L->row_token,
                             L->slot_row, nullptr, L->ws, L->ws_bytes) != MOE_OK) return false;
  if (L->d % 64 != 0 || L->f <= 0 || L->f % 64 != 0 || static_cast<unsigned long long>(L->T) * L->d * sizeof(moe_bf16) > 0xFFFFFFFFull - 65536)
    return false;
  const void* used[] = {L->logits, L->topk_w, L->x, L->Wg, L->Wu, L->Wd, L->g, L->u, L->h, L->yp};
  if (L->path == MOE_LAYER_FOLD && (!L->row_weight || !moe_aligned16(L->row_weight))) return false;
  for (const void* p : used) if (!p || !moe_aligned16(p)) return false;
  return true;
}
// Routing with gate_up: worth it, and no output of one lies where another workgroup still reads for the other, or over the other's outputs
// (the stages by themselves have read their inputs when the next one writes, and the later one's results stay).
bool route_and_gate_up_in_one(const moe_layer* L) {
  if (!moe_route_gate_up_fits(L->T, L->E, L->k, L->e_count, L->f)) return false;
  const size_t pairs = static_cast<size_t>(L->T) * L->k, rows = pairs * L->f * sizeof(moe_bf16);
  const size_t weights = sizeof(moe_bf16) * L->e_count * L->f * L->d;
  struct Range { const void* p; size_t bytes; };
  const Range routed[] = {{L->topk_idx, 4 * pairs}, {L->topk_w, 4 * pairs}, {L->row_token, 4 * pairs}, {L->slot_row, 4 * pairs},
                          {L->path == MOE_LAYER_FOLD ? L->row_weight : L->topk_w, 4 * pairs},
                          {L->expert_offsets, sizeof(int32_t) * (L->e_count + 1)}};
  const Range logits = {L->logits, sizeof(float) * L->T * L->E}, products[] = {{L->g, rows}, {L->u, rows}, {L->h, rows}};
  const Range read[] = {logits, {L->x, sizeof(moe_bf16) * L->T * L->d}, {L->Wg, weights}, {L->Wu, weights}};
  const auto meet = [](const Range& a, const Range& b) { return overlap(a.p, a.bytes, b.p, b.bytes); };
  for (const Range& o : routed) {
    for (const Range& q : products) if (meet(o, q)) return false;
    for (const Range& q : read) if (meet(o, q)) return false;
  }
  for (const Range& o : products) if (meet(o, logits)) return false;
  return true;
}
// down with the combine: worth it, and `out` lies nowhere that another workgroup still reads.
bool down_and_combine_in_one(const moe_layer* L, long long rows) {
  if (!moe_down_combine_fits(L->T, L->k, L->d, L->f, rows) || !L->out || !moe_aligned16(L->out)) return false;
  const size_t pairs = static_cast<size_t>(L->T) * L->k, out = sizeof(moe_bf16) * L->T * L->d;
  return !overlap(L->out, out, L->h, pairs * L->f * sizeof(moe_bf16)) && !overlap(L->out, out, L->yp, pairs * L->d * sizeof(moe_bf16)) &&
         !overlap(L->out, out, L->Wd, sizeof(moe_bf16) * L->e_count * L->d * L->f) && !overlap(L->out, out, L->slot_row, 4 * pairs) &&
         !overlap(L->out, out, L->expert_offsets, sizeof(int32_t) * (L->e_count + 1)) && !overlap(L->out, out, L->topk_w, 4 * pairs);
}
}  // namespace

extern "C" int moe_layer_run(const moe_layer* L, int what, void* stream) {
  if (!L || (what & ~(MOE_LAYER_ROUTER | MOE_LAYER_FWD | MOE_LAYER_BWD | MOE_LAYER_ROUTER_BWD))) return MOE_ERR_INVALID;
  if (L->path < MOE_LAYER_PLAIN || L->path > MOE_LAYER_FOLD) return MOE_ERR_INVALID;
  if (L->T <= 0 || L->k <= 0 || L->E <= 0 || L->e_count <= 0 || static_cast<long long>(L->T) * L->k > 0x7FFFFFFFll / 2)
    return MOE_ERR_INVALID;
  const int T = L->T, d = L->d, E = L->E, k = L->k, f = L->f, nl = L->e_count, R_cap = T * k;
  const long long rows = (static_cast<long long>(R_cap) * nl + E - 1) / E;
  const bool fold = L->path == MOE_LAYER_FOLD, plain = L->path == MOE_LAYER_PLAIN;
  const bool sparse = 2ll * nl <= E;   // few of a token's slots have a local row
  const bool both = !fold && (what & MOE_LAYER_FWD) && (what & MOE_LAYER_BWD) && combine_in_one(L);
  int rc = MOE_OK;
  if (what & MOE_LAYER_ROUTER) {
    if ((rc = moe_router_fwd(L->x, L->Wr, T, d, E, L->logits, stream)) != MOE_OK) return rc;
  }
  if (what & MOE_LAYER_FWD) {
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool few = few_gathered(L), front = few && route_and_gate_up_in_one(L);
    const bool back = few && !both && down_and_combine_in_one(L, rows);
    if (front) {
      rc = moe_route_gate_up(L, rows, s);
    } else {
      rc = moe_route_permute(L->logits, plain ? L->x : nullptr, T, d, E, k, L->renormalize, L->e_begin, nl, L->topk_idx, L->topk_w,
                             L->expert_offsets, L->row_token, L->slot_row, fold ? L->row_weight : nullptr,
                             plain ? L->xp : nullptr, L->ws, L->ws_bytes, stream);
    }
    if (rc != MOE_OK) return rc;
    if (fold && (!L->row_weight || !moe_aligned16(L->row_weight))) return MOE_ERR_INVALID;
    StreamFwdArgs p{}, q{};
    p.offsets = q.offsets = L->expert_offsets; p.E = q.E = nl; p.max_rows = q.max_rows = R_cap;
    if (back && !front) {
      p.A = L->x; p.row_token = L->row_token; p.row_weight = fold ? L->row_weight : nullptr;
      p.B0 = L->Wg; p.B1 = L->Wu; p.O0 = L->g; p.O1 = L->u; p.O2 = L->h; p.K = d; p.N = f;
      rc = moe_stream_gate_up(p, rows, s);
      if (rc != MOE_OK) return rc;
    }
    if (back) {
      rc = moe_down_combine(L, s);
    } else if (front) {
      q.A = L->h; q.B0 = L->Wd; q.O0 = L->yp; q.K = f; q.N = d;
      rc = moe_stream_down(q, rows, s);
    } else if (plain) {
      rc = moe_gemm_fwd(L->xp, nullptr, nullptr, L->expert_offsets, L->Wg, L->Wu, L->Wd, nl, R_cap, rows, T, d, f, L->g, L->u, L->h,
                        L->yp, stream);
    } else {
      rc = moe_gemm_fwd_gather(L->x, T, L->row_token, fold ? L->row_weight : nullptr, L->expert_offsets, L->Wg, L->Wu, L->Wd, nl,
                               R_cap, rows, d, f, L->g, L->u, L->h, L->yp, stream);
    }
    if (rc != MOE_OK) return rc;
    // with the backward in the same call the rows of yp are read once, for both
    if (!fold && !L->topk_w) return MOE_ERR_INVALID;
    if (back) rc = MOE_OK;
    else if (both) rc = moe_combine_both(L->dout, L->yp, L->slot_row, L->topk_w, T, k, d, L->out, L->dyp, L->dgate, stream);
    else if (sparse) rc = moe_combine_sparse(L->yp, L->slot_row, fold ? nullptr : L->topk_w, T, k, d, L->out, "combine", stream);
    else if (fold) rc = moe_unpermute_sum(L->yp, L->slot_row, T, k, d, L->out, stream);
    else rc = moe_unpermute_combine(L->yp, L->slot_row, L->topk_w, T, k, d, L->out, stream);
    if (rc != MOE_OK) return rc;
  }
  if (what & MOE_LAYER_BWD) {
    if (!plain && !L->row_token) return MOE_ERR_INVALID;   // without it moe_gemm_bwd would take x for T * k grouped rows
    if (!L->dgate || !moe_aligned16(L->dgate)) return MOE_ERR_INVALID;
    const bool adds_dgate = fold && moe_permute_bwd_adds_dgate(T, k, d);
    if (fold) {
      rc = moe_gemm_bwd_folded(L->dout, L->x, T, k, L->row_token, L->row_weight, L->slot_row, L->g, L->u, L->h,
                               L->expert_offsets, L->Wg, L->Wu, L->Wd, nl, R_cap, rows, d, f, L->dxp, L->dWg, L->dWu, L->dWd,
                               adds_dgate ? nullptr : L->dgate, L->ws, L->ws_bytes, stream);
    } else {
      if (!both) rc = moe_unpermute_combine_bwd(L->dout, L->yp, L->slot_row, L->topk_w, T, k, d, L->dyp, L->dgate, stream);
      if (rc != MOE_OK) return rc;
      rc = moe_gemm_bwd(L->dyp, plain ? L->xp : L->x, T, plain ? nullptr : L->row_token, L->g, L->u, L->h, L->expert_offsets,
                        L->Wg, L->Wu, L->Wd, nl, R_cap, rows, d, f, L->dxp, L->dWg, L->dWu, L->dWd, L->ws, L->ws_bytes, stream);
    }
    if (rc != MOE_OK) return rc;
    rc = adds_dgate ? moe_permute_bwd_dgate(L->dxp, L->slot_row, T, k, d, L->dx, moe_folded_part(L->ws, R_cap, f), f / 64, L->dgate, stream)
         : sparse   ? moe_combine_sparse(L->dxp, L->slot_row, nullptr, T, k, d, L->dx, "permute_bwd", stream)
                    : moe_permute_bwd(L->dxp, L->slot_row, T, k, d, L->dx, stream);
    if (rc != MOE_OK) return rc;
  }
  if (what & MOE_LAYER_ROUTER_BWD) {
    if ((rc = moe_route_bwd(L->logits, L->topk_idx, L->dgate, T, E, k, L->renormalize, L->dlogits, stream)) != MOE_OK) return rc;
    rc = moe_router_bwd(L->x, L->Wr, L->dlogits, T, d, E, L->dx, L->dWr, L->ws, L->ws_bytes, stream);
  }
  return rc;
}
