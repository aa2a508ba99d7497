// Stage 1 of Algorithm 1: Softmax over the experts, then TopK.
//
// A group of G lanes (G a power of two, 8..64) owns one token and keeps
// ceil(E/G) logits per lane in registers.  Selection runs on the logits (the
// softmax is monotone): each becomes a 32-bit key, the order-preserving image of
// the fp32 value.  k rounds pick the k winners: the maximum over the group, then
// the lowest expert id among the lanes' keys that equal it, which the owner
// retires; the value comes back out of the key.  Gates are exp(l - max)
// divided by the sum over all experts, or over the winners when renormalising.
//
// What bounds it is the vector ALU (large passes) and the chain of rounds (small ones): a round is some 50 instructions, all of them
// single ones whose partners come through lane permutations.  With 64-bit keys (value and id in one maximum) it was some 110, every
// compare and select doubled, and the value went through LDS.  Routing launch before -> now, us (between events),
// 8 winners: 24576 tokens of 240 experts 34.1 -> 28.1, 8192 of 64 10.7 -> 8.5, 501 of 64 9.8 -> 8.2, 48 of 64 in one workgroup 10.0 -> 9.1.
//
// When the index generation of Stages 2-3 follows in the same call, a workgroup routes a chunk of
// tokens (one or more passes of 256 / G tokens) and counts its winners per local expert straight from
// the registers that hold them: the [chunk][expert] table of the counting sort is then a by-product
// of the routing and the pairs need not be read back for it.
#include "route_token.h"

namespace {

// COUNT: also write hist[blockIdx.x][local expert] = winners of this workgroup's tokens per local expert.
template <int G, int VPL, bool COUNT>
__global__ __launch_bounds__(256) void route_kernel(const float* __restrict__ logits, int T, int E, int k,
                                                    int renormalize, int32_t* __restrict__ topk_idx,
                                                    float* __restrict__ topk_w, int passes, int e_begin, int e_count,
                                                    int nbits, int32_t* __restrict__ hist) {
  constexpr int GROUPS_PER_BLOCK = 256 / G;
  __shared__ int wcnt[COUNT ? PERM_WAVES : 1][COUNT ? MOE_MAX_EXPERTS : 1];   // per wave: winners per local expert
  const int tid = threadIdx.x;
  const int gl = tid % G;  // lane inside the group
  if constexpr (COUNT) {
    for (int e = tid; e < e_count; e += 256) {
#pragma unroll
      for (int v = 0; v < PERM_WAVES; ++v) wcnt[v][e] = 0;
    }
    __syncthreads();
  }

  auto load_row = [&](int pass, float (&val)[VPL]) {
    const int t = (blockIdx.x * passes + pass) * GROUPS_PER_BLOCK + tid / G;
    const int tt = t < T ? t : T - 1;  // idle groups shadow the last token and store nothing
#pragma unroll
    for (int j = 0; j < VPL; ++j) {
      const int e = gl + j * G;
      val[j] = e < E ? logits[static_cast<size_t>(tt) * E + e] : 0.f;
    }
  };
  float nxt[VPL];
  load_row(0, nxt);

  for (int pass = 0; pass < passes; ++pass) {
    const int t = (blockIdx.x * passes + pass) * GROUPS_PER_BLOCK + tid / G;
    const bool live = t < T;
    float val[VPL];
#pragma unroll
    for (int j = 0; j < VPL; ++j) val[j] = nxt[j];
    if (pass + 1 < passes) load_row(pass + 1, nxt);   // the next pass's logits arrive during this pass's selection
    int my_idx[VPL];
    float my_w[VPL];
    route_token<G, VPL>(val, gl, E, k, renormalize, my_idx, my_w);

#pragma unroll
    for (int j = 0; j < VPL; ++j) {
      const int i = gl + j * G;
      if (i < k) {
        if (live) {
          topk_idx[static_cast<size_t>(t) * k + i] = my_idx[j];
          topk_w[static_cast<size_t>(t) * k + i] = my_w[j];
        }
      }
    }
    if constexpr (COUNT) {
      // The winners are counted where they are: slot j of the wave's lanes is one batch of up to 64 pairs (lane gl
      // of a group holds winner gl + j G), counted with the ballots of the counting sort; the lowest lane of every
      // group of equal experts adds the group's size to the wave's own LDS row.
      int* cnt = wcnt[tid / MOE_WAVE];
      const int lane = tid % MOE_WAVE;
#pragma unroll
      for (int j = 0; j < VPL; ++j) {
        if (j * G < k) {   // uniform: some lane holds a winner in this slot
          int le = (live && gl + j * G < k) ? my_idx[j] - e_begin : -1;
          if (le < 0 || le >= e_count) le = -1;
          const uint64_t m = same_expert_mask(le, nbits);
          if (m != 0 && lane == __builtin_ctzll(m)) cnt[le] += __builtin_popcountll(m);
          __builtin_amdgcn_wave_barrier();
        }
      }
    }
  }

  if constexpr (COUNT) {
    __syncthreads();
    for (int e = tid; e < e_count; e += 256) {
      int s = 0;
#pragma unroll
      for (int v = 0; v < PERM_WAVES; ++v) s += wcnt[v][e];
      hist[static_cast<size_t>(blockIdx.x) * e_count + e] = s;
    }
  }
}

template <int G, int VPL>
void launch_route(const float* logits, int T, int E, int k, int renorm, int32_t* idx, float* w, hipStream_t s) {
  const int groups = 256 / G;
  dim3 grid((T + groups - 1) / groups), block(256);
  MOE_LAUNCH("route", (route_kernel<G, VPL, false>), grid, block, 0, s, logits, T, E, k, renorm, idx, w, 1, 0, 0, 0,
             static_cast<int32_t*>(nullptr));
}

// Tokens per workgroup: whole passes of 256 / G tokens; as few passes as keep the chunks at perm_max_chunks
// or fewer and the [chunk][expert] table inside the workspace the caller gave (a workspace of the minimum
// size holds one table row per 256 pairs, which can mean several passes when k is small).
template <int G, int VPL>
bool launch_route_count(const float* logits, int T, int E, int k, int renorm, int e_begin, int e_count, int nbits,
                        int32_t* idx, float* w, int32_t* hist, size_t hist_cells, int* chunk, int* nblocks, hipStream_t s) {
  const int groups = 256 / G;
  const long long rows_fit = static_cast<long long>(hist_cells / static_cast<size_t>(e_count));
  const long long max_chunks = rows_fit < perm_max_chunks(e_count) ? rows_fit : perm_max_chunks(e_count);
  if (max_chunks < 1) return false;
  const long long cap = groups * max_chunks;
  const int passes = static_cast<int>((T + cap - 1) / cap);
  if (static_cast<long long>(passes) * groups * k > 0x3FFFFFFF) return false;
  const int tokens = passes * groups;
  *chunk = tokens * k;
  *nblocks = (T + tokens - 1) / tokens;
  MOE_LAUNCH("route_count", (route_kernel<G, VPL, true>), dim3(*nblocks), dim3(256), 0, s, logits, T, E, k, renorm, idx, w,
             passes, e_begin, e_count, nbits, hist);
  return true;
}

// Stages 1-3 of a call with few tokens in ONE workgroup and launch: routes all tokens, keeps the pairs' local
// experts in LDS and sorts them there.  Wave w owns pairs 64 w .. 64 w + 63 (at most RS_PAIRS in all): it counts
// them per expert with the ballots of the counting sort, one thread per expert turns the waves' counts into first
// rows, and every pair finds its row as permute_place does.  Results are those of the two launches, bit for bit.
constexpr int RS_THREADS = 1024, RS_WAVES = RS_THREADS / MOE_WAVE;
template <int G, int VPL>
__global__ __launch_bounds__(RS_THREADS) void route_small_kernel(const float* __restrict__ logits, int T, int E, int k,
                                                                int renormalize, int e_begin, int e_count, int nbits,
                                                                int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
                                                                int32_t* __restrict__ expert_offsets,
                                                                int32_t* __restrict__ row_token, int32_t* __restrict__ slot_row,
                                                                float* __restrict__ row_weight) {
  constexpr int GROUPS = RS_THREADS / G;
  __shared__ int s_e[RS_PAIRS];
  __shared__ float s_w[RS_PAIRS];
  __shared__ int s_sum[MOE_MAX_EXPERTS / MOE_WAVE];
  extern __shared__ int s_cnt[];              // [used waves][e_count]
  const int tid = threadIdx.x, lane = tid % MOE_WAVE, w = tid / MOE_WAVE;
  const int n = T * k, waves = (n + MOE_WAVE - 1) / MOE_WAVE;
  const int gl = tid % G;
  for (int i = tid; i < waves * e_count; i += RS_THREADS) s_cnt[i] = 0;
  for (int t0 = 0; t0 < T; t0 += GROUPS) {
    const int t = t0 + tid / G;
    if (t0 + w * (MOE_WAVE / G) >= T) break;          // the whole wave is past the last token
    const int tt = t < T ? t : T - 1;
    float val[VPL];
#pragma unroll
    for (int j = 0; j < VPL; ++j) {
      const int e = gl + j * G;
      val[j] = e < E ? logits[static_cast<size_t>(tt) * E + e] : 0.f;
    }
    int my_idx[VPL];
    float my_w[VPL];
    route_token<G, VPL>(val, gl, E, k, renormalize, my_idx, my_w);
#pragma unroll
    for (int j = 0; j < VPL; ++j) {
      const int i = gl + j * G;
      if (i < k && t < T) {
        const int p = t * k + i;
        topk_idx[p] = my_idx[j];
        topk_w[p] = my_w[j];
        const int le = my_idx[j] - e_begin;
        s_e[p] = le < 0 || le >= e_count ? -1 : le;
        s_w[p] = my_w[j];
      }
    }
  }
  __syncthreads();
  // counts of the wave's 64 pairs per expert
  const int e = tid < n ? s_e[tid] : -1;
  const uint64_t m = w < waves ? same_expert_mask(e, nbits) : 0;
  if (m != 0 && lane == __builtin_ctzll(m)) s_cnt[w * e_count + e] = __builtin_popcountll(m);
  __syncthreads();
  // thread x < e_count: rows of expert x in front of each wave, and the scan over the experts
  int total = 0;
  if (tid < e_count) {
    for (int v = 0; v < waves; ++v) {
      const int c = s_cnt[v * e_count + tid];
      s_cnt[v * e_count + tid] = total;
      total += c;
    }
  }
  const int inc = wave_incl_scan(total);
  if (lane == MOE_WAVE - 1 && w < MOE_MAX_EXPERTS / MOE_WAVE) s_sum[w] = inc;
  __syncthreads();
  if (tid < e_count) {
    int base = 0;
    for (int v = 0; v < w; ++v) base += s_sum[v];
    const int first = base + inc - total;
    expert_offsets[tid] = first;
    if (tid == e_count - 1) expert_offsets[e_count] = first + total;
    for (int v = 0; v < waves; ++v) s_cnt[v * e_count + tid] += first;
  }
  __syncthreads();
  if (tid < n) {
    int row = -1;
    if (m != 0) {
      row = s_cnt[w * e_count + e] + __builtin_popcountll(m & lanemask_lt());
      row_token[row] = tid / k;
      if (row_weight != nullptr) row_weight[row] = s_w[tid];
    }
    slot_row[tid] = row;
  }
}

}  // namespace

bool moe_launch_route_count(const float* logits, int T, int E, int k, int renormalize, int e_begin, int e_count,
                            int nbits, int32_t* topk_idx, float* topk_w, int32_t* hist, size_t hist_cells, int* chunk,
                            int* nblocks, hipStream_t s) {
  if (E > MOE_MAX_EXPERTS) return false;
#define MOE_ROUTE_COUNT(G, VPL) \
  launch_route_count<G, VPL>(logits, T, E, k, renormalize, e_begin, e_count, nbits, topk_idx, topk_w, hist, hist_cells, chunk, \
                             nblocks, s)
  // eight logits per lane where the expert count allows: twice the tokens per pass of the plain launch, so
  // that one pass already fills a chunk at the usual shapes (a second pass would run after the first)
  if (E <= 8) return MOE_ROUTE_COUNT(8, 1);
  if (E <= 16) return MOE_ROUTE_COUNT(8, 2);
  if (E <= 32) return MOE_ROUTE_COUNT(8, 4);
  if (E <= 64) return MOE_ROUTE_COUNT(8, 8);
  if (E <= 128) return MOE_ROUTE_COUNT(16, 8);
  if (E <= 256) return MOE_ROUTE_COUNT(32, 8);
  return MOE_ROUTE_COUNT(64, 8);
#undef MOE_ROUTE_COUNT
}

bool moe_launch_route_small(const float* logits, int T, int E, int k, int renormalize, int e_begin, int e_count, int nbits,
                            int32_t* topk_idx, float* topk_w, int32_t* expert_offsets, int32_t* row_token,
                            int32_t* slot_row, float* row_weight, hipStream_t s) {
  if (E > MOE_MAX_EXPERTS || static_cast<long long>(T) * k > RS_PAIRS) return false;
  // the lane groups of the plain launch (same bits)
  const int G = E <= 64 ? 8 : E <= 128 ? 16 : E <= 256 ? 32 : 64;
  if (T > 2 * (RS_THREADS / G)) return false;
  const size_t lds = static_cast<size_t>((T * k + MOE_WAVE - 1) / MOE_WAVE) * e_count * sizeof(int);
#define MOE_ROUTE_SMALL(G, VPL)                                                                                            \
  MOE_LAUNCH("route_small", (route_small_kernel<G, VPL>), dim3(1), dim3(RS_THREADS), lds, s, logits, T, E, k, renormalize, \
             e_begin, e_count, nbits, topk_idx, topk_w, expert_offsets, row_token, slot_row, row_weight)
  if (E <= 8) MOE_ROUTE_SMALL(8, 1);
  else if (E <= 16) MOE_ROUTE_SMALL(8, 2);
  else if (E <= 32) MOE_ROUTE_SMALL(8, 4);
  else if (E <= 64) MOE_ROUTE_SMALL(8, 8);
  else if (E <= 128) MOE_ROUTE_SMALL(16, 8);
  else if (E <= 256) MOE_ROUTE_SMALL(32, 8);
  else MOE_ROUTE_SMALL(64, 8);
#undef MOE_ROUTE_SMALL
  return true;
}

extern "C" int moe_route(const float* logits, int T, int E, int k, int renormalize, int32_t* topk_idx,
                         float* topk_w, void* stream) {
  if (!logits || !topk_idx || !topk_w) return MOE_ERR_INVALID;
  if (T <= 0 || E <= 0 || k <= 0 || k > E || E > MOE_MAX_EXPERTS) return MOE_ERR_INVALID;
  if (!moe_aligned16(logits) || !moe_aligned16(topk_idx) || !moe_aligned16(topk_w)) return MOE_ERR_INVALID;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int r = renormalize != 0;
  // the same lane groups as the counting variant, so that both give the same bits (the order of the
  // sums in the softmax denominator follows the group shape)
  if (E <= 8) launch_route<8, 1>(logits, T, E, k, r, topk_idx, topk_w, s);
  else if (E <= 16) launch_route<8, 2>(logits, T, E, k, r, topk_idx, topk_w, s);
  else if (E <= 32) launch_route<8, 4>(logits, T, E, k, r, topk_idx, topk_w, s);
  else if (E <= 64) launch_route<8, 8>(logits, T, E, k, r, topk_idx, topk_w, s);
  else if (E <= 128) launch_route<16, 8>(logits, T, E, k, r, topk_idx, topk_w, s);
  else if (E <= 256) launch_route<32, 8>(logits, T, E, k, r, topk_idx, topk_w, s);
  else launch_route<64, 8>(logits, T, E, k, r, topk_idx, topk_w, s);
  return moe_check_launch();
}
