// Stage 5 of Algorithm 1 (ExpertOutputReductionForward / Backward) and the
// derivative of the Stage-4 gather, which is the same reduction with unit weights.
//
// The paper maps one thread to one output element (forward) or one routed row
// (backward).  Here one wave owns a token, or 64 or 128 pieces (16 B) of its row where tokens
// are few: every load and store is a full, coalesced row segment, the k source rows are
// summed in slot order in fp32, and the token's own row (out / dout) is touched
// exactly once.  No atomics, so results are reproducible.
#include <type_traits>
#include "gemm.h"

namespace {
// A routed row is read once per kernel: the load is marked non-temporal, so that the rows stream through the
// caches instead of displacing each other there (measured on the headline shape: 13 % less time when the rows
// come from HBM, 8 % inside the step).
typedef unsigned int u32x4_nt __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 nt_load(const uint4* p) {
  const u32x4_nt v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_nt*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ void fma8(float acc[8], const uint4& v, float w) {
  acc[0] += w * bf16lo(v.x); acc[1] += w * bf16hi(v.x);
  acc[2] += w * bf16lo(v.y); acc[3] += w * bf16hi(v.y);
  acc[4] += w * bf16lo(v.z); acc[5] += w * bf16hi(v.z);
  acc[6] += w * bf16lo(v.w); acc[7] += w * bf16hi(v.w);
}
__device__ __forceinline__ uint4 pack8(const float a[8]) {
  return make_uint4(pack_bf16(a[0], a[1]), pack_bf16(a[2], a[3]), pack_bf16(a[4], a[5]), pack_bf16(a[6], a[7]));
}
__device__ __forceinline__ float dot8(const uint4& a, const uint4& b) {
  return bf16lo(a.x) * bf16lo(b.x) + bf16hi(a.x) * bf16hi(b.x) + bf16lo(a.y) * bf16lo(b.y) + bf16hi(a.y) * bf16hi(b.y) +
         bf16lo(a.z) * bf16lo(b.z) + bf16hi(a.z) * bf16hi(b.z) + bf16lo(a.w) * bf16lo(b.w) + bf16hi(a.w) * bf16hi(b.w);
}
__device__ __forceinline__ uint4 scale8(const uint4& v, float w) {
  return make_uint4(pack_bf16(w * bf16lo(v.x), w * bf16hi(v.x)), pack_bf16(w * bf16lo(v.y), w * bf16hi(v.y)),
                    pack_bf16(w * bf16lo(v.z), w * bf16hi(v.z)), pack_bf16(w * bf16lo(v.w), w * bf16hi(v.w)));
}

// The next SLOTS slots of a token that have a local row, in slot order: mask holds those not yet taken (one bit per lane, lane i holds
// slot i's row), and what is taken leaves it.  Where fewer are left the first is repeated, so that every row can be loaded
// without a test; live says which count.
template <int SLOTS> struct SlotGroup {
  int lane[SLOTS], row[SLOTS];
  bool live[SLOTS];
  __device__ __forceinline__ SlotGroup(uint64_t& mask, int my_row) {
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
      live[s] = mask != 0;
      lane[s] = s == 0 || live[s] ? __builtin_ctzll(mask) : lane[0];
      mask &= mask - 1;
      row[s] = wave_lane(my_row, lane[s]);
    }
  }
};

// out[t] = sum_i w[t,i] * src[slot_row[t,i]]   (WEIGHTED)  or  sum_i src[slot_row[t,i]]
// A wave owns 64 VPT pieces of a token's row at a time (blockIdx.y: of every gridDim.y-th such part).  The token's slot rows and
// weights are fetched once (lane i holds slot i); the row loads of SLOTS slots are in flight together, without a branch between
// them (a lane without a piece reads the row's last one); the sum runs in slot order.
// PART: also dgate[t, i] = sum over c of part[slot_row[t, i] * strips + c], what the grouped products leave of the gradient of a
// folded gate weight (in the order of dgate_finish, the kernel of its own that larger passes have for it).
template <int VPT, int SLOTS, bool WEIGHTED, bool PART>
__global__ __launch_bounds__(256) void combine_kernel(const uint4* __restrict__ src, const int32_t* __restrict__ slot_row,
                                                      const float* __restrict__ topk_w, int T, int k, int chunks,
                                                      uint4* __restrict__ out, const float* __restrict__ part, int strips,
                                                      float* __restrict__ dgate) {
  const int lane = threadIdx.x % MOE_WAVE;
  const int t = blockIdx.x * (256 / MOE_WAVE) + threadIdx.x / MOE_WAVE;
  if (t >= T) return;
  for (int c0 = blockIdx.y * (MOE_WAVE * VPT); c0 < chunks; c0 += gridDim.y * (MOE_WAVE * VPT)) {
    float acc[VPT][8];
    int piece[VPT];
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
      piece[j] = min(c0 + j * MOE_WAVE + lane, chunks - 1);
#pragma unroll
      for (int q = 0; q < 8; ++q) acc[j][q] = 0.f;
    }
    for (int i0 = 0; i0 < k; i0 += MOE_WAVE) {
      const int kk = min(k - i0, MOE_WAVE);
      int my_row = -1;
      float my_w = 0.f;
      if (lane < kk) {
        my_row = slot_row[static_cast<size_t>(t) * k + i0 + lane];
        if (WEIGHTED) my_w = topk_w[static_cast<size_t>(t) * k + i0 + lane];
      }
      uint64_t mask = __ballot(my_row >= 0);
      while (mask != 0) {
        const SlotGroup<SLOTS> g(mask, my_row);
        uint4 v[SLOTS][VPT];
#pragma unroll
        for (int s = 0; s < SLOTS; ++s)
#pragma unroll
          for (int j = 0; j < VPT; ++j) v[s][j] = nt_load(src + static_cast<size_t>(g.row[s]) * chunks + piece[j]);
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
          if (g.live[s]) {
            const float w = WEIGHTED ? __int_as_float(wave_lane(__float_as_int(my_w), g.lane[s])) : 1.0f;
#pragma unroll
            for (int j = 0; j < VPT; ++j) fma8(acc[j], v[s][j], w);
          }
        }
      }
      if (PART && c0 == 0 && lane < kk) {
        float sum = 0.f;
        if (my_row >= 0) {
          const float* p = part + static_cast<size_t>(my_row) * strips;
#pragma unroll 8
          for (int c = 0; c < strips; ++c) sum += p[c];
        }
        dgate[static_cast<size_t>(t) * k + i0 + lane] = sum;
      }
    }
    uint4* o = out + static_cast<size_t>(t) * chunks;
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
      const int c = c0 + j * MOE_WAVE + lane;
      if (c < chunks) o[c] = pack8(acc[j]);
    }
  }
}

// The same, two slots at a time and under a mask, all parts of a row in one wave: for rows of at most 64 pieces, and for large passes
// most of whose slots have a row.  The former take a few us of latency whatever is done, and behind the other kernels of a layer,
// with its code not in the instruction cache, the short body is the quicker one (2 tokens of d 512, 8 slots: 22.3 us for the pass,
// 22.8-23.1 with the body above; 120 tokens of d 192 28.3 and 29.0).  The latter run at the rate of memory in either form, within
// the step a little better here (8192 tokens of d 2048, 8 slots 53.8 / 57.1 us; 20257 tokens of d 2368, 4 slots 80 / 84 us).
template <int VPT, bool WEIGHTED>
__global__ __launch_bounds__(256) void combine_pairs_kernel(const uint4* __restrict__ src, const int32_t* __restrict__ slot_row,
                                                            const float* __restrict__ topk_w, int T, int k, int chunks,
                                                            uint4* __restrict__ out) {
  const int lane = threadIdx.x % MOE_WAVE;
  const int t = blockIdx.x * (256 / MOE_WAVE) + threadIdx.x / MOE_WAVE;
  if (t >= T) return;
  for (int c0 = 0; c0 < chunks; c0 += MOE_WAVE * VPT) {
    float acc[VPT][8];
#pragma unroll
    for (int j = 0; j < VPT; ++j)
#pragma unroll
      for (int q = 0; q < 8; ++q) acc[j][q] = 0.f;
    for (int i0 = 0; i0 < k; i0 += MOE_WAVE) {
      const int kk = min(k - i0, MOE_WAVE);
      int my_row = -1;
      float my_w = 0.f;
      if (lane < kk) {
        my_row = slot_row[static_cast<size_t>(t) * k + i0 + lane];
        if (WEIGHTED) my_w = topk_w[static_cast<size_t>(t) * k + i0 + lane];
      }
      for (int i = 0; i < kk; i += 2) {
        const int row0 = __shfl(my_row, i, MOE_WAVE);
        const int row1 = i + 1 < kk ? __shfl(my_row, i + 1, MOE_WAVE) : -1;
        const float w0 = WEIGHTED ? __shfl(my_w, i, MOE_WAVE) : 1.0f;
        const float w1 = WEIGHTED ? __shfl(my_w, (i + 1) & (MOE_WAVE - 1), MOE_WAVE) : 1.0f;
        uint4 v0[VPT], v1[VPT];
#pragma unroll
        for (int j = 0; j < VPT; ++j) {
          const int c = c0 + j * MOE_WAVE + lane;
          const bool ok = c < chunks;
          v0[j] = ok && row0 >= 0 ? nt_load(src + static_cast<size_t>(row0) * chunks + c) : make_uint4(0, 0, 0, 0);
          v1[j] = ok && row1 >= 0 ? nt_load(src + static_cast<size_t>(row1) * chunks + c) : make_uint4(0, 0, 0, 0);
        }
        if (row0 >= 0) {
#pragma unroll
          for (int j = 0; j < VPT; ++j) fma8(acc[j], v0[j], w0);
        }
        if (row1 >= 0) {
#pragma unroll
          for (int j = 0; j < VPT; ++j) fma8(acc[j], v1[j], w1);
        }
      }
    }
    uint4* o = out + static_cast<size_t>(t) * chunks;
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
      const int c = c0 + j * MOE_WAVE + lane;
      if (c < chunks) o[c] = pack8(acc[j]);
    }
  }
}

// dyp[row(t,i)] = w[t,i] * dout[t];  dgate[t,i] = <yp[row(t,i)], dout[t]>;  OUT: also out[t] = sum_i w[t,i] * yp[row(t,i)], for a
// caller that runs the forward pass's combine and its backward one behind the other: the rows of yp are then read once.
// The token's dout segment is loaded once and kept in registers for all of its slots; the loads of SLOTS rows are in flight
// together; lane i collects the dot product of slot i (k <= 64 slots per pass over the lanes).
template <int VPT, int SLOTS, bool OUT>
__global__ __launch_bounds__(256) void combine_bwd_kernel(const uint4* __restrict__ dout, const uint4* __restrict__ yp,
                                                          const int32_t* __restrict__ slot_row,
                                                          const float* __restrict__ topk_w, int T, int k, int chunks,
                                                          uint4* __restrict__ dyp, float* __restrict__ dgate,
                                                          uint4* __restrict__ out) {
  const int lane = threadIdx.x % MOE_WAVE;
  const int t = blockIdx.x * (256 / MOE_WAVE) + threadIdx.x / MOE_WAVE;
  if (t >= T) return;
  const uint4* g = dout + static_cast<size_t>(t) * chunks;
  for (int i0 = 0; i0 < k; i0 += MOE_WAVE) {
    const int kk = min(k - i0, MOE_WAVE);
    // this pass's slots: lane i holds row and weight of slot i0 + i
    int my_row = -1;
    float my_w = 0.f, my_dot = 0.f;
    if (lane < kk) {
      my_row = slot_row[static_cast<size_t>(t) * k + i0 + lane];
      my_w = topk_w[static_cast<size_t>(t) * k + i0 + lane];
    }
    const uint64_t live = __ballot(my_row >= 0);
    // WHOLE: every lane has all of its pieces.  A row's ragged end is loaded under a mask: lanes that repeat its last piece would cost
    // as much as lanes that have one (d 768, 16384 tokens of 1 slot 18.8 / 14.3 us).
    auto part = [&](int c0, auto whole_tag) __attribute__((always_inline)) {
      constexpr bool WHOLE = decltype(whole_tag)::value;
      uint4 gv[VPT];
      bool has[VPT];
      float acc[OUT ? VPT : 1][8];
#pragma unroll
      for (int j = 0; j < VPT; ++j) {
        has[j] = WHOLE || c0 + j * MOE_WAVE + lane < chunks;
        gv[j] = has[j] ? g[c0 + j * MOE_WAVE + lane] : make_uint4(0, 0, 0, 0);
        if constexpr (OUT) {
#pragma unroll
          for (int q = 0; q < 8; ++q) acc[j][q] = 0.f;
        }
      }
      uint64_t mask = live;
      while (mask != 0) {
        const SlotGroup<SLOTS> sg(mask, my_row);
        uint4 yv[SLOTS][VPT];
#pragma unroll
        for (int s = 0; s < SLOTS; ++s)
#pragma unroll
          for (int j = 0; j < VPT; ++j)
            yv[s][j] = has[j] ? nt_load(yp + static_cast<size_t>(sg.row[s]) * chunks + c0 + j * MOE_WAVE + lane) : make_uint4(0, 0, 0, 0);
        float dot[SLOTS];
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
          dot[s] = 0.f;
          if (sg.live[s]) {
            const float w = __int_as_float(wave_lane(__float_as_int(my_w), sg.lane[s]));
            uint4* dy = dyp + static_cast<size_t>(sg.row[s]) * chunks + c0 + lane;
#pragma unroll
            for (int j = 0; j < VPT; ++j) {
              dot[s] += dot8(yv[s][j], gv[j]);
              if (has[j]) dy[j * MOE_WAVE] = scale8(gv[j], w);
              if constexpr (OUT) fma8(acc[j], yv[s][j], w);
            }
          }
        }
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
          dot[s] = group_sum<MOE_WAVE>(dot[s]);
          if (lane == sg.lane[s] && sg.live[s]) my_dot += dot[s];
        }
      }
      if constexpr (OUT) {       // k <= 64: the only pass over the slots
        uint4* o = out + static_cast<size_t>(t) * chunks + c0 + lane;
#pragma unroll
        for (int j = 0; j < VPT; ++j)
          if (has[j]) o[j * MOE_WAVE] = pack8(acc[j]);
      }
    };
    int c0 = 0;
    for (; c0 + MOE_WAVE * VPT <= chunks; c0 += MOE_WAVE * VPT) part(c0, std::true_type{});
    if (c0 < chunks) part(c0, std::false_type{});
    if (lane < kk) dgate[static_cast<size_t>(t) * k + i0 + lane] = my_dot;
  }
}

#define COMBINE(VPT, SLOTS, PART, PARTS)                                                                                           \
  MOE_LAUNCH(name, (combine_kernel<VPT, SLOTS, WEIGHTED, PART>), dim3((T + 3) / 4, PARTS), dim3(256), 0, s, a, slot_row, w, T, k, \
             chunks, o, part, strips, dgate)
#define COMBINE_PAIRS(VPT) \
  MOE_LAUNCH(name, (combine_pairs_kernel<VPT, WEIGHTED>), dim3((T + 3) / 4), dim3(256), 0, s, a, slot_row, w, T, k, chunks, o)
// A pass over so few bytes of rows is bound by latency or by loads in flight, not by the rate of memory.  With few waves: one for every
// 64 pieces, four slots at a time.  With more of them, fewer slots or rows of several pieces per lane: one for every 128 pieces, two
// slots at a time, since what a wave loads for slots that are not there (it repeats the first) then counts, and the waves alone keep
// enough in flight.  Whole kernel, us, (pairs of slots, all of a row in one wave) / (1 piece per lane, 4 slots) / (2, 2):
//   8 slots  d 2048:  40 tokens  6.1 / 4.2 / 5.5   1000 tokens   9.7 /  8.2 /  9.1   2048 (more than 48 MB) 15.1 / 16.3 / 14.9
//   6 slots  d 1536:  40 tokens  4.3 / 3.2 / 3.7   1000 tokens   6.7 /  6.1 /  7.0   2048  9.4 / 10.0 /  9.1
//   2 slots  d 2048:  40 tokens  3.4 / 2.8 / 2.9   1000 tokens   4.5 /  4.7 /  4.4   2048  6.9 /  7.5 /  6.4   4096 10.8 / 13.1 / 11.0
//   2 slots  d 768:                                1000 tokens   3.4 /  3.5 /  3.6   8192  8.4 / 10.8 /  8.4
//   1 slot   d 2048:  40 tokens  3.2 / 2.7 / 2.7   1000 tokens   3.9 /  3.9 /  3.6   8192 15.5 / 18.1 / 14.4
// (393 sizes, 1 to 8 slots, d 128 to 4096: the form chosen is at most 2.4 % behind the pairs and on average 8 % ahead of them.)
bool few_bytes(int T, int k, int d) { return static_cast<long long>(T) * k * d * 2 < (48 << 20); }

// sparse: most slots are expected to have no local row.  They are left out beforehand there: 24576 tokens of d 3072, 8 slots, one of
// twelve local, 55 -> 49 us (sum) and 50 -> 43 us (backward of the gather) against the pairs.
template <bool WEIGHTED>
int launch_combine(const moe_bf16* src, const int32_t* slot_row, const float* w, int T, int k, int d, moe_bf16* out,
                   hipStream_t s, const char* name, bool sparse, const float* part = nullptr, int strips = 0, float* dgate = nullptr) {
  const int chunks = d / 8;
  const uint4* a = reinterpret_cast<const uint4*>(src);
  uint4* o = reinterpret_cast<uint4*>(out);
  const bool few = few_bytes(T, k, d);
  const long long waves = static_cast<long long>(T) * ((chunks + 63) / 64), long_rows = (chunks + 255) / 256;
  if (part != nullptr) {
    if constexpr (!WEIGHTED) { if (chunks <= 64) COMBINE(1, 2, true, 1); else COMBINE(1, 4, true, (chunks + 63) / 64); }
  } else if (chunks <= 64) {
    COMBINE_PAIRS(1);
  } else if (few && waves <= (k > 2 ? 4096 : 1536) * long_rows) {
    COMBINE(1, 4, false, (chunks + 63) / 64);
  } else if (few && (sparse || k == 1 || (chunks > 128 && waves <= 8192 * long_rows))) {
    COMBINE(2, 2, false, (chunks + 127) / 128);
  } else if (chunks <= 128) {
    COMBINE_PAIRS(2);
  } else if (sparse) {
    COMBINE(4, 2, false, 1);
  } else {
    COMBINE_PAIRS(4);
  }
  return moe_check_launch();
}
#undef COMBINE_PAIRS
#undef COMBINE

#define COMBINE_BWD(VPT, SLOTS, OUT)                                                                                                   \
  MOE_LAUNCH(name, (combine_bwd_kernel<VPT, SLOTS, OUT>), dim3((T + 3) / 4), dim3(256), 0, s, a, y, slot_row, topk_w, T, k, chunks, o, \
             dgate, ov)
template <bool OUT>
int launch_combine_bwd(const moe_bf16* dout, const moe_bf16* yp, const int32_t* slot_row, const float* topk_w, int T, int k, int d,
                       moe_bf16* dyp, float* dgate, moe_bf16* out, hipStream_t s, const char* name) {
  const int chunks = d / 8;
  const uint4* a = reinterpret_cast<const uint4*>(dout);
  const uint4* y = reinterpret_cast<const uint4*>(yp);
  uint4* o = reinterpret_cast<uint4*>(dyp);
  uint4* ov = reinterpret_cast<uint4*>(out);
  // Slots in flight.  What is loaded for slots that are not there costs as much as for those that are, and rows of several pieces per
  // lane and many waves keep enough in flight by themselves.  combine_bwd, us, 1 / 2 / 4 slots in flight:
  //   1 slot   d 512, 40 tokens 2.7 / 2.7 / 2.9   d 320, 16384 tokens  8.4 /  8.7 / 10.0   d 2560,  4096 tokens 11.6 / 11.6 / 14.1
  //   2 slots  d 512, 40 tokens 2.8 / 2.8 / 3.0   d 320, 16384 tokens 11.4 / 11.0 / 12.3   d  768,  8192 tokens 11.4 / 12.8 / 14.3
  //   3 slots                                     d 128, 32768 tokens 21.4 / 20.1 / 19.4   d  768, 16384 tokens 30.5 / 31.5 / 32.7
  //   8 slots  d 512, 40 tokens 4.0 / 4.1 / 4.0   d 128, 32768 tokens 43.0 / 34.5 / 33.1   d 2048,  8192 tokens  103 /  103 /  103
  // Before (one slot at a time, the reductions through LDS): 3.0, 8.8, 11.9; 3.4, 12.2, 11.8; 23.3, 30.7; 6.3, 48.2, 106 for these.
  // Three pieces per lane for rows that mostly fill the third: d 1536, 1 slot, 8192 tokens 15.1 (four pieces) / 13.8, before 14.0; 8 slots,
  // 40 tokens 6.5 / 5.0 (d 1088, 2 slots, 8192 tokens 17.4 / 17.8).
  // combine and combine_bwd apart / in one (OUT): d 2048, 48 tokens 10.6 / 8.2 and a launch, 8192 tokens 158 / 119; d 1024, 24576
  // tokens of 2 slots 65 / 47.
  const int slots = k == 1 || (k < 4 && chunks > 64 && T > 2048) ? 1 : k == 2 || (chunks > 64 && T > 512) ? 2 : 4;
  if (chunks <= 64) { if (slots == 1) COMBINE_BWD(1, 1, OUT); else if (slots == 2) COMBINE_BWD(1, 2, OUT); else COMBINE_BWD(1, 4, OUT); }
  else if (chunks <= 128) { if (slots == 1) COMBINE_BWD(2, 1, OUT); else if (slots == 2) COMBINE_BWD(2, 2, OUT); else COMBINE_BWD(2, 4, OUT); }
  else if (chunks > 160 && chunks <= 192) { if (slots == 1) COMBINE_BWD(3, 1, OUT); else if (slots == 2) COMBINE_BWD(3, 2, OUT); else COMBINE_BWD(3, 4, OUT); }
  else { if (slots == 1) COMBINE_BWD(4, 1, OUT); else if (slots == 2) COMBINE_BWD(4, 2, OUT); else COMBINE_BWD(4, 4, OUT); }
  return moe_check_launch();
}
#undef COMBINE_BWD

bool bad_dims(int T, int k, int d) { return T <= 0 || k <= 0 || d <= 0 || d % 8 != 0; }

}  // namespace

extern "C" int moe_unpermute_combine(const moe_bf16* yp, const int32_t* slot_row, const float* topk_w, int T, int k, int d,
                                     moe_bf16* out, void* stream) {
  if (!yp || !slot_row || !topk_w || !out || bad_dims(T, k, d)) return MOE_ERR_INVALID;
  if (!moe_aligned16(yp) || !moe_aligned16(out) || !moe_aligned16(slot_row) || !moe_aligned16(topk_w)) return MOE_ERR_INVALID;
  return launch_combine<true>(yp, slot_row, topk_w, T, k, d, out, static_cast<hipStream_t>(stream), "combine", false);
}

extern "C" int moe_permute_bwd(const moe_bf16* dxp, const int32_t* slot_row, int T, int k, int d, moe_bf16* dx,
                               void* stream) {
  if (!dxp || !slot_row || !dx || bad_dims(T, k, d)) return MOE_ERR_INVALID;
  if (!moe_aligned16(dxp) || !moe_aligned16(dx) || !moe_aligned16(slot_row)) return MOE_ERR_INVALID;
  return launch_combine<false>(dxp, slot_row, nullptr, T, k, d, dx, static_cast<hipStream_t>(stream), "permute_bwd", false);
}

// Saves the launch of dgate_finish (4 us) where the whole backward of the gather takes a few us; larger passes would wait for the
// strips (24576 tokens, one twelfth of their slots local: 50 + 8 us apart, 82 in one).
bool moe_permute_bwd_adds_dgate(int T, int k, int d) { return few_bytes(T, k, d) && static_cast<long long>(T) * k <= 16384; }

int moe_permute_bwd_dgate(const moe_bf16* dxp, const int32_t* slot_row, int T, int k, int d, moe_bf16* dx, const float* part,
                          int strips, float* dgate, void* stream) {
  if (!dxp || !slot_row || !dx || !part || !dgate || strips <= 0 || bad_dims(T, k, d)) return MOE_ERR_INVALID;
  if (!moe_aligned16(dxp) || !moe_aligned16(dx) || !moe_aligned16(slot_row) || !moe_aligned16(dgate)) return MOE_ERR_INVALID;
  return launch_combine<false>(dxp, slot_row, nullptr, T, k, d, dx, static_cast<hipStream_t>(stream), "permute_bwd", false, part, strips, dgate);
}

extern "C" int moe_unpermute_sum(const moe_bf16* ypw, const int32_t* slot_row, int T, int k, int d, moe_bf16* out,
                                 void* stream) {
  if (!ypw || !slot_row || !out || bad_dims(T, k, d)) return MOE_ERR_INVALID;
  if (!moe_aligned16(ypw) || !moe_aligned16(out) || !moe_aligned16(slot_row)) return MOE_ERR_INVALID;
  return launch_combine<false>(ypw, slot_row, nullptr, T, k, d, out, static_cast<hipStream_t>(stream), "combine", false);
}

extern "C" int moe_unpermute_combine_bwd(const moe_bf16* dout, const moe_bf16* yp, const int32_t* slot_row,
                                         const float* topk_w, int T, int k, int d, moe_bf16* dyp, float* dgate,
                                         void* stream) {
  if (!dout || !yp || !slot_row || !topk_w || !dyp || !dgate || bad_dims(T, k, d)) return MOE_ERR_INVALID;
  if (!moe_aligned16(dout) || !moe_aligned16(yp) || !moe_aligned16(dyp) || !moe_aligned16(slot_row) ||
      !moe_aligned16(topk_w) || !moe_aligned16(dgate))
    return MOE_ERR_INVALID;
  return launch_combine_bwd<false>(dout, yp, slot_row, topk_w, T, k, d, dyp, dgate, nullptr, static_cast<hipStream_t>(stream), "combine_bwd");
}

int moe_combine_sparse(const moe_bf16* src, const int32_t* slot_row, const float* topk_w, int T, int k, int d, moe_bf16* out,
                       const char* name, void* stream) {
  if (!src || !slot_row || !out || bad_dims(T, k, d)) return MOE_ERR_INVALID;
  const void* ptrs[] = {src, slot_row, topk_w, out};
  for (const void* p : ptrs) if (!moe_aligned16(p)) return MOE_ERR_INVALID;
  hipStream_t s = static_cast<hipStream_t>(stream);
  return topk_w != nullptr ? launch_combine<true>(src, slot_row, topk_w, T, k, d, out, s, name, true)
                           : launch_combine<false>(src, slot_row, nullptr, T, k, d, out, s, name, true);
}

int moe_combine_both(const moe_bf16* dout, const moe_bf16* yp, const int32_t* slot_row, const float* topk_w, int T, int k, int d,
                     moe_bf16* out, moe_bf16* dyp, float* dgate, void* stream) {
  if (k > MOE_WAVE) {
    const int rc = moe_unpermute_combine(yp, slot_row, topk_w, T, k, d, out, stream);
    return rc != MOE_OK ? rc : moe_unpermute_combine_bwd(dout, yp, slot_row, topk_w, T, k, d, dyp, dgate, stream);
  }
  if (!dout || !yp || !slot_row || !topk_w || !dyp || !dgate || !out || bad_dims(T, k, d)) return MOE_ERR_INVALID;
  const void* ptrs[] = {dout, yp, dyp, slot_row, topk_w, dgate, out};
  for (const void* p : ptrs) if (!moe_aligned16(p)) return MOE_ERR_INVALID;
  return launch_combine_bwd<true>(dout, yp, slot_row, topk_w, T, k, d, dyp, dgate, out, static_cast<hipStream_t>(stream), "combine+bwd");
}
