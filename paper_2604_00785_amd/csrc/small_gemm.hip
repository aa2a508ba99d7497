// Grouped products for experts with few rows (a decoding step, a short prompt): what bounds them is the one pass
// over the weights of the experts that have rows, 2 bytes for at most 2 * 16 operations.  The tiled kernel of
// grouped_gemm.hip, made for many rows, has one workgroup per compute unit and spends as long between its tiles as
// they take to stream here; with one token its eight experts are 64 tiles for 256 compute units.
//
// Here a workgroup owns 64 weight rows (32 of Wg and the same 32 of Wu, or 64 of Wd) of one expert and up to 16 activation
// rows.  Each wave streams its FR fragments of 16 weight rows: FR = 4 is one wave for the whole tile, FR = 2 two waves that share it (and load
// the activations twice).  Loads go straight into a ring in LDS that only this wave uses, eight rows of 128 bytes an instruction; fragments
// are read from there, and there is no barrier in the loop.  A weight byte passes through one wave of the chip once, and the waves
// of a compute unit overlap each other's start and end.
//
// (Loaded from memory into the registers of the matrix instruction, whose neighbouring lanes hold different rows, each load touches 64
// lines with 16 bytes: 64 cycles of the compute unit's one address path instead of 16, which bounded a token's products at some 4
// TB/s.  Same card, whole forward pass, d 2048, f 1024, 64 experts, 8 per token, registers -> LDS: 16 tokens 153 -> 145 us, 48 tokens 169 -> 164 us, 64 tokens with
// a zipf load 166 -> 146 us; 24 tokens of d 1088, f 576, 96 experts 59 -> 56 us; with the joined kernels below one token 34.4 -> 29.2 us.)
//
// A wave takes the WHOLE reduction in its order and so gives the bits of the tiled kernel: a row's result does not depend
// on how many rows the call has.  Splitting the reduction over four waves rounds differently; it was 2-6 % faster at 8 to 32
// tokens of d 2048, f 1024, 64 experts, 10 % with 8 experts of d 4096, and up to 15 % slower elsewhere (narrow experts,
// skewed loads).
#include "dma.h"
#include "route_token.h"
#include "small_gemm.h"

namespace {

constexpr int ST_KB = 64;             // reduction elements of a piece: 128 bytes of a weight row
constexpr int ST_ROWS = 16;           // activation rows of a tile
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

__device__ __forceinline__ float st_sigmoid(float g) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g));
}
__device__ __forceinline__ int sfirst(int v) { return __builtin_amdgcn_readfirstlane(v); }

struct StTile { int e, m0, m_end, col; };

// The tile of this workgroup: expert, rows, column tile; false if there are fewer tiles (the grid covers the most there
// can be).  An expert's tiles are numbered column tile by column tile, its row tiles innermost, and an XCD gets a run
// of consecutive numbers, so that row tiles that share weights share an L2.  Every wave looks its tile up by itself.
__device__ __forceinline__ bool st_find_tile(const int32_t* __restrict__ offsets, int E, int ncol, StTile& t) {
  const int lane = threadIdx.x & 63;
  int lo[MOE_MAX_EXPERTS / 64], hi[MOE_MAX_EXPERTS / 64], inc[MOE_MAX_EXPERTS / 64];
  int total = 0;
#pragma unroll
  for (int c = 0; c < MOE_MAX_EXPERTS / 64; ++c) {
    lo[c] = 0; hi[c] = 0;
    const int e = c * 64 + lane;
    if (c * 64 < E && e < E) { lo[c] = offsets[e]; hi[c] = offsets[e + 1]; }
  }
#pragma unroll
  for (int c = 0; c < MOE_MAX_EXPERTS / 64; ++c) {
    inc[c] = 0;
    if (c * 64 < E) {
      inc[c] = total + wave_incl_scan((hi[c] - lo[c] + ST_ROWS - 1) / ST_ROWS);
      total = wave_lane(inc[c], 63);
    }
  }
  total *= ncol;
  const int per_xcd = (total + 7) >> 3;
  const int b = blockIdx.x;
  const int q = (b & 7) * per_xcd + (b >> 3);
  if ((b >> 3) >= per_xcd || q >= total) return false;
#pragma unroll
  for (int c = 0; c < MOE_MAX_EXPERTS / 64; ++c) {
    if (c * 64 < E) {
      const int rt = (hi[c] - lo[c] + ST_ROWS - 1) / ST_ROWS;
      const int excl = inc[c] - rt;
      const unsigned long long hit = __ballot(rt > 0 && excl * ncol <= q && q < inc[c] * ncol);
      if (hit) {
        const int l = __ffsll(hit) - 1;
        t.e = c * 64 + l;
        const int r = wave_lane(rt, l);
        const int in = q - wave_lane(excl, l) * ncol;
        t.col = in / r;
        t.m0 = wave_lane(lo[c], l) + (in - t.col * r) * ST_ROWS;
        t.m_end = wave_lane(hi[c], l);
        return true;
      }
    }
  }
  return false;
}

// A wave's own ring in LDS: RING pieces of FR fragments of 16 weight rows and 8 XL activation rows, 128 bytes each.
template <int FR, int XL> constexpr int st_piece_bytes() { return (2 * FR + XL) * 1024; }
typedef const __attribute__((address_space(3))) bf16x8_t* LdsFrag;
// The 16-byte piece `logical` of a row lies at physical piece (logical + row) mod 8, as in the tiles of grouped_gemm.hip; the lane's
// share of it in a load that fills 8 rows: row lane / 8, physical piece lane % 8.
__device__ __forceinline__ uint32_t st_lane_piece(int lane) { return static_cast<uint32_t>(((lane & 7) - (lane >> 3)) & 7) * 16u; }

// Streams the FR fragments of 16 weight rows at wb (lane offsets wl of rows 0-7 and 8-15) against the activation rows at xb (xl; XL = 1:
// eight rows stand for all sixteen) and adds the products to acc: np pieces of the reduction.
// RING - 1 pieces are in flight; nobody but the wave touches its ring, so there is no barrier.
template <int FR, int XL, int RING>
__device__ __forceinline__ void st_stream(const char* const (&wb)[FR], const uint32_t (&wl)[2], const char* xb, const uint32_t (&xl)[XL],
                                          int np, const char* ring, f32x4_t (&acc)[FR]) {
  constexpr int LOADS = 2 * FR + XL, BYTES = st_piece_bytes<FR, XL>();
  const int lane = threadIdx.x & 63, i16 = lane & 15, g4 = lane >> 4;
  const uint32_t lds = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(reinterpret_cast<size_t>(LDS_PTR(ring))));
  auto load = [&](int p, int slot) __attribute__((always_inline)) {
    const int ko = p * (ST_KB * 2);
    uint32_t at = lds + slot * BYTES;
    auto rows = [&](const char* base, const uint32_t* off, int n) __attribute__((always_inline)) {
      base += ko;
      settle(base);
#pragma unroll
      for (int i = 0; i < n; ++i, at += 1024) {
        set_m0_rt(__builtin_amdgcn_readfirstlane(at));
        dma16_imm<0>(off[i], base);
      }
    };
#pragma unroll
    for (int j = 0; j < FR; ++j) rows(wb[j], wl, 2);
    rows(xb, xl, XL);
  };
#pragma unroll
  for (int p = 0; p < RING - 1; ++p) if (p < np) load(p, p);
  // lane addresses of the two halves of a piece: rows i16 of the weights and of the activations
  const uint32_t wr = lds + i16 * 128, xr = lds + FR * 2048 + (i16 & (8 * XL - 1)) * 128;
  const uint32_t half[2] = {((g4 + i16) & 7) * 16u, ((4 + g4 + i16) & 7) * 16u};
  int slot = 0, next = RING - 1;
#pragma clang loop unroll(disable)
  for (int p = 0; p < np; ++p) {
    if (p + RING - 1 <= np) wait_vm<(RING - 2) * LOADS>(); else wait_vm<0>();   // piece p is here
    if (p + RING - 1 < np) load(p + RING - 1, next);                           // where piece p - 1 was, which has been read
    const uint32_t o = slot * BYTES;
    bf16x8_t w[2][FR], x[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      x[h] = *(LdsFrag)(xr + o + half[h]);
#pragma unroll
      for (int j = 0; j < FR; ++j) w[h][j] = *(LdsFrag)(wr + o + j * 2048 + half[h]);
    }
    lds_wait<0>();
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < FR; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[h][j], x[h], acc[j], 0, 0, 0);
    slot = slot + 1 == RING ? 0 : slot + 1;
    next = next + 1 == RING ? 0 : next + 1;
  }
}

// One tile.  Its 64 weight rows are four fragments of 16 (GATE_UP: 0, 1 = 32 rows of Wg, 2, 3 = the same rows of Wu), FR of them
// to a wave.  Weight row and lane are matched so that a lane of the epilogue ends up with neighbouring output columns
// (16-byte stores).  row_token, row_weight: as in the arguments, or what the workgroup itself has found.
template <bool GATE_UP, int FR, int RING>
__device__ __forceinline__ void st_fwd_tile(const StreamFwdArgs& a, const StTile& t, const int32_t* row_token, const float* row_weight,
                                            char* lds) {
  constexpr int NB = 4;
  constexpr int NBC = GATE_UP ? 2 : 4;                  // fragments per tensor; a lane ends up with 4 * NBC columns
  const int tid = threadIdx.x, lane = tid & 63, wave = sfirst(tid >> 6);
  const int i16 = lane & 15, g4 = lane >> 4;
  const int K = a.K;
  const int n0 = t.col * (16 * NBC);
  const int np = K / ST_KB;

  f32x4_t acc[FR];
#pragma unroll
  for (int j = 0; j < FR; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // weights: fragment q, lane i16 -> output column n0 + (i16 / 4) * 4 NBC + 4 (q % NBC) + i16 % 4
  const char* wb[FR];
#pragma unroll
  for (int j = 0; j < FR; ++j) {
    const int q = wave * FR + j;
    wb[j] = reinterpret_cast<const char*>((GATE_UP && q >= NBC ? a.B1 : a.B0) +
                                          (static_cast<size_t>(t.e) * a.N + n0 + 4 * (q % NBC)) * K);
  }
  uint32_t wl[2], xl[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int m = 8 * i + (lane >> 3);                  // row of a fragment, of the activations
    wl[i] = static_cast<uint32_t>(((m >> 2) * 4 * NBC + (m & 3)) * K) * 2u + st_lane_piece(lane);
    const int r = t.m0 + m < t.m_end ? t.m0 + m : t.m_end - 1;
    const uint32_t row = row_token != nullptr ? static_cast<uint32_t>(row_token[r]) : static_cast<uint32_t>(r - t.m0);
    xl[i] = row * static_cast<uint32_t>(K) * 2u + st_lane_piece(lane);
  }
  const char* xb = reinterpret_cast<const char*>(a.A + (row_token != nullptr ? 0 : static_cast<size_t>(t.m0) * K));
  st_stream<FR, 2, RING>(wb, wl, xb, xl, np, lds + wave * (RING * st_piece_bytes<FR, 2>()), acc);
  __syncthreads();                                      // every wave is done with its ring
  f32x4_t* const part = reinterpret_cast<f32x4_t*>(lds);
  // the fragments' sums meet in LDS, where a lane of the epilogue finds its neighbouring columns
#pragma unroll
  for (int j = 0; j < FR; ++j) part[(wave * FR + j) * 64 + lane] = acc[j];
  __syncthreads();
  if (wave == 0) {
    f32x4_t v[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) v[j] = part[j * 64 + lane];
    const int r = t.m0 + i16;
    if (r < t.m_end) {
      const size_t o = static_cast<size_t>(r) * a.N + n0 + g4 * 4 * NBC;
      auto put8 = [&](uint16_t* p, const f32x4_t& lo, const f32x4_t& hi) __attribute__((always_inline)) {
        *reinterpret_cast<u32x4*>(p) = u32x4{pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3]), pack_bf16(hi[0], hi[1]), pack_bf16(hi[2], hi[3])};
      };
      if constexpr (GATE_UP) {
        const float rw = row_weight != nullptr ? row_weight[r] : 1.f;
        f32x4_t h[2];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int c = 0; c < 4; ++c) h[j][c] = v[j][c] * st_sigmoid(v[j][c]) * v[j + 2][c] * rw;
        put8(a.O0 + o, v[0], v[1]);
        put8(a.O1 + o, v[2], v[3]);
        put8(a.O2 + o, h[0], h[1]);
      } else {
        put8(a.O0 + o, v[0], v[1]);
        put8(a.O0 + o + 8, v[2], v[3]);
      }
    }
  }
}

template <bool GATE_UP, int FR, int RING>
__global__ __launch_bounds__(256 / FR) void stream_fwd_kernel(StreamFwdArgs a) {
  __shared__ __attribute__((aligned(1024))) char lds[4 / FR * RING * st_piece_bytes<FR, 2>()];
  const int rows = a.offsets[a.E];
  StTile t;
  if (!st_find_tile(a.offsets, a.E, a.N / (GATE_UP ? 32 : 64), t) || rows > a.max_rows) return;
  st_fwd_tile<GATE_UP, FR, RING>(a, t, a.row_token, a.row_weight, lds);
}

template <bool GATE_UP, int FR, int RING>
int launch_fwd(const StreamFwdArgs& a, hipStream_t s, const char* name) {
  const int ncol = a.N / (GATE_UP ? 32 : 64);
  const long long row_tiles = a.max_rows / ST_ROWS + (a.E < a.max_rows ? a.E : a.max_rows);
  const long long tiles = (row_tiles * ncol + 7) & ~7ll;
  if (tiles > 0x7FFFFFFFll) return MOE_ERR_INVALID;
  MOE_LAUNCH(name, (stream_fwd_kernel<GATE_UP, FR, RING>), dim3(static_cast<unsigned>(tiles)), dim3(256 / FR), 0, s, a);
  return moe_check_launch();
}
// Under an even load rows * E / (rows + E) experts, roughly, have a row.
long long st_expected_tiles(long long rows, int E, int ncol) { return rows * E / (rows + E) * ncol; }
// With few tiles for the 256 compute units two waves share a tile and each keeps three pieces in flight; beyond that one wave takes a
// tile with two pieces in flight, and five of them on a compute unit overlap (30 KB of LDS each).  The number of tiles is that of an even
// load; a skewed one uses fewer experts, so the second variant must do for few tiles too: rings of two pieces, eight waves on a compute
// unit, are up to 3 % faster at 770 to 1540 tiles of an even load, and 11 tokens of d 4096, f 2048, 61 experts, 1 per token, zipf load, took 91 us
// with them and 69 us before.  6300 calls of 1 to 64 tokens, gate_up in each variant, forward time over the best one's, mean and 95th percentile:
//                          even load: 2 waves, 4 pieces | 1, 2 | 1, 3     zipf load
//   128 to 255 tiles           1.01 1.04 | 1.27 1.55 | 1.05 1.13     1.00 1.03 | 1.29 1.60 | 1.06 1.15
//   256 to 383                 1.02 1.04 | 1.17 1.31 | 1.01 1.03     1.01 1.05 | 1.21 1.46 | 1.03 1.12
//   384 to 512                 1.02 1.05 | 1.08 1.17 | 1.00 1.02     1.02 1.05 | 1.16 1.38 | 1.02 1.09
//   513 to 768                 1.03 1.06 | 1.04 1.07 | 1.01 1.04     1.02 1.05 | 1.10 1.27 | 1.01 1.05
//   769 to 1536                1.03 1.07 | 1.01 1.07 | 1.03 1.07     1.03 1.07 | 1.05 1.23 | 1.01 1.05
//   from 1537                  1.01 1.07 | 1.04 1.08 | 1.01 1.03     1.04 1.11 | 1.02 1.09 | 1.02 1.06
// (down: the same order, half the differences.)  Where weight rows are multiples of 4096 bytes, waves that run in step read the same few bytes of each,
// which lie in a fraction of the memory channels; more pieces in flight spread over more of them (from 513 tiles on 1.01 | 1.03 | 1.03 for an even load,
// 1.02 | 1.07 | 1.02 for a zipf load).  d 2048, f 1024, 64 experts, 8 per token, gate_up in the three variants, forward in us: 16 tokens
// 151 / 163 / 159, 48 tokens 165 / 177 / 172, 64 tokens 176 / 203 / 182, with a zipf load 156 / 178 / 161 (48 tokens with the same kernels: 147 to 177,
// by where the weights lie in memory).  The rule is 0.9 % off the best of five variants on average
// in gate_up and 0.5 % in down, 7 % and 4 % off in one call of a hundred (the line at 512 tiles and rings of two: 1.7 and 1.0 %, 21 and 11 %).
template <bool GATE_UP>
int launch_fwd_any(const StreamFwdArgs& a, long long rows, hipStream_t s, const char* name) {
  if (st_expected_tiles(rows, a.E, a.N / (GATE_UP ? 32 : 64)) < 384 || a.K % 2048 == 0) return launch_fwd<GATE_UP, 2, 4>(a, s, name);
  return launch_fwd<GATE_UP, 4, 3>(a, s, name);
}

// ---- A decoding step of a few sequences in fewer launches -----------------------------------------------------------------
// The layer is then four kernels of a few us (routing, gate_up, down, combine) that each wait for the one before and reach their rate of
// memory late; here every wave of gate_up routes the tokens by itself, and down also combines.  Forward pass in us, four launches / routing with gate_up /
// down with the combine / both (the same products): one token of d 2048, f 1024, 64 experts, 8 per token 33.5 / 31.1 / 31.4 / 29.1; one of d 4096,
// f 2048, 64 experts, 2 per token 37.2 / 35.1 / 32.1 / 29.7; 2 of d 1088, f 576, 96 experts, 4 per token 21.3 / 18.9 / 18.4 / 16.3; 4 of d 512, f 256,
// 128 experts, 8 per token 20.1 / 18.7 / 17.3 / 16.1; 8 of d 2048, f 1024, 64 experts, 4 per token 77.4 / 74.2.

// Stages 1 to 3 and gate_up, at most 64 (token, slot) pairs.  A wave routes all tokens (lane groups, selection and sums of route.hip), finds
// the pairs' rows among its 64 lanes with ballots, as the counting sort does, and takes its tile from there; the last workgroup writes what
// Stages 1 to 3 leave behind.
struct StRouteArgs {
  const float* logits;
  int32_t* topk_idx;
  float* topk_w;
  int32_t *offsets, *row_token, *slot_row;
  float* row_weight;            // may be null
  int T, E, k, renormalize, e_begin, nbits;
};
template <int G, int VPL, int FR, int RING>
__global__ __launch_bounds__(256 / FR) void route_gate_up_kernel(StRouteArgs r, StreamFwdArgs a) {
  constexpr int WAVES = 4 / FR;
  __shared__ __attribute__((aligned(1024))) char lds[WAVES * RING * st_piece_bytes<FR, 2>()];
  __shared__ int s_e[WAVES][MOE_WAVE], s_token[WAVES][MOE_WAVE];
  __shared__ float s_w[WAVES][MOE_WAVE], s_weight[WAVES][MOE_WAVE];
  const int lane = threadIdx.x % MOE_WAVE, wave = sfirst(threadIdx.x / MOE_WAVE), gl = lane % G;
  const int n = r.T * r.k;
  for (int t0 = 0; t0 < r.T; t0 += MOE_WAVE / G) {
    const int t = t0 + lane / G, tt = t < r.T ? t : r.T - 1;
    float val[VPL], my_w[VPL];
    int my_idx[VPL];
#pragma unroll
    for (int j = 0; j < VPL; ++j) {
      const int e = gl + j * G;
      val[j] = e < r.E ? r.logits[static_cast<size_t>(tt) * r.E + e] : 0.f;
    }
    route_token<G, VPL>(val, gl, r.E, r.k, r.renormalize, my_idx, my_w);
#pragma unroll
    for (int j = 0; j < VPL; ++j) {
      const int i = gl + j * G;
      if (i < r.k && t < r.T) { s_e[wave][t * r.k + i] = my_idx[j]; s_w[wave][t * r.k + i] = my_w[j]; }
    }
  }
  __builtin_amdgcn_wave_barrier();
  const int expert = lane < n ? s_e[wave][lane] : -1;
  const float weight = lane < n ? s_w[wave][lane] : 0.f;
  int e = expert - r.e_begin;
  if (expert < 0 || e < 0 || e >= a.E) e = -1;
  uint64_t smaller;
  const uint64_t same = same_expert_mask(e, r.nbits, smaller);
  const int first = __builtin_popcountll(smaller), rank = __builtin_popcountll(same & lanemask_lt());
  const int row = e >= 0 ? first + rank : -1;
  if (row >= 0) { s_token[wave][row] = lane / r.k; s_weight[wave][row] = weight; }
  __builtin_amdgcn_wave_barrier();
  if (blockIdx.x == gridDim.x - 1) {
    if (wave != 0) return;
    if (lane < n) {
      r.topk_idx[lane] = expert;
      r.topk_w[lane] = weight;
      r.slot_row[lane] = row;
      if (row >= 0) {
        r.row_token[row] = lane / r.k;
        if (r.row_weight != nullptr) r.row_weight[row] = weight;
      }
    }
    for (int x0 = 0; x0 <= a.E; x0 += MOE_WAVE) {
      int below = 0;
      for (int q = 0; q < n; ++q) {
        const int eq = wave_lane(e, q);
        below += eq >= 0 && eq < x0 + lane ? 1 : 0;
      }
      if (x0 + lane <= a.E) r.offsets[x0 + lane] = below;
    }
    return;
  }
  // an XCD gets a run of consecutive tiles, as in st_find_tile; no expert has more rows than a tile
  const uint64_t heads = __ballot(e >= 0 && rank == 0);
  const int ncol = a.N / 32, total = __builtin_popcountll(heads) * ncol, per_xcd = (total + 7) >> 3;
  const int q = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (static_cast<int>(blockIdx.x >> 3) >= per_xcd || q >= total) return;
  const int index = q / ncol;
  const uint64_t hit = __ballot(e >= 0 && rank == 0 && __builtin_popcountll(smaller & heads) == index);
  const int l = __ffsll(static_cast<unsigned long long>(hit)) - 1;
  StTile t;
  t.e = wave_lane(e, l);
  t.m0 = wave_lane(first, l);
  t.m_end = t.m0 + wave_lane(__builtin_popcountll(same), l);
  t.col = q - index * ncol;
  st_fwd_tile<true, FR, RING>(a, t, s_token[wave], r.row_weight != nullptr ? s_weight[wave] : nullptr, lds);
}

// down and combine.  A workgroup owns a token and 16 output columns, a wave one of the token's slots: it streams the 16 rows of its
// expert's Wd against the slot's row of h.  The rows of yp are rounded to bf16 (and written) as down does and added in slot order as combine
// does.  Weights of an expert that several tokens chose are read by each of them.
struct StDownArgs {
  const uint16_t *h, *Wd;
  const int32_t *offsets, *slot_row;
  const float* topk_w;          // null: rows of h carry their weights
  uint16_t *yp, *out;
  int T, k, E, K, N;
};
constexpr int ST_DOWN_SLOTS = 8, ST_DOWN_RING = 6;
__global__ __launch_bounds__(ST_DOWN_SLOTS * MOE_WAVE) void down_combine_kernel(StDownArgs a) {
  __shared__ __attribute__((aligned(1024))) char lds[ST_DOWN_SLOTS * ST_DOWN_RING * st_piece_bytes<1, 1>()];
  __shared__ float s_y[ST_DOWN_SLOTS][16], s_w[ST_DOWN_SLOTS];
  __shared__ int s_row[ST_DOWN_SLOTS];
  const int lane = threadIdx.x % MOE_WAVE, slot = sfirst(threadIdx.x / MOE_WAVE);
  const int i16 = lane & 15, g4 = lane >> 4;
  // the workgroups of a column tile follow each other on one XCD
  const int per = 8 * a.T, col = blockIdx.x / per * 8 + (blockIdx.x & 7), t = blockIdx.x % per >> 3;
  if (col >= a.N / 16) return;
  const int n0 = col * 16, pair = t * a.k + slot;
  const int end = lane < a.E ? a.offsets[lane + 1] : 0x7FFFFFFF;
  const int row = sfirst(a.slot_row[pair]);
  if (lane == 0) {
    s_row[slot] = row;
    s_w[slot] = a.topk_w != nullptr ? a.topk_w[pair] : 1.f;
  }
  if (row >= 0) {
    // the row's expert, from what the stages read: a caller may have laid topk_idx, which none reads behind the routing, under their results
    int e = __builtin_popcountll(__ballot(end <= row));
    for (int x0 = MOE_WAVE; x0 < a.E; x0 += MOE_WAVE) {
      const int x = x0 + lane;
      e += __builtin_popcountll(__ballot(x < a.E && a.offsets[x + 1] <= row));
    }
    e = sfirst(e);
    f32x4_t acc[1] = {f32x4_t{0.f, 0.f, 0.f, 0.f}};
    const char* const wb[1] = {reinterpret_cast<const char*>(a.Wd + (static_cast<size_t>(e) * a.N + n0) * a.K)};
    const uint32_t wl[2] = {static_cast<uint32_t>((lane >> 3) * a.K) * 2u + st_lane_piece(lane),
                            static_cast<uint32_t>((8 + (lane >> 3)) * a.K) * 2u + st_lane_piece(lane)};
    const uint32_t xl[1] = {st_lane_piece(lane)};
    st_stream<1, 1, ST_DOWN_RING>(wb, wl, reinterpret_cast<const char*>(a.h + static_cast<size_t>(row) * a.K), xl, a.K / ST_KB,
                                  lds + slot * (ST_DOWN_RING * st_piece_bytes<1, 1>()), acc);
    if (i16 == 0) {
      typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
      const u32x2 y = {pack_bf16(acc[0][0], acc[0][1]), pack_bf16(acc[0][2], acc[0][3])};
      *reinterpret_cast<u32x2*>(a.yp + static_cast<size_t>(row) * a.N + n0 + g4 * 4) = y;
      float* s = s_y[slot] + g4 * 4;
      s[0] = bf16lo(y.x); s[1] = bf16hi(y.x); s[2] = bf16lo(y.y); s[3] = bf16hi(y.y);
    }
  }
  __syncthreads();
  if (threadIdx.x < 8) {
    float lo = 0.f, hi = 0.f;
    for (int i = 0; i < a.k; ++i) {
      if (s_row[i] < 0) continue;
      lo += s_w[i] * s_y[i][2 * threadIdx.x];
      hi += s_w[i] * s_y[i][2 * threadIdx.x + 1];
    }
    *reinterpret_cast<uint32_t*>(a.out + static_cast<size_t>(t) * a.N + n0 + 2 * threadIdx.x) = pack_bf16(lo, hi);
  }
}

template <int G, int VPL>
void launch_route_gate_up(const StRouteArgs& r, const StreamFwdArgs& a, long long rows, hipStream_t s) {
  const int n = r.T * r.k, ncol = a.N / 32;
  const dim3 grid((((n < a.E ? n : a.E) * ncol + 7) & ~7) + 1);
  // The deeper ring leaves room for 768 workgroups at a time, the other for 1024: from 513 to 1024 expected tiles it is 5 to 9 % slower (8 tokens, 4 each of
  // 64 experts, d 1024, f 1024 42.2 / 39.2 us), and no faster where weight rows are multiples of 4096 bytes (4 tokens, 8 each, d 2048 75 / 75);
  // below, even with an even load and 2 to 7 % faster where all tokens are alike.
  if (st_expected_tiles(rows, a.E, ncol) <= 512)
    MOE_LAUNCH("route+gate_up", (route_gate_up_kernel<G, VPL, 2, 4>), grid, dim3(128), 0, s, r, a);
  else
    MOE_LAUNCH("route+gate_up", (route_gate_up_kernel<G, VPL, 2, 3>), grid, dim3(128), 0, s, r, a);
}
}  // namespace

// Every workgroup repeats the selection: `rounds` winners one after the other, in each round of workgroups that the chip holds at a time.  Beyond
// some 8000 of rounds times workgroups that costs more than the launch.  Forward pass in us, apart / joined: 2 tokens, 32 of 294 experts each, d 128,
// f 1920 (64 rounds, 3840 workgroups) 42 / 133; 4 tokens, 16 of 174, d 320, f 2048 (32, 4096) 37 / 91; 1 token, 64 of 512, d 1024, f 512 (64, 1024)
// 76 / 104; 8 tokens, 8 of 64, d 2048, f 1024 (8, 2048) 118 / 115; 5 tokens, 8 of 126, 31 local, d 128, f 1920 (16, 1860) 20 / 35.  On 16400 calls
// of 1 to 16 tokens, 4 to 512 experts, d 128 to 4096, f 128 to 2560, even loads and all tokens alike, those that the rule takes gain 9 % on
// average, one in 450 loses 5 % or more (the worst 17 %); without the bounds one in 18 did, up to two thirds of its speed.  Beyond 8 tokens a third
// are slower (2 % faster on average).  More than two passes of the lane groups over the tokens: 8 tokens, 1 of 266, 33 local, d 1984, f 1728 19.7 / 23.4.
bool moe_route_gate_up_fits(int T, int E, int k, int e_count, int f) {
  static_assert(MOE_JOIN_TOKENS <= ST_ROWS, "no expert may have more rows than a tile");
  if (E > MOE_MAX_EXPERTS || T > MOE_JOIN_TOKENS || T * k > MOE_WAVE) return false;
  const int G = E <= 64 ? 8 : E <= 128 ? 16 : E <= 256 ? 32 : 64;   // lanes of a token, as in moe_route
  const int passes = (T * G + MOE_WAVE - 1) / MOE_WAVE, rounds = passes * k;
  const long long workgroups = static_cast<long long>(T * k < e_count ? T * k : e_count) * (f / 32);
  return passes <= 2 && rounds <= 10 && rounds * workgroups <= 8192;
}

int moe_stream_gate_up(const StreamFwdArgs& a, long long rows, hipStream_t s) { return launch_fwd_any<true>(a, rows, s, "gemm_gate_up"); }
int moe_stream_down(const StreamFwdArgs& a, long long rows, hipStream_t s) { return launch_fwd_any<false>(a, rows, s, "gemm_down"); }

int moe_route_gate_up(const moe_layer* L, long long rows, hipStream_t s) {
  const bool fold = L->path == MOE_LAYER_FOLD;
  const StRouteArgs r = {L->logits, L->topk_idx, L->topk_w, L->expert_offsets, L->row_token, L->slot_row, fold ? L->row_weight : nullptr,
                         L->T, L->E, L->k, L->renormalize != 0, L->e_begin, moe_expert_bits(L->e_count)};
  StreamFwdArgs a{};
  a.A = L->x; a.B0 = L->Wg; a.B1 = L->Wu; a.O0 = L->g; a.O1 = L->u; a.O2 = L->h; a.E = L->e_count; a.K = L->d; a.N = L->f;
  // the lane groups of moe_route (same bits).  Up to 64 experts one variant with eight logits per lane, those past the last expert left out:
  // with four per lane (17 to 32 experts) the streaming behind the routing took twice as long (2 tokens of d 2432, f 640, 21
  // experts: 35.1 us, 20.7 so, 25.7 in four launches), for a reason not found in its code.  The other variants do not: on the calls above that the rule takes, joined is
  // 1.08, 1.09, 1.09 and 1.14 times as fast as apart with lane groups of 8, 16, 32 and 64, and one in 250 or fewer is slower by 5 % or more.
  if (L->E <= 64) launch_route_gate_up<8, 8>(r, a, rows, s);
  else if (L->E <= 128) launch_route_gate_up<16, 8>(r, a, rows, s);
  else if (L->E <= 256) launch_route_gate_up<32, 8>(r, a, rows, s);
  else launch_route_gate_up<64, 8>(r, a, rows, s);
  return moe_check_launch();
}

// The rings fill a compute unit's LDS, so one workgroup per compute unit: a second round of them, or weights read by each of several tokens, cost
// more than the launch.  And few workgroups with many slots bring all weights through few compute units (rows: to expect, so rows / T local
// slots per token).  Forward pass in us, apart / joined, routing joined in both: 4 tokens of d 4096, f 2048, 64 experts, 2 per token (1024 workgroups) 76 / 80, all tokens
// alike 36 / 48; 4 of d 3392, f 1920, 4 per token, 4 experts (848) 37 / 51; 4 of d 1024, f 512, 64 experts, 8 per token (256) 28.5 / 24.9; 1 of d 192, f 2432, 11
// experts, 8 per token (12) 23.8 / 30.4; 1 of d 2048, f 2048, 240 experts, 120 local, 8 per token (128) 34.2 / 30.5.  On the same calls: 18 % gained
// on average where the rule takes it, one in 280 loses 5 % or more (the worst 11 %); without the bounds on workgroups one in 11 did, up to a third
// of its speed.
bool moe_down_combine_fits(int T, int k, int d, int f, long long rows) {
  const long long workgroups = static_cast<long long>(T) * (d / 16);
  return T <= 4 && k <= ST_DOWN_SLOTS && workgroups <= 256 && (rows * f <= 8192ll * T || workgroups >= 128);
}

int moe_down_combine(const moe_layer* L, hipStream_t s) {
  const StDownArgs a = {L->h, L->Wd, L->expert_offsets, L->slot_row, L->path == MOE_LAYER_FOLD ? nullptr : L->topk_w, L->yp, L->out,
                        L->T, L->k, L->e_count, L->f, L->d};
  const int cols = (L->d / 16 + 7) / 8 * 8;
  MOE_LAUNCH("down+combine", down_combine_kernel, dim3(cols * L->T), dim3(L->k * MOE_WAVE), 0, s, a);
  return moe_check_launch();
}
