// Grouped products for experts with few rows (a decoding step, a short prompt): what bounds them is the one pass
// over the weights of the experts that have rows, 2 bytes for at most 2 * 16 operations.  The tiled kernel of
// grouped_gemm.hip, made for many rows, has one workgroup per compute unit and spends as long between its tiles as
// they take to stream here; with one token its eight experts are 64 tiles for 256 compute units.
//
// Here a workgroup owns 64 weight rows (32 of Wg and the same 32 of Wu, or 64 of Wd) of one expert and up to 16 activation
// rows.  Each wave streams its FR fragments of 16 weight rows from memory straight into registers in the layout of the
// matrix instruction and multiplies, with no LDS and no barrier in the loop: FR = 4 is one wave for the whole tile, FR = 2
// two waves that share it (and load the activations twice).  A weight byte passes through one wave of the chip once, up to
// sixteen waves per compute unit overlap each other's start and end, and 8 experts are 256 workgroups.
//
// A wave takes the WHOLE reduction in its order and so gives the bits of the tiled kernel: a row's result does not depend
// on how many rows the call has.  Splitting the reduction over four waves rounds differently; it was 2-6 % faster at 8 to 32
// tokens of d 2048, f 1024, 64 experts, 10 % with 8 experts of d 4096, and up to 15 % slower elsewhere (narrow experts,
// skewed loads).  Loads three blocks deep instead of two were 1-10 % slower.
// Measured, whole forward pass, other weights in every pass, tiled kernel -> here: d 2048, f 1024, 64 experts, 8 per token: one
// token 79 -> 36 us; 16 tokens (59 experts, 740 MB of weights) 173 -> 153 us; 48 tokens 184 -> 171 us, 4.7 TB/s with routing
// and combine.  d 1088, f 576, 96 experts, 4 per token: 24 tokens 94 -> 64 us.
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

// One tile.  Its 64 weight rows are four fragments of 16 (GATE_UP: 0, 1 = 32 rows of Wg, 2, 3 = the same rows of Wu), FR of them
// to a wave.  Weight row and lane are matched so that a lane of the epilogue ends up with neighbouring output columns
// (16-byte stores).  Blocks of PIECES pieces are loaded one ahead of their use; loads past the end repeat the last piece (a
// cache hit), so that every step has the same number of loads in flight.
template <bool GATE_UP, int FR, int PIECES>
__device__ __forceinline__ void st_fwd_tile(const StreamFwdArgs& a, const StTile& t, f32x4_t* part) {
  constexpr int NB = 4, DEPTH = 2;
  constexpr int NBC = GATE_UP ? 2 : 4;                  // fragments per tensor; a lane ends up with 4 * NBC columns
  const int tid = threadIdx.x, lane = tid & 63, wave = sfirst(tid >> 6);
  const int i16 = lane & 15, g4 = lane >> 4;
  const int K = a.K;
  const int n0 = t.col * (16 * NBC);
  const int np = K / ST_KB, nb = (np + PIECES - 1) / PIECES, first = first_k_step(t.e, K);

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
  const uint32_t wl = static_cast<uint32_t>((((i16 >> 2) * 4 * NBC + (i16 & 3)) * K) * 2 + g4 * 16);
  int r = t.m0 + i16;
  if (r > t.m_end - 1) r = t.m_end - 1;
  const uint32_t row = a.row_token != nullptr ? static_cast<uint32_t>(a.row_token[r]) : static_cast<uint32_t>(r - t.m0);
  const uint32_t al = row * static_cast<uint32_t>(K) * 2u + g4 * 16;
  const char* ab = reinterpret_cast<const char*>(a.A + (a.row_token != nullptr ? 0 : static_cast<size_t>(t.m0) * K));

  bf16x8_t w[DEPTH][FR][2 * PIECES], x[DEPTH][2 * PIECES];
  auto load = [&](int s, int kb) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < PIECES; ++q) {
      int p = kb * PIECES + q;
      p = first + (p < np ? p : np - 1);
      const size_t ko = static_cast<size_t>(p < np ? p : p - np) * (ST_KB * 2);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int j = 0; j < FR; ++j) w[s][j][2 * q + h] = *reinterpret_cast<const bf16x8_t*>(wb[j] + ko + h * 64 + wl);
        x[s][2 * q + h] = *reinterpret_cast<const bf16x8_t*>(ab + ko + h * 64 + al);
      }
    }
  };
#pragma unroll
  for (int s = 0; s < DEPTH - 1; ++s) load(s, s);
  for (int kb = 0; kb < nb; kb += DEPTH) {
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) {
      if (kb + s >= nb) break;
      load((s + DEPTH - 1) % DEPTH, kb + s + DEPTH - 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < PIECES; ++q) {
        if (q > 0 && (kb + s) * PIECES + q >= np) break;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int j = 0; j < FR; ++j)
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[s][j][2 * q + h], x[s][2 * q + h], acc[j], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // the fragments' sums meet in LDS, where a lane of the epilogue finds its neighbouring columns
#pragma unroll
  for (int j = 0; j < FR; ++j) part[(wave * FR + j) * 64 + lane] = acc[j];
  __syncthreads();
  if (wave == 0) {
    f32x4_t v[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) v[j] = part[j * 64 + lane];
    r = t.m0 + i16;
    if (r < t.m_end) {
      const size_t o = static_cast<size_t>(r) * a.N + n0 + g4 * 4 * NBC;
      auto put8 = [&](uint16_t* p, const f32x4_t& lo, const f32x4_t& hi) __attribute__((always_inline)) {
        *reinterpret_cast<u32x4*>(p) = u32x4{pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3]), pack_bf16(hi[0], hi[1]), pack_bf16(hi[2], hi[3])};
      };
      if constexpr (GATE_UP) {
        const float rw = a.row_weight != nullptr ? a.row_weight[r] : 1.f;
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

template <bool GATE_UP, int FR, int PIECES>
__global__ __launch_bounds__(256 / FR, 4) void stream_fwd_kernel(StreamFwdArgs a) {
  __shared__ f32x4_t part[4 * 64];
  const int rows = a.offsets[a.E];
  StTile t;
  if (!st_find_tile(a.offsets, a.E, a.N / (GATE_UP ? 32 : 64), t) || rows > a.max_rows) return;
  st_fwd_tile<GATE_UP, FR, PIECES>(a, t, part);
}

template <bool GATE_UP, int FR, int PIECES>
int launch_fwd(const StreamFwdArgs& a, hipStream_t s, const char* name) {
  const int ncol = a.N / (GATE_UP ? 32 : 64);
  const long long row_tiles = a.max_rows / ST_ROWS + (a.E < a.max_rows ? a.E : a.max_rows);
  const long long tiles = (row_tiles * ncol + 7) & ~7ll;
  if (tiles > 0x7FFFFFFFll) return MOE_ERR_INVALID;
  MOE_LAUNCH(name, (stream_fwd_kernel<GATE_UP, FR, PIECES>), dim3(static_cast<unsigned>(tiles)), dim3(256 / FR), 0, s, a);
  return moe_check_launch();
}
// What is left of a wave's loads in flight decides: with fewer tiles than the 256 compute units two waves per tile with blocks of
// 128 elements, up to about two tiles per compute unit two waves with blocks of 64, beyond one wave.  Under an even load
// rows * E / (rows + E) experts, roughly, have a row.  Forward pass in us, in that order of variants:
//   96 tiles (one token, d 4096, f 1536) 40 / 52 / 60; 256 tiles (one token over eight experts of d 2048) 36 / 41 / 45
//   384 tiles (d 4096) 72 / 66 / 77; 512 tiles (two tokens, d 2048) 56 / 53 / 58
//   1130 tiles (d 1088, 24 tokens) 67 / 64 / 64; 2050 tiles (64 tokens, d 2048) 186 / 179 / 172
template <bool GATE_UP>
int launch_fwd_any(const StreamFwdArgs& a, long long rows, hipStream_t s, const char* name) {
  const long long tiles = rows * a.E / (rows + a.E) * (a.N / (GATE_UP ? 32 : 64));
  if (tiles < 256) return launch_fwd<GATE_UP, 2, 2>(a, s, name);
  if (tiles <= 512) return launch_fwd<GATE_UP, 2, 1>(a, s, name);
  return launch_fwd<GATE_UP, 4, 1>(a, s, name);
}

}  // namespace

int moe_stream_gate_up(const StreamFwdArgs& a, long long rows, hipStream_t s) { return launch_fwd_any<true>(a, rows, s, "gemm_gate_up"); }
int moe_stream_down(const StreamFwdArgs& a, long long rows, hipStream_t s) { return launch_fwd_any<false>(a, rows, s, "gemm_down"); }
