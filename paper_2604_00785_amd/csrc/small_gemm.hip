// Grouped products for experts with few rows (a decoding step, a short prompt): what bounds them is the one pass
// over the weights of the experts that have rows, 2 bytes for at most 2 * 32 operations.  The tiled kernel of
// grouped_gemm.hip, made for many rows, has one workgroup per compute unit and spends as long between its tiles as
// they take to stream here; with one token its eight experts are 64 tiles for 256 compute units.
//
// Here a workgroup of four waves owns 64 weight rows (32 of Wg and the same 32 of Wu, or 64 of Wd) of one expert and
// its (up to) 16 or 32 activation rows, and the WAVES SPLIT THE REDUCTION: each streams its quarter of the weight
// rows from memory straight into registers in the layout of the matrix instruction and multiplies, with no LDS and
// no barrier in the loop; the four partial sums meet in LDS at the end and are added in wave order.  A weight byte
// passes through one wave of the chip once, three or four workgroups per compute unit overlap each other's start
// and end, and 8 experts are 256 workgroups.  Measured (d 2048, f 1024, 64 experts, 8 per token; gate/up and down,
// with the two events around them): one token 50 + 28 us in the tiled kernel, 17 + 12 us here; 16 tokens (56 experts, 470 +
// 235 MB) 129 + 62 -> 91 + 50 us, 5.2 and 4.7 TB/s; 48 tokens 127 + 64 -> 105 + 58 us.  Loading three or four blocks ahead
// instead of one was 5-8 % slower, non-temporal weight loads 10-20 %, five workgroups per compute unit (spills) 1.7x.
#include "small_gemm.h"

namespace {

constexpr int ST_THREADS = 256, ST_WAVES = 4;
constexpr int ST_KB = 64;             // reduction elements of a block: 128 bytes of a weight row

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

__device__ __forceinline__ float st_sigmoid(float g) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g));
}
__device__ __forceinline__ int st_incl_scan(int v, int lane) {
#pragma unroll
  for (int s = 1; s < 64; s <<= 1) {
    const int u = __shfl_up(v, s, 64);
    if (lane >= s) v += u;
  }
  return v;
}
__device__ __forceinline__ int sfirst(int v) { return __builtin_amdgcn_readfirstlane(v); }

struct StTile { int e, m0, m_end, col; };

// The tile of this workgroup: expert, rows, column tile; false if there are fewer tiles (the grid covers the most there
// can be).  An expert's tiles are numbered column tile by column tile, its row tiles innermost, and an XCD gets a run
// of consecutive numbers, so that row tiles that share weights share an L2.  Every wave looks its tile up by itself.
template <int ST_ROWS> __device__ __forceinline__ bool st_find_tile(const int32_t* __restrict__ offsets, int E, int ncol, StTile& t) {
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
      inc[c] = total + st_incl_scan((hi[c] - lo[c] + ST_ROWS - 1) / ST_ROWS, lane);
      total = __shfl(inc[c], 63, 64);
    }
  }
  total = sfirst(total) * ncol;
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
        const int r = sfirst(__shfl(rt, l, 64));
        const int in = q - sfirst(__shfl(excl, l, 64)) * ncol;
        t.col = in / r;
        t.m0 = sfirst(__shfl(lo[c], l, 64)) + (in - t.col * r) * ST_ROWS;
        t.m_end = sfirst(__shfl(hi[c], l, 64));
        return true;
      }
    }
  }
  return false;
}

// One tile of 16 MB rows.  Four weight fragments of 16 rows each: GATE_UP: 0, 1 = 32 rows of Wg, 2, 3 = the same rows of
// Wu.  Weight row and lane are matched so that a lane ends up with neighbouring output columns (16-byte stores).
// Blocks are loaded one ahead of their use; the last load of a wave repeats its last block (a cache hit), so that
// every step has the same number of loads in flight.
template <bool GATE_UP, int MB>
__device__ __forceinline__ void st_fwd_tile(const StreamFwdArgs& a, const StTile& t, f32x4_t* part) {
  constexpr int NB = 4;
  constexpr int DEPTH = 2;
  constexpr int NBC = GATE_UP ? 2 : 4;                  // fragments per tensor; a lane ends up with 4 * NBC columns
  const int tid = threadIdx.x, lane = tid & 63, wave = sfirst(tid >> 6);
  const int i16 = lane & 15, g4 = lane >> 4;
  const int K = a.K;
  const int n0 = t.col * (16 * NBC);
  const int nb = K / ST_KB;
  const int b0 = nb * wave / ST_WAVES, b1 = nb * (wave + 1) / ST_WAVES;

  f32x4_t acc[MB][NB];
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[m][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  if (b0 < b1) {
    // weights: fragment j, lane i16 -> output column n0 + (i16 / 4) * 4 NBC + 4 j + i16 % 4
    const size_t woff = (static_cast<size_t>(t.e) * a.N + n0) * K;
    const char* wb[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j)
      wb[j] = reinterpret_cast<const char*>((GATE_UP && j >= NBC ? a.B1 : a.B0) + woff + static_cast<size_t>(4 * (j % NBC)) * K);
    const uint32_t wl = static_cast<uint32_t>((((i16 >> 2) * 4 * NBC + (i16 & 3)) * K) * 2 + g4 * 16);
    uint32_t al[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) {
      int r = t.m0 + m * 16 + i16;
      if (r > t.m_end - 1) r = t.m_end - 1;
      const uint32_t row = a.row_token != nullptr ? static_cast<uint32_t>(a.row_token[r]) : static_cast<uint32_t>(r);
      al[m] = (a.row_token != nullptr ? row : static_cast<uint32_t>(r - t.m0)) * static_cast<uint32_t>(K) * 2u + g4 * 16;
    }
    const char* ab = reinterpret_cast<const char*>(a.A + (a.row_token != nullptr ? 0 : static_cast<size_t>(t.m0) * K));

    bf16x8_t w[DEPTH][NB][2], x[DEPTH][MB][2];
    auto load = [&](int s, int kb) __attribute__((always_inline)) {
      kb = kb < b1 ? kb : b1 - 1;
      const size_t ko = static_cast<size_t>(kb) * (ST_KB * 2);
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int h = 0; h < 2; ++h) w[s][j][h] = *reinterpret_cast<const bf16x8_t*>(wb[j] + ko + h * 64 + wl);
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int h = 0; h < 2; ++h) x[s][m][h] = *reinterpret_cast<const bf16x8_t*>(ab + ko + h * 64 + al[m]);
    };
#pragma unroll
    for (int s = 0; s < DEPTH - 1; ++s) load(s, b0 + s);
    for (int kb = b0; kb < b1; kb += DEPTH) {
#pragma unroll
      for (int s = 0; s < DEPTH; ++s) {
        if (kb + s >= b1) break;
        load((s + DEPTH - 1) % DEPTH, kb + s + DEPTH - 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int j = 0; j < NB; ++j)
              acc[m][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[s][j][h], x[s][m][h], acc[m][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  // the waves' partial sums meet in LDS and are added in wave order
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int j = 0; j < NB; ++j) part[((wave * MB + m) * NB + j) * 64 + lane] = acc[m][j];
  __syncthreads();
  if (wave < MB) {
    const int m = wave;
    f32x4_t v[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      v[j] = part[(m * NB + j) * 64 + lane];
#pragma unroll
      for (int u = 1; u < ST_WAVES; ++u) v[j] += part[((u * MB + m) * NB + j) * 64 + lane];
    }
    const int r = t.m0 + m * 16 + i16;
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

template <bool GATE_UP, int MB>
__global__ __launch_bounds__(ST_THREADS, MB == 1 ? 4 : 3) void stream_fwd_kernel(StreamFwdArgs a) {
  __shared__ f32x4_t part[ST_WAVES * MB * 4 * 64];
  StTile t;
  if (!st_find_tile<16 * MB>(a.offsets, a.E, a.N / (GATE_UP ? 32 : 64), t)) return;
  st_fwd_tile<GATE_UP, MB>(a, t, part);
}

template <bool GATE_UP, int MB>
int launch_fwd(const StreamFwdArgs& a, int R_cap, hipStream_t s, const char* name) {
  const int ncol = a.N / (GATE_UP ? 32 : 64);
  const long long row_tiles = R_cap / (16 * MB) + (a.E < R_cap ? a.E : R_cap);
  const long long tiles = (row_tiles * ncol + 7) & ~7ll;
  if (tiles > 0x7FFFFFFFll) return MOE_ERR_INVALID;
  MOE_LAUNCH(name, (stream_fwd_kernel<GATE_UP, MB>), dim3(static_cast<unsigned>(tiles)), dim3(ST_THREADS), 0, s, a);
  return moe_check_launch();
}
// 16-row tiles up to 8 rows per expert on average (few experts then have more than 16), 32-row tiles beyond: with
// 12 rows per expert 16-row tiles would read every other expert's weights twice.
template <bool GATE_UP>
int launch_fwd_any(const StreamFwdArgs& a, int R_cap, long long rows, hipStream_t s, const char* name) {
  if (rows <= 8ll * a.E) return launch_fwd<GATE_UP, 1>(a, R_cap, s, name);
  return launch_fwd<GATE_UP, 2>(a, R_cap, s, name);
}

}  // namespace

int moe_stream_gate_up(const StreamFwdArgs& a, int R_cap, long long rows, hipStream_t s) { return launch_fwd_any<true>(a, R_cap, rows, s, "gemm_gate_up"); }
int moe_stream_down(const StreamFwdArgs& a, int R_cap, long long rows, hipStream_t s) { return launch_fwd_any<false>(a, R_cap, rows, s, "gemm_down"); }
