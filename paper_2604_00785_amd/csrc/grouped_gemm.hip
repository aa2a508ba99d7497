// Stage 4 of Algorithm 1 (the three Grouped_mm calls around Silu(gate)*up) and
// its derivative, as grouped bf16 MFMA GEMMs: one launch covers every expert.
//
// One workgroup of FOUR waves (one per SIMD, 512 registers each) computes one 256x256 output tile
// with a 64-deep K step; the waves form a 2 x 2 grid and each owns a 128x128 piece = 8x8
// v_mfma_f32_16x16x32_bf16 accumulators, which live in the 256 accumulation registers.  Against
// eight waves with 128x64 pieces this reads a third less operand data out of LDS per FLOP, and the
// 16x16x32 form draws less power per FLOP than the 32x32x16 form (the chip is power-limited on
// real data), but with one wave per SIMD nothing covers a wave's own stalls, so the main loop is
// written instruction by instruction:
//   * MFMAs, LDS fragment reads and direct-to-LDS loads are inline assembly in program order; the
//     accumulators are pinned to accumulation registers, so the compiler has nothing to move;
//   * between two MFMAs there is at most one other instruction (a fragment read, or a load);
//   * no vector-ALU instruction and no branch inside a K step: loads use a scalar base that is
//     advanced by scalar adds plus a 32-bit lane offset computed once per tile; the eight loads a
//     wave issues per operand tile share one M0 value (the instruction's immediate offset moves
//     the LDS address; the lane offset takes the same amount out of the global address again);
//   * the last three K steps of a tile (the last one that loads, which is the one that may load a
//     partial step of a weight gradient; the one that only awaits; the last one) are separate copies
//     of the step, and a tile enters the ring of LDS slots at the phase that puts those three on
//     phases 0, 1 and 2.
//
// The whole of it exists a second time with tiles of 128x128: four waves of 64x64 pieces = 4x4 accumulators, 80 KB of LDS and
// less than 256 registers, so that two workgroups share a compute unit.  The sums run in the same order and give the same
// bits; which size a launch takes is a rule on its expected tiles (TileCost).  What is said here in numbers is about the large tiles.
//
// The two operand tiles of a step (32 KB each) live in a ring of five LDS slots (160 KB, all
// there is): A(t) in slot 2t mod 5, B(t) in slot (2t+1) mod 5, so two and a half steps are
// resident (a small tile that holds all of an expert's few rows has a ring of its own, see few_rows_loop).
// Step t loads A(t+2) during its first 32-deep sub-step, into the slot B(t-1) left;
// its barrier follows that sub-step: behind it the tiles of step t+1 are complete (the wave's own
// loads of A(t+2) may still be in flight) and every wave is done with A(t), whose slot B(t+2) is
// loaded into during the second sub-step.  Fragments are double-buffered in registers: the reads
// of the next sub-step are issued between the MFMAs of the current one.
//
// Tile layouts.  An operand that is contiguous along K in memory (activations [rows, K],
// forward weights [N, K]) is kept as [256 rows][64 k] with 128-byte rows whose eight 16-byte
// pieces are rotated by the row (fragment = one ds_read_b128 per lane); the swizzle is
// applied on the global side of the fill, since a direct-to-LDS load writes LDS linearly.  An
// operand that is contiguous along its other dimension (weights in dgrad, both operands in
// wgrad) is kept as it lies in memory, [64 k][256 n] with 512-byte rows, and read with the
// transposing LDS load ds_read_b64_tr_b16, two per fragment (it moves half the bytes per cycle
// of ds_read_b128, which makes the weight gradients LDS-bound).
//
// The MFMAs are issued as (weight fragment) x (activation fragment), so a lane ends up with
// four consecutive output COLUMNS of one row.  The epilogue reads the accumulators by hand, rounds
// to bf16, stages 16 or 32 rows of the wave's 128x128 piece at a time in the wave's own 8 KB of LDS
// and writes them out in full 256-byte row segments; the SwiGLU forward and backward formulas are
// applied on the way, on the fp32 accumulators.
//
// Tiles of the row-grouped products are found on the device from expert_offsets: every wave
// turns the tile number into (expert, first row, column tile); inside an expert the row tiles are
// innermost; experts without rows own no tile; rows past an expert's end are clamped on load and
// dropped on store by the range check of buffer resources, and 32-row groups without a valid row issue no MFMA.
#include <climits>
#include <type_traits>
#include <utility>
#include "common.h"
#include "dma.h"
#include "gemm.h"
#include "small_gemm.h"

namespace {

constexpr int BK = 64;
constexpr int GEMM_THREADS = 256;
constexpr int NSLOT = 5;                              // ring of operand tile slots
// What follows from the edge S of the output tile, 256 or 128 (see TileCost).  Four waves as 2 x 2 in either case.
template <int S> struct Tile {
  static_assert(S == 256 || S == 128);
  static constexpr int BYTES = S * BK * 2;            // one operand tile: 32 or 16 KB
  static constexpr int LDS = NSLOT * BYTES;           // 160 KB, everything a compute unit has; or 80 KB, two workgroups on it
  static constexpr int PER_CU = 256 / S;              // workgroups per compute unit
  static constexpr int HALF = S / 2;                  // rows and columns of a wave's piece
  static constexpr int NB = S / 32;                   // 16 x 16 blocks along each side of it
  static constexpr int NL = S / 32;                   // direct-to-LDS loads (1 KB each) per wave and operand tile
  static constexpr int SHARE = BYTES / 4;             // a wave's share of a slot: what it fills, and stages in
  static constexpr int KN_ROW = S * 2;                // bytes of a row of a [64 k][S n] tile
  static constexpr int KN_PIECES = S / 8;             // 16-byte pieces of it
  static constexpr int KN_RPL = 64 / KN_PIECES;       // rows of it that one load fills
  static constexpr int SLOTS_PER_SET = 65536 / BYTES; // slots that an LDS read's immediate offset reaches
  static constexpr int SETS = (NSLOT + SLOTS_PER_SET - 1) / SLOTS_PER_SET;
};
// few_rows_loop: up to 64 rows, RING steps of one 16 KB slot for B and 8 KB for A behind the B slots
constexpr int FEW_ROWS = 64, FEW_RING = 3, FEW_A_BYTES = FEW_ROWS * BK * 2;
static_assert(FEW_RING * (Tile<128>::BYTES + FEW_A_BYTES) <= Tile<128>::LDS);
constexpr int LOAD_BIAS = 4096;                       // see dma16_imm
constexpr int slot_of_a(int p) { return (2 * p) % NSLOT; }       // p = ring phase of the step
constexpr int slot_of_b(int p) { return (2 * p + 1) % NSLOT; }

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef short s16x4 __attribute__((ext_vector_type(4)));

template <int N> using IC = std::integral_constant<int, N>;
template <typename F, int... I> __device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(IC<I>{}), ...);
}
template <int N, typename F> __device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(static_cast<F&&>(f), std::make_integer_sequence<int, N>{});
}

enum GemmMode { GATE_UP = 0, DOWN = 1, DGRAD_H = 2, DGRAD_X = 3, WGRAD = 4, WGRAD_GATHER = 5, DGRAD_H_GATE = 6,
                WGRAD_GATHER_A = 7 };
// WGRAD_GATHER / WGRAD_GATHER_A: a weight gradient whose B / A operand rows are token rows found through
// row_token.  DGRAD_H_GATE: DGRAD_H for a forward pass that folded the gate weight into h: its A rows are
// rows of dout found through row_token, its epilogue scales by the row's gate weight and also emits the
// row's partial dot product with h = silu(g) u (the gradient of the gate weight).
constexpr bool is_wgrad(int mode) { return mode == WGRAD || mode == WGRAD_GATHER || mode == WGRAD_GATHER_A; }
constexpr bool is_dgrad_h(int mode) { return mode == DGRAD_H || mode == DGRAD_H_GATE; }

struct GemmArgs {
  // row-grouped products (modes 0-3, 6)
  const uint16_t* A0;   // [R_cap, K]   activations (phase 0)
  const uint16_t* A1;   // second K phase of DGRAD_X (du), else unused
  const uint16_t* B0;   // weights, stacked over experts
  const uint16_t* B1;   // Wu (GATE_UP: the up half of the column tile; DGRAD_X: second K phase)
  const uint16_t* G;    // DGRAD_H epilogue inputs
  const uint16_t* U;
  uint16_t* O0;         // g | yp | dg | dxp | dW
  uint16_t* O1;         // u | du
  uint16_t* O2;         // h
  const int32_t* offsets;
  const int32_t* row_token;   // not null: rows of the activation operand are gathered, row r lies at A0[row_token[r]]
                              // (GATE_UP, DGRAD_H_GATE, WGRAD_GATHER_A: the A operand; WGRAD_GATHER: the B operand)
  const float* row_weight;    // GATE_UP: not null = h is scaled by the row's gate weight; DGRAD_H_GATE: required
  float* dgate_part;          // DGRAD_H_GATE: [R_cap][N / 64] partial dot products, one per row and 64-column strip
  int E;
  int K;                // reduction length of one phase (row-grouped products)
  int N;                // output columns (per half for GATE_UP)
  int n_tiles;          // column tiles
  int m_tiles_cap;      // upper bound on row tiles (row-grouped products); row tiles of one dW (WGRAD)
  int stream_rows;      // GATE_UP, DOWN: nothing is done where there are at most this many rows (0: always): a launch of
                        // the streaming kernel in front has done it
  // WGRAD: out[e][M][N] = sum over the expert's rows of A[r][M] * B[r][N]
  int M;
};

// 512 bytes of zeros: what the reduction rows past an expert's end read in the weight-gradient products.
__device__ __attribute__((aligned(512))) uint32_t g_zero_block[128];

// [256 rows][64 k] tile, 128-byte rows: the 16-byte piece `logical` (0..7) of `row` lies at physical piece
// (logical + row) mod 8.  A fragment read (16 rows x 4 neighbouring pieces per instruction) then costs 8.5
// cycles per CU, as a linear read does; XOR-ing the piece with (row ^ row >> 3) & 7 costs 8.9, no swizzle 16.
// This is the inverse: which logical piece a fill has to fetch for physical piece `phys`.
__device__ __forceinline__ int kc_logical_piece(int row, int phys) { return (phys - row) & 7; }
// [64 k][S n] tile: 16-byte pieces of a k row are XOR-swizzled with 4*(k & 3), which spreads the
// four k rows that 16 lanes of a transposing read touch over four different 64-byte bank groups.
__device__ __forceinline__ int kn_piece(int krow, int piece) { return piece ^ ((krow & 3) << 2); }

// Everything the main loop issues is inline assembly in program order (asm volatile statements keep
// their order), with immediate offsets, and is awaited by hand: fragments are read one sub-step
// ahead and loads several steps ahead, which the compiler's own wait insertion cannot express.
template <int OFF> __device__ __forceinline__ bf16x8_t lds_read_b128(uint32_t addr) {
  bf16x8_t v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
  return v;
}
template <int OFF> __device__ __forceinline__ s16x4 lds_read_tr_b64(uint32_t addr) {
  s16x4 v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
  return v;
}
// Direct-to-LDS loads, 16 bytes per lane: lane l lands at M0 + OFF + 16 l, and reads global address
// (scalar base) + (32-bit lane offset) + OFF.  The immediate moves both addresses: a wave's eight loads
// of a tile use OFF = (i - 4) * 1024 with one M0 value, their lane offsets carry -OFF, and LOAD_BIAS
// (subtracted from the scalar base, added to every lane offset) keeps the lane offsets non-negative.
// Nothing else in this file uses M0.
template <int OFF> __device__ __forceinline__ void set_m0(uint32_t lds_base) {
  asm volatile("s_add_i32 m0, %0, %1" :: "s"(lds_base), "n"(OFF) : "memory", "scc");
}
// the same with a 64-bit address per lane (used once per tile at most, for rows past an expert's end)
template <int OFF> __device__ __forceinline__ void dma16_lane_imm(const char* p) {
  asm volatile("global_load_lds_dwordx4 %0, off offset:%1" :: "v"(p), "n"(OFF) : "memory");
}
// A 4-byte load as (scalar base) + (32-bit lane offset) + immediate, awaited by hand like the loads above.
template <int OFF> __device__ __forceinline__ int load_i32(uint32_t voff, const int32_t* sbase) {
  int v;
  asm volatile("global_load_dword %0, %1, %2 offset:%3" : "=v"(v) : "v"(voff), "s"(sbase), "n"(OFF) : "memory");
  return v;
}
__device__ __forceinline__ void wg_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
}

// A fragment of a [64 k][256 n] tile: two transposing reads (k rows +0..3 and +4..7 of the lane's column).
union KnFrag {
  s16x4 h[2];
  bf16x8_t v;
};

// sigmoid through the hardware exp2 and reciprocal (each about 1 ulp): far inside bf16 rounding.
// exp2 overflows to +inf for very negative g and the reciprocal then returns 0, as it should.
__device__ __forceinline__ float sigmoid_f(float g) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g));
}
__device__ __forceinline__ float silu_f(float g) { return g * sigmoid_f(g); }

// Row tiles of the grouped products: expert e owns ceil(rows_e / S) consecutive tile numbers (S: the tile's edge).
// Both functions are evaluated by a whole wave (64 experts per pass) and return wave-uniform values.
template <int S> __device__ __forceinline__ int count_row_tiles(const int32_t* offsets, int E, int lane) {
  int total = 0;
  for (int e0 = 0; e0 < E; e0 += 64) {
    const int ee = e0 + lane;
    const int rows = ee < E ? offsets[ee + 1] - offsets[ee] : 0;
    total += wave_lane(wave_incl_scan((rows + S - 1) / S), 63);
  }
  return total;
}
// Tile number `tile` of a row-grouped product -> expert, first row, column tile.  An expert's tiles are
// numbered column tile by column tile, its row tiles innermost: the workgroups of an XCD, which take a
// run of consecutive tiles, then share each weight panel among all row tiles of the expert at the same
// time, so that it is fetched from memory once (weights are the larger operand and are used by only
// rows_e / 256 tiles each; activations of a row tile recur every rows_e / 256 tiles).
//
// With at most 128 experts (two per lane) the experts are not listed in index order: those whose tile count
// is a whole number of XCD runs come first, then those that fill half a run, then the rest.  The first
// two groups then start on run boundaries, so such an expert's tiles are worked on by one XCD at one
// time and its activation rows are fetched into one L2 once; an expert that straddles two runs has its
// rows fetched by both.  The lane keeps its expert's row range and first list position for the whole
// kernel, so the lookup needs no memory access (which would otherwise sit in front of every tile's
// first loads) and no scan.
// (kept as six plain registers: a struct of arrays behind a reference ends up in scratch memory)
__device__ __forceinline__ void sorted_first_tiles(int tiles0, int tiles1, int run, int& first0, int& first1) {
  const int r0 = tiles0 % run, r1 = tiles1 % run;
  const int cls0 = r0 == 0 ? 0 : (2 * r0 == run ? 1 : 2);
  const int cls1 = r1 == 0 ? 0 : (2 * r1 == run ? 1 : 2);
  int base = 0;
  first0 = 0;
  first1 = 0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const int mine0 = cls0 == c ? tiles0 : 0;
    const int inc0 = wave_incl_scan(mine0);
    if (cls0 == c) first0 = base + inc0 - mine0;
    base += wave_lane(inc0, 63);
    const int mine1 = cls1 == c ? tiles1 : 0;
    const int inc1 = wave_incl_scan(mine1);
    if (cls1 == c) first1 = base + inc1 - mine1;
    base += wave_lane(inc1, 63);
  }
}
constexpr int LANE_EXPERTS_MAX = 128;
// One half (experts 64 h .. 64 h + 63, one per lane) of the register-resident lookup.
template <int S>
__device__ __forceinline__ bool find_tile_half(int h, int lo, int hi, int first, int n_tiles, int tile, int& e, int& m0,
                                               int& m_end, int& nt, int& rt) {
  const int row_tiles = (hi - lo + S - 1) / S;
  const int tiles = row_tiles * n_tiles;
  const unsigned long long hit = __ballot(tiles > 0 && first <= tile && tile < first + tiles);
  if (!hit) return false;
  const int l = __ffsll(hit) - 1;
  e = h * 64 + l;
  const int q = tile - wave_lane(first, l);
  rt = wave_lane(row_tiles, l);
  nt = q / rt;
  m0 = wave_lane(lo, l) + (q - nt * rt) * S;
  m_end = wave_lane(hi, l);
  return true;
}
template <int S>
__device__ __forceinline__ void find_tile(const int32_t* offsets, int E, int lo0, int hi0, int first0, int lo1, int hi1,
                                          int first1, int n_tiles, int tile, int lane, int& e, int& m0, int& m_end, int& nt,
                                          int& rt) {
  e = 0; m0 = 0; m_end = 0; nt = 0; rt = 0;
  if (E <= LANE_EXPERTS_MAX) {
    if (find_tile_half<S>(0, lo0, hi0, first0, n_tiles, tile, e, m0, m_end, nt, rt)) return;
    find_tile_half<S>(1, lo1, hi1, first1, n_tiles, tile, e, m0, m_end, nt, rt);
    return;
  }
  int base = 0;
  for (int e0 = 0; e0 < E; e0 += 64) {
    const int ee = e0 + lane;
    const int lo = ee < E ? offsets[ee] : 0, hi = ee < E ? offsets[ee + 1] : 0;
    const int row_tiles = (hi - lo + S - 1) / S;
    const int tiles = row_tiles * n_tiles;
    const int inc = wave_incl_scan(tiles);
    const int excl = base + inc - tiles;
    const unsigned long long hit = __ballot(tiles > 0 && excl <= tile && tile < excl + tiles);
    if (hit) {
      const int l = __ffsll(hit) - 1;
      e = e0 + l;
      const int q = tile - wave_lane(excl, l);
      rt = wave_lane(row_tiles, l);
      nt = q / rt;
      m0 = wave_lane(lo, l) + (q - nt * rt) * S;
      m_end = wave_lane(hi, l);
      return;
    }
    base += wave_lane(inc, 63);
  }
}

// The kernel arguments again, through a pointer the compiler cannot see through: what is read from
// it is loaded afresh (scalar loads from the argument segment) instead of being kept in scalar
// registers across the main loop.
typedef const __attribute__((address_space(4))) GemmArgs* ArgPtr;
template <int ARG> __device__ __forceinline__ ArgPtr reload_args() {   // ARG: which of the kernel's GemmArgs
  ArgPtr p = (ArgPtr)__builtin_amdgcn_kernarg_segment_ptr() + ARG;
  asm volatile("" : "+s"(p));
  return p;
}

// A wave-uniform pointer as two scalar registers.  readfirstlane returns a signed int: it is widened
// through uint32_t, or a set bit 31 of the low half would smear into the high half.
__device__ __forceinline__ const char* scalarize(const char* p) {
  const uint64_t u = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(u)));
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(u >> 32)));
  return reinterpret_cast<const char*>((static_cast<uint64_t>(hi) << 32) | static_cast<uint64_t>(lo));
}

// What a workgroup knows about one tile: where it lies, where its operand loads come from, how many
// K steps it has.
template <int S>
struct TileState {
  int e, m0, m_end, nt, n0;     // expert, first output row, end of the valid rows, column tile, first output column
  int r0;                       // first of this wave's rows inside the tile
  int m_wave;                   // end of the valid rows that are this wave's
  int nv;                       // 32-row groups that every wave works on, 1 .. HALF / 32 (the others issue no load and no MFMA)
  bool few;                     // tiles of 128: takes few_rows_loop, whose ring lies across the slots of the other tiles and the shares of
                                // the waves: only in a list with no more tiles than workgroups, the first of its launch
  bool second;                  // tile of the second weight gradient of a pair
  int nk, nk_phase;             // K steps in total / in the first K phase
  int nmain, p0;                // steps in front of the last three; ring phase of step 0
  int k_lo, k_hi;               // weight gradients: the expert's row range is the reduction
  bool last_partial;            // weight gradients: the last step holds fewer than 64 rows
  uint32_t voa[Tile<S>::NL], vob[Tile<S>::NL];   // lane offsets of a wave's loads per operand tile, in bytes
  uint32_t vcb[Tile<S>::NL];    // gathered operand: lane offset of a load without its token row
  int tokn[Tile<S>::NL];        // gathered operand: tokens of the lane's reduction rows of a coming step
  const char* sa_next;          // scalar bases of the next A / B tile to load (LOAD_BIAS low)
  const char* sb_next;
  const char* sa_phase1;        // DGRAD_X: bases of the second K phase
  const char* sb_phase1;
  size_t a_step, b_step;        // bytes per step
  const int32_t* row_tok;       // gathered operand: token of the expert's first reduction row onwards
};

// One product's tile list, walked by this workgroup from list position first_tile in steps of
// gridDim.x.  Returns the position at which the workgroup left the list, counted from its end:
// where it enters a list that follows in the same launch.
template <int MODE, int S, int ARG>
__device__ __forceinline__ int gemm_tile_list(const GemmArgs& a, int first_tile) {
  using TL = Tile<S>;
  using TileState = TileState<S>;
  constexpr int NL = TL::NL, NB = TL::NB, HALF = TL::HALF, TILE_BYTES = TL::BYTES;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid0 = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid0 >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  constexpr bool A_KN = is_wgrad(MODE);                                           // stored [k][m]
  constexpr bool B_KN = (is_wgrad(MODE) || is_dgrad_h(MODE) || MODE == DGRAD_X);  // stored [k][n]
  constexpr bool GATHER_B = (MODE == WGRAD_GATHER);
  constexpr bool GATHER_A = (MODE == WGRAD_GATHER_A);

  // ---------------- tile list ---------------------------------------------------
  int total;
  // experts `lane` and `lane + 64`: row range and list position of the first tile, kept for the whole kernel
  // when E <= LANE_EXPERTS_MAX
  int lo0 = 0, hi0 = 0, first0 = 0, lo1 = 0, hi1 = 0, first1 = 0;
  // WGRAD / WGRAD_GATHER with a second A operand (A1 -> O1): two weight gradients that share their B
  // operand in one launch; an expert's tiles of the first come before its tiles of the second
  int wpair = 1;
  if constexpr (MODE == WGRAD_GATHER || MODE == WGRAD) wpair = a.A1 != nullptr ? 2 : 1;
  if constexpr (is_wgrad(MODE)) {
    total = a.E * a.m_tiles_cap * a.n_tiles * wpair;
  } else {
    total = count_row_tiles<S>(a.offsets, a.E, tid0 & 63) * a.n_tiles;
    if constexpr (MODE == GATE_UP || MODE == DOWN) {
      if (a.stream_rows > 0 && a.offsets[a.E] <= a.stream_rows) total = 0;
    }
    if (a.E <= LANE_EXPERTS_MAX) {
      const int e0 = tid0 & 63, e1 = 64 + (tid0 & 63);
      if (e0 < a.E) { lo0 = a.offsets[e0]; hi0 = a.offsets[e0 + 1]; }
      if (e1 < a.E) { lo1 = a.offsets[e1]; hi1 = a.offsets[e1 + 1]; }
      sorted_first_tiles((hi0 - lo0 + S - 1) / S * a.n_tiles, (hi1 - lo1 + S - 1) / S * a.n_tiles, gridDim.x >> 3, first0, first1);
    }
  }
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<size_t>(LDS_PTR(lds)));
  // M0 base of this wave's loads: the middle of its share of tile slot 0 (immediates reach -4096 .. +3072)
  const uint32_t lds_fill = __builtin_amdgcn_readfirstlane(lds0 + wave * TL::SHARE + NL / 2 * 1024);

  // few_rows_loop: the same for its A tiles, 2 KB of a wave each
  const uint32_t few_a = __builtin_amdgcn_readfirstlane(lds0 + FEW_RING * TILE_BYTES + wave * 2048 + NL / 2 * 1024);

  const int lane = tid0 & 63;
  // k row (of a [64 k][S n] tile) that load i of this wave fills from this lane
  auto kn_load_row = [&](int i, int lane) __attribute__((always_inline)) { return (wave * NL + i) * TL::KN_RPL + lane / TL::KN_PIECES; };
  // Everything about tile number `tile` of the list that does not depend on the K step.
  auto setup_tile = [&](int tile, TileState& t) __attribute__((always_inline)) {
  // the thread id is laundered per tile so that the lane-dependent pieces of the load offsets are recomputed for
  // every tile instead of staying live (and spilling) across the main loop
  int tid = tid0;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  int e, m0, m_end, nt, rt = 0;
  bool second = false;
  if constexpr (is_wgrad(MODE)) {
    nt = tile % a.n_tiles;
    const int rest = tile / a.n_tiles;
    const int per_expert = a.m_tiles_cap * wpair;
    e = rest / per_expert;
    int mi = rest % per_expert;
    if (mi >= a.m_tiles_cap) { mi -= a.m_tiles_cap; second = true; }
    m0 = mi * S;                        // output row of dW
    m_end = a.M;
  } else {
    find_tile<S>(a.offsets, a.E, lo0, hi0, first0, lo1, hi1, first1, a.n_tiles, tile, lane, e, m0, m_end, nt, rt);
    nt = __builtin_amdgcn_readfirstlane(nt);
  }
  // tile coordinates are wave-uniform: keep them in scalar registers, so that everything derived
  // from them (operand base addresses in particular) is scalar too
  e = __builtin_amdgcn_readfirstlane(e);
  m0 = __builtin_amdgcn_readfirstlane(m0);
  m_end = __builtin_amdgcn_readfirstlane(m_end);
  const int n0 = nt * (MODE == GATE_UP ? HALF : S);
  t.e = e; t.m0 = m0; t.m_end = m_end; t.nt = nt; t.n0 = n0; t.second = second;
  // The tile's 32-row groups that hold a valid row are shared out evenly between the two pairs of waves, the last of an odd
  // number together with a dead one: a ragged tile keeps both pairs busy for half the time instead of one for all of it, and
  // rows of dead groups are not loaded (but for that one).
  int nv = HALF / 32, r0 = wm * HALF, m_wave = m_end;
  if constexpr (!is_wgrad(MODE)) {
    int groups = (m_end - m0 + 31) >> 5;
    groups = groups > S / 32 ? S / 32 : groups;
    nv = __builtin_amdgcn_readfirstlane((groups + 1) >> 1);
    r0 = wm * 32 * nv;
    m_wave = m_end < m0 + r0 + 32 * nv ? m_end : m0 + r0 + 32 * nv;
    r0 = __builtin_amdgcn_readfirstlane(r0);
    m_wave = __builtin_amdgcn_readfirstlane(m_wave);
  }
  t.nv = nv; t.r0 = r0; t.m_wave = m_wave;
  t.few = S == 128 && !is_wgrad(MODE) && nv == 1 && rt == 1 && total <= static_cast<int>(gridDim.x);

  // ---------------- operand sources -------------------------------------------
  // Per K step and operand tile a wave issues NL direct-to-LDS loads of 1 KB each:
  //  K-contiguous source ([row][k]): load i of wave w fills LDS rows 8 (NL w + i) .. + 8;
  //    lane l -> row + l/8, physical piece l%8, i.e. logical piece kc_logical_piece(row, l%8).
  //    The base advances by 64 elements per step.  B: these are the tile's rows.  A: they hold its rows 32 i + 8 w .. + 8, so that
  //    the first 2 nv loads of every wave bring the rows of the 2 nv live groups, and the others are left out.
  //  n-contiguous source ([k][n]): load i of wave w fills the KN_RPL (2 or 4) k rows from KN_RPL (NL w + i) on;
  //    with P = KN_PIECES (32 or 16) lane l -> k row + l/P, physical piece l%P = logical piece kn_piece(k row, l%P).
  //    The base advances by 64 rows per step.
  // Lane offsets carry LOAD_BIAS - (i - NL / 2) * 1024 (see dma16_imm); the scalar bases lie LOAD_BIAS low.
  uint32_t (&voa)[NL] = t.voa;          // lane offsets in bytes
  uint32_t (&vob)[NL] = t.vob;
  const char* abase;                    // step 0 of phase 0, without the bias
  const char* bbase;
  ptrdiff_t a_phase = 0, b_phase = 0;   // byte offset of the second K phase (DGRAD_X)
  size_t a_step, b_step;                // bytes per step
  int k_lo = 0, k_hi = 0;               // WGRAD: the expert's row range is the reduction
  const int32_t* row_tok = nullptr;     // GATHER_A/B: token of the expert's first reduction row onwards
  uint32_t (&vcb)[NL] = t.vcb;          // GATHER_A/B: lane offset of a load without its token row
#pragma unroll
  for (int i = 0; i < NL; ++i) { t.vcb[i] = 0; t.tokn[i] = 0; }
  int nk, nk_phase;                     // steps in total / in the first K phase

  if constexpr (is_wgrad(MODE)) {
    k_lo = __builtin_amdgcn_readfirstlane(a.offsets[e]);
    k_hi = __builtin_amdgcn_readfirstlane(a.offsets[e + 1]);
    nk = (k_hi - k_lo + BK - 1) / BK;
    nk_phase = nk;
    if constexpr (GATHER_A) {
      abase = reinterpret_cast<const char*>(a.A0 + m0);
      a_step = 0;
      row_tok = a.row_token + k_lo;
    } else {
      abase = reinterpret_cast<const char*>((second ? a.A1 : a.A0) + static_cast<size_t>(k_lo) * a.M + m0);
      a_step = static_cast<size_t>(BK) * a.M * 2;
    }
    if constexpr (GATHER_B) {
      // the base stays at the first token row; a load's lane offset carries its token (set per step)
      bbase = reinterpret_cast<const char*>(a.B0 + n0);
      b_step = 0;
      row_tok = a.row_token + k_lo;
    } else {
      bbase = reinterpret_cast<const char*>(a.B0 + static_cast<size_t>(k_lo) * a.N + n0);
      b_step = static_cast<size_t>(BK) * a.N * 2;
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int krow = kn_load_row(i, lane);
      const int piece = kn_piece(krow, lane % TL::KN_PIECES);
      int ca = piece * 8;  if (m0 + ca > a.M - 8) ca = a.M - 8 - m0;
      int cb = piece * 8;  if (n0 + cb > a.N - 8) cb = a.N - 8 - n0;
      const uint32_t fix = static_cast<uint32_t>(LOAD_BIAS - (i - NL / 2) * 1024);
      voa[i] = static_cast<uint32_t>((krow * a.M + ca) * 2) + fix;
      vob[i] = static_cast<uint32_t>((krow * a.N + cb) * 2) + fix;
      if constexpr (GATHER_B) vcb[i] = static_cast<uint32_t>(cb * 2) + fix;
      if constexpr (GATHER_A) vcb[i] = static_cast<uint32_t>(ca * 2) + fix;
    }
  } else {
    nk = a.K / BK;
    nk_phase = nk;
    abase = reinterpret_cast<const char*>(a.A0 + static_cast<size_t>(m0) * a.K);
    a_step = BK * 2;
    bool gathered = false;
    if constexpr (MODE == GATE_UP) gathered = a.row_token != nullptr;
    if constexpr (MODE == DGRAD_H_GATE) gathered = true;
    if (gathered) abase = reinterpret_cast<const char*>(a.A0);   // lane offsets carry the token row
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int row = i * 32 + wave * 8 + (lane >> 3);
      const int chunk = kc_logical_piece(row, lane & 7);
      int r = row;
      if (m0 + r > m_end - 1) r = m_end - 1 - m0;
      const uint32_t fix = static_cast<uint32_t>(LOAD_BIAS - (i - NL / 2) * 1024);
      if (gathered) voa[i] = (static_cast<uint32_t>(a.row_token[m0 + r]) * a.K + chunk * 8) * 2u + fix;
      else voa[i] = static_cast<uint32_t>((r * a.K + chunk * 8) * 2) + fix;
    }
    if constexpr (MODE == DGRAD_X) { a_phase = (a.A1 - a.A0) * 2; nk *= 2; }
    const size_t wsz = static_cast<size_t>(a.N) * a.K;
    if constexpr (!B_KN) {
      // GATE_UP: with Q = S / 4 a wave's 2 Q tile rows are Q rows of Wg and the same Q rows of Wu: tile rows
      // [0,Q) Wg n0.., [Q,2Q) Wu n0.., [2Q,3Q) Wg n0+Q.., [3Q,4Q) Wu n0+Q.. (wave w fills rows Q w .. of them)
      const uint16_t* w = a.B0;
      int first_col = wave * (S / 4);
      if constexpr (MODE == GATE_UP) {
        if (wave & 1) w = a.B1;
        first_col = (wave >> 1) * (S / 4);
      }
      bbase = reinterpret_cast<const char*>(w + static_cast<size_t>(e) * wsz + static_cast<size_t>(n0) * a.K);
      b_step = BK * 2;
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int row = (wave * NL + i) * 8 + (lane >> 3);   // LDS row of the B tile
        const int chunk = kc_logical_piece(row, lane & 7);
        int col = first_col + i * 8 + (lane >> 3);
        if (n0 + col > a.N - 1) col = a.N - 1 - n0;
        vob[i] = static_cast<uint32_t>((col * a.K + chunk * 8) * 2) + static_cast<uint32_t>(LOAD_BIAS - (i - NL / 2) * 1024);
      }
    } else {  // DGRAD_H / DGRAD_X: weights stored [K][N]
      bbase = reinterpret_cast<const char*>(a.B0 + static_cast<size_t>(e) * wsz + n0);
      b_step = static_cast<size_t>(BK) * a.N * 2;
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int krow = kn_load_row(i, lane);
        int cb = kn_piece(krow, lane % TL::KN_PIECES) * 8;
        if (n0 + cb > a.N - 8) cb = a.N - 8 - n0;
        vob[i] = static_cast<uint32_t>((krow * a.N + cb) * 2) + static_cast<uint32_t>(LOAD_BIAS - (i - NL / 2) * 1024);
      }
      if constexpr (MODE == DGRAD_X) b_phase = (a.B1 - a.B0) * 2;
    }
  }

  // Both bases live in scalar registers and are advanced by scalar adds: steps are loaded in order.
  t.sa_next = scalarize(abase - LOAD_BIAS);
  t.sb_next = scalarize(bbase - LOAD_BIAS);
  t.sa_phase1 = nullptr;
  t.sb_phase1 = nullptr;
  if constexpr (MODE == DGRAD_X) { t.sa_phase1 = scalarize(abase + a_phase - LOAD_BIAS); t.sb_phase1 = scalarize(bbase + b_phase - LOAD_BIAS); }
  t.a_step = a_step; t.b_step = b_step; t.k_lo = k_lo; t.k_hi = k_hi; t.row_tok = row_tok; t.nk = nk; t.nk_phase = nk_phase;
  t.last_partial = is_wgrad(MODE) && ((k_hi - k_lo) % BK) != 0;
  // The last three steps of a tile are copies of their own: the last step that loads (it loads the tile's last
  // step, the one that may be partial in a weight gradient), the step that only awaits, and the last one.
  // The tile enters the ring at the phase p0 that puts these three on phases 0, 1 and 2, so that the steps
  // before them end on a round of the five phases.
  t.nmain = nk >= 3 ? nk - 3 : 0;
  t.p0 = nk >= 3 ? (NSLOT - t.nmain % NSLOT) % NSLOT : (nk == 2 ? 1 : 2);
  };


  // Load i of the A / B tile of step kt (M0 must point at the tile's slot already).  In the weight gradients the
  // last step of an expert may be partial (its row count is no multiple of 64): reduction rows at or past the
  // expert's end then read zeros in one operand (per-lane 64-bit addresses) and a valid row in the other.
  // SP 0: the step is known to be whole; 1: known to be the partial one; 2: look (first loads of a tile).
  auto a_part = [&](TileState& t, int kt, auto i_tag, auto sp_tag) __attribute__((always_inline)) {
    constexpr int i = decltype(i_tag)::value, SP = decltype(sp_tag)::value;
    constexpr int OFF = (i - NL / 2) * 1024;
    if constexpr (is_wgrad(MODE) && !GATHER_A && SP != 0) {
      if (SP == 1 || (t.last_partial && kt == t.nk - 1)) {
        const int krow = t.k_lo + kt * BK + kn_load_row(i, lane);
        dma16_lane_imm<OFF>(krow < t.k_hi ? t.sa_next + t.voa[i]
                                        : reinterpret_cast<const char*>(g_zero_block) + lane % TL::KN_PIECES * 16 - OFF);
        return;
      }
    }
    dma16_imm<OFF>(t.voa[i], t.sa_next);   // GATHER_A: rows past the expert's end were clamped when their tokens were fetched
  };
  auto b_part = [&](TileState& t, int kt, auto i_tag, auto sp_tag) __attribute__((always_inline)) {
    constexpr int i = decltype(i_tag)::value, SP = decltype(sp_tag)::value;
    constexpr int OFF = (i - NL / 2) * 1024;
    if constexpr ((GATHER_A || MODE == WGRAD) && SP != 0) {
      if (SP == 1 || (t.last_partial && kt == t.nk - 1)) {
        const int krow = t.k_lo + kt * BK + kn_load_row(i, lane);
        if constexpr (GATHER_A) {
          // the gathered operand repeats the expert's last row past its end: this one reads zeros there
          dma16_lane_imm<OFF>(krow < t.k_hi ? t.sb_next + t.vob[i]
                                          : reinterpret_cast<const char*>(g_zero_block) + lane % TL::KN_PIECES * 16 - OFF);
        } else {
          // ... and the other operand reads its last valid row there, so that zero times it is zero
          dma16_lane_imm<OFF>(t.sb_next + t.vob[i] - (krow < t.k_hi ? 0 : static_cast<size_t>(krow - (t.k_hi - 1)) * a.N * 2));
        }
        return;
      }
    }
    dma16_imm<OFF>(t.vob[i], t.sb_next);   // GATHER_B: rows past the expert's end were clamped when their tokens were fetched
  };
  auto a_end = [&](TileState& t, int kt) __attribute__((always_inline)) {
    t.sa_next += t.a_step;
    if constexpr (MODE == DGRAD_X) {
      if (kt + 1 == t.nk_phase) t.sa_next = t.sa_phase1;
    }
  };
  auto b_end = [&](TileState& t, int kt) __attribute__((always_inline)) {
    t.sb_next += t.b_step;
    if constexpr (MODE == DGRAD_X) {
      if (kt + 1 == t.nk_phase) t.sb_next = t.sb_phase1;
    }
  };
  // GATHER_A/B: the tokens of the lane's NL reduction rows of step kt (kn_load_row), loaded
  // without any vector-ALU work except in an expert's last, partial step (rows past its end repeat its last
  // row: the other operand is zero there), and their turn into lane offsets of the gathered operand's loads.
  // The loads are asynchronous: apply_tok may only run after a wait that covers them.
  const uint32_t tok_voff = static_cast<uint32_t>(kn_load_row(0, lane) * 4);   // row of load 0; load i: + KN_RPL i rows
  auto fetch_tok = [&](TileState& t, int kt, int (&tk)[NL]) __attribute__((always_inline)) {
    if constexpr (GATHER_B || GATHER_A) {
      if (t.k_lo + (kt + 1) * BK > t.k_hi) {
        settle(t.row_tok);
        const int last = t.k_hi - t.k_lo - 1;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          int r = kt * BK + kn_load_row(i, lane);
          if (r > last) r = last;
          tk[i] = load_i32<0>(static_cast<uint32_t>(r) * 4u, t.row_tok);
        }
      } else {
        const int32_t* base = t.row_tok + static_cast<size_t>(kt) * BK;
        settle(base);
        static_for<NL>([&](auto i_tag) {
          constexpr int i = decltype(i_tag)::value;
          tk[i] = load_i32<i * TL::KN_RPL * 4>(tok_voff, base);
        });
      }
    }
  };
  auto apply_tok = [&](TileState& t, int (&tk)[NL]) __attribute__((always_inline)) {
    if constexpr (GATHER_B || GATHER_A) {
      const uint32_t row_bytes = static_cast<uint32_t>(GATHER_B ? a.N : a.M) * 2u;
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        asm volatile("" : "+v"(tk[i]));   // not before the wait that precedes this call
        const uint32_t off = static_cast<uint32_t>(tk[i]) * row_bytes + t.vcb[i];
        if constexpr (GATHER_B) t.vob[i] = off; else t.voa[i] = off;
      }
    }
  };

  // ---------------- fragment addresses ------------------------------------------
  // Slot, block and sub-step are immediate offsets of the LDS reads, which reach 64 KB: one set of per-lane addresses
  // serves slots 0-1, one slots 2-3, one slot 4 (S = 128: slots 0-3, slot 4); up to four addresses per set and operand.
  //  [row][k] tile: block b = rows 16 b + (lane & 15), sub-step s (32 k) = logical piece 4 s + lane / 16.
  //    The row's share of the swizzle is lane & 7 whatever the block, so the address of (b, s) is
  //    base[s] + 2048 b.
  //  [k][n] tile: block b = columns 16 b + (lane & 15); within 16 lanes, lane i supplies the address of four
  //    consecutive n of k row i / 4, n group i % 4, and lane l receives k rows 0..3 of column l; lanes
  //    16 g .. 16 g + 15 take k rows 8 g .. of the sub-step.  The k-row swizzle XORs bits 1-2 of the block
  //    number (counted over the whole row), so the address of block b is base[b / 2] + 32 (b & 1); the second half of a
  //    fragment lies 4 k rows further, sub-step 1 32 k rows.
  //  The row-grouped A operand is kept as eight rows per wave of every 32-row group (see the loads): row 32 i + 8 w + s lies
  //    at LDS row 8 (NL w + i) + s, so block b begins at LDS rows 16 NL (b & 1) + 8 (b / 2) and its second half 8 NL rows further.
  //    Its addresses carry the wave's first row r0, which depends on the tile (a multiple of 32, that is 8 LDS rows).
  uint32_t fa_base[TL::SETS][4], fb_base[TL::SETS][4];
#pragma unroll
  for (int st = 0; st < TL::SETS; ++st) {
    const uint32_t org = lds0 + st * TL::SLOTS_PER_SET * TILE_BYTES;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int i16 = lane & 15;
      // [row][k]
      const int pc = ((x & 1) * 4 + (lane >> 4) + (lane & 7)) & 7;   // sub-step x & 1; the block is an immediate offset
      const uint32_t kc_a = org + (i16 >> 3) * (NL * 1024) + (lane & 7) * 128 + pc * 16;   // + 32 r0 of the tile, see main_loop
      const uint32_t kc_b = org + (wn * HALF + i16) * 128 + pc * 16;
      // [k][n]
      const int krow = (lane >> 4) * 8 + (i16 >> 2);
      const int sw = krow & 3;
      const uint32_t kn_lane = org + krow * TL::KN_ROW + ((i16 >> 1) & 1) * 16 + (i16 & 1) * 8;
      const uint32_t kn_a = kn_lane + (((wm * (NB / 2) + x) ^ sw) << 6);   // 64-byte group of block 2 x in the row
      const uint32_t kn_b = kn_lane + (((wn * (NB / 2) + x) ^ sw) << 6);
      fa_base[st][x] = A_KN ? kn_a : kc_a;
      fb_base[st][x] = B_KN ? kn_b : kc_b;
    }
  }
  int fa_r0 = 0;                 // the r0 that the A addresses carry

  // ---------------- main loop ----------------------------------------------------
  f32x4_t acc[NB][NB];

  // two fragment sets: one feeds the MFMAs while the other is being read
  KnFrag fa[2][NB], fb[2][NB];
  constexpr int A_OPS_PER_BLK = A_KN ? 2 : 1, B_OPS_PER_BLK = B_KN ? 2 : 1, SPS = TL::SLOTS_PER_SET;
  // Read instruction number `op` of a sub-step: the A blocks first (only the live ones), then the B blocks.
  auto read_op = [&](auto slot_a_tag, auto slot_b_tag, auto s_tag, auto set_tag, auto nv_tag, auto op_tag) __attribute__((always_inline)) {
    constexpr int SA = decltype(slot_a_tag)::value, SB = decltype(slot_b_tag)::value, SUB = decltype(s_tag)::value;
    constexpr int SET = decltype(set_tag)::value, NV = decltype(nv_tag)::value, OP = decltype(op_tag)::value;
    constexpr int A_OPS = 2 * NV * A_OPS_PER_BLK;
    if constexpr (OP < A_OPS) {
      constexpr int blk = OP / A_OPS_PER_BLK;
      if constexpr (A_KN) {
        constexpr int half = OP % 2;
        fa[SET][blk].h[half] = lds_read_tr_b64<SA % SPS * TILE_BYTES + SUB * 32 * TL::KN_ROW + half * 4 * TL::KN_ROW + (blk & 1) * 32>(fa_base[SA / SPS][blk >> 1]);
      } else {
        fa[SET][blk].v = lds_read_b128<SA % SPS * TILE_BYTES + (blk & 1) * 2 * NL * 1024 + (blk >> 1) * 1024>(fa_base[SA / SPS][SUB]);
      }
    } else {
      constexpr int OB = OP - A_OPS;
      constexpr int blk = OB / B_OPS_PER_BLK;
      if constexpr (B_KN) {
        constexpr int half = OB % 2;
        fb[SET][blk].h[half] = lds_read_tr_b64<SB % SPS * TILE_BYTES + SUB * 32 * TL::KN_ROW + half * 4 * TL::KN_ROW + (blk & 1) * 32>(fb_base[SB / SPS][blk >> 1]);
      } else {
        fb[SET][blk].v = lds_read_b128<SB % SPS * TILE_BYTES + blk * 2048>(fb_base[SB / SPS][SUB]);
      }
    }
  };
  // weight fragment first: the lane then holds 4 consecutive output columns of one row
  auto mma = [&](auto set_tag, auto i_tag, auto j_tag) __attribute__((always_inline)) {
    constexpr int SET = decltype(set_tag)::value, i = decltype(i_tag)::value, j = decltype(j_tag)::value;
    f32x4_t& c = acc[i][j];
    const bf16x8_t& wfrag = fb[SET][j].v;
    const bf16x8_t& afrag = fa[SET][i].v;
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(wfrag), "v"(afrag));
  };

  // One 32-deep sub-step: the live MFMAs of fragment set SET, in 2 x 2 blocks of accumulators so that within a block every product shares an operand
  // with the one before it, now the weights and now the rows; from one block to the next of the same pair of rows neither is shared (12 of the 63 steps of a
  // whole wave's piece).  The chip runs at its power limit here, and operands that were read a
  // moment ago cost less than new ones: with nothing but these MFMAs 1.007 us per K step in this order, 1.041 row by row (one operand held for
  // eight), 1.081 in scattered order; with the loop's reads, loads and barriers 1.225 / 1.256 us, the clock 1.82 / 1.78 GHz.
  // Products of 65536 rows, d 2048, f 1024, 64 experts, row by row -> 2 x 2: gate_up 440 -> 434 us, down of 2048 steps 422 -> 419, dgrad_x 419 -> 412,
  // the weight gradients 806 -> 799 and 423 -> 417.  Between the MFMAs (one per gap) stand the read
  // instructions of the next sub-step and, in a step that loads, the wave's LOADS loads of one
  // tile.  Gap g is the place after MFMA g: reads take the even gaps 0, 2, .. (every gap when they would not fit
  // otherwise), M0 is set in gap 1, loads take gaps 3, 7, .., 4 LOADS - 1; what does not fit behind
  // the last live MFMA follows it.
  constexpr auto a_loads = [](int nv) { return is_wgrad(MODE) ? NL : 2 * nv; };   // A loads per wave and step
  auto sub_step = [&](auto set_tag, auto nv_tag, auto nreads_tag, auto reader, auto loads_tag, auto set_m0_fn, auto loader)
      __attribute__((always_inline)) {
    constexpr int SET = decltype(set_tag)::value, NV = decltype(nv_tag)::value;
    constexpr int NREADS = decltype(nreads_tag)::value;
    constexpr int LOADS = decltype(loads_tag)::value;   // how many, 0: none
    constexpr int ML = 2 * NB * NV;                     // live MFMAs: blocks i < 2 NV, all j
    constexpr int RSTRIDE = 2 * NREADS > NB * NB ? 1 : 2;
    constexpr int LAST_LOAD = 4 * LOADS - 1;
    constexpr int LAST_GAP = (NREADS - 1) * RSTRIDE > LAST_LOAD ? (NREADS - 1) * RSTRIDE : LAST_LOAD;
    constexpr int SLOTS = ML > LAST_GAP + 1 ? ML : LAST_GAP + 1;
    static_for<SLOTS>([&](auto g_tag) {
      constexpr int g = decltype(g_tag)::value;
      if constexpr (g < ML) {
        constexpr int pair = g / (2 * NB), q = g % 4, at = g % (2 * NB) / 4, jj = pair & 1 ? NB / 2 - 1 - at : at;
        mma(IC<SET>{}, IC<2 * pair + q / 2>{}, IC<2 * jj + ((q & 1) ^ (q >> 1))>{});
      }
      if constexpr (g % RSTRIDE == 0 && g / RSTRIDE < NREADS) reader(IC<g / RSTRIDE>{});
      if constexpr (LOADS > 0) {
        if constexpr (g == 1) set_m0_fn();
        if constexpr (g >= 3 && g <= LAST_LOAD && (g - 3) % 4 == 0) loader(IC<(g - 3) / 4>{});
      }
    });
  };

  // Step kt at ring phase P.  KIND 2: a step that loads A(kt+2) (before its barrier, into B(kt-1)'s old slot) and
  // B(kt+2) (behind it, into A(kt)'s slot); KIND 1: the second to last step (nothing left to load); KIND 0: the
  // last step (no barrier, no next fragments).
  auto step = [&](TileState& t, int kt, auto phase_tag, auto kind_tag, auto nv_tag, auto sp_tag) __attribute__((always_inline)) {
    constexpr int P = decltype(phase_tag)::value, KIND = decltype(kind_tag)::value, NV = decltype(nv_tag)::value;
    using SA = IC<slot_of_a(P)>;
    using SB = IC<slot_of_b(P)>;
    using NextA = IC<slot_of_a((P + 1) % NSLOT)>;
    using NextB = IC<slot_of_b((P + 1) % NSLOT)>;
    constexpr int LA = slot_of_a((P + 2) % NSLOT);
    constexpr int ALOADS = a_loads(NV);
    constexpr int NREADS = 2 * NV * A_OPS_PER_BLK + NB * B_OPS_PER_BLK;
    if constexpr (KIND == 2 && GATHER_A) {
      // the tokens of A(kt+2) were fetched a step ago and are covered by that step's wait; those of A(kt+3)
      // are requested before the loads of A(kt+2), the only ones this step's wait leaves in flight
      apply_tok(t, t.tokn);
      if (kt + 3 < t.nk) fetch_tok(t, kt + 3, t.tokn);
    }
    sub_step(IC<0>{}, nv_tag, IC<NREADS>{},
             [&](auto op) __attribute__((always_inline)) { read_op(SA{}, SB{}, IC<1>{}, IC<1>{}, nv_tag, op); },
             IC<KIND == 2 ? ALOADS : 0>{},
             [&]() __attribute__((always_inline)) { set_m0<LA * TILE_BYTES>(lds_fill); settle(t.sa_next); },
             [&](auto i) __attribute__((always_inline)) { a_part(t, kt + 2, i, sp_tag); });
    if constexpr (KIND == 2) a_end(t, kt + 2);
    lds_wait<0>();
    if constexpr (KIND >= 1) {
      if constexpr (KIND == 2) wait_vm<ALOADS>(); else wait_vm<0>();   // this wave's loads of A(kt+2) may stay in flight
      wg_barrier();
    }
    if constexpr (KIND == 2 && GATHER_B) apply_tok(t, t.tokn);   // fetched a step ago, older than the loads of A(kt+2)
    sub_step(IC<1>{}, nv_tag, IC<KIND >= 1 ? NREADS : 0>{},
             [&](auto op) __attribute__((always_inline)) { read_op(NextA{}, NextB{}, IC<0>{}, IC<0>{}, nv_tag, op); },
             IC<KIND == 2 ? NL : 0>{},
             [&]() __attribute__((always_inline)) { set_m0<SA::value * TILE_BYTES>(lds_fill); settle(t.sb_next); },
             [&](auto i) __attribute__((always_inline)) { b_part(t, kt + 2, i, sp_tag); });
    if constexpr (KIND == 2) {
      b_end(t, kt + 2);
      if constexpr (GATHER_B) {
        // a whole step ahead of their use; the next step's wait covers them (they are older than its A loads)
        if (kt + 3 < t.nk) fetch_tok(t, kt + 3, t.tokn);
      }
    }
    lds_wait<0>();
  };

  // The first loads of a tile: steps 0 and 1 into the slots of phases p0 and p0 + 1.  They are requested BEFORE the epilogue
  // of the tile before, which is staged in the slot that they leave free (spare_slot; the SwiGLU derivative needs two, so
  // that B(1) waits until it is done), and awaited when the tile's main loop starts.
  // What a tile waits for between main loops counts where tiles are short: a training step of 2048 tokens (d 2048, f 1024, 64
  // experts, 4 steps per weight gradient) 885 -> 868 us, the forward of 4001 tokens over 128 experts of f 512 328 -> 322 us;
  // at 1024 rows per expert and more the chip is power-limited and the step takes as long as before (0-1.5 % less).
  // A tile with few rows is the only one of its workgroup's list (see TileState::few): there is no epilogue before it.
  auto spare_slot = [&](const TileState& t) __attribute__((always_inline)) { return (2 * t.p0 + 4) % NSLOT; };
  auto spare_slot2 = [&](const TileState& t) __attribute__((always_inline)) { return (2 * t.p0 + 3) % NSLOT; };
  auto a_unit = [&](TileState& t, int kt) __attribute__((always_inline)) {   // kt: 0 or 1
    int at = lds_fill + (2 * t.p0 + 2 * kt) % NSLOT * TILE_BYTES;
    if (t.few) at = few_a + kt * FEW_A_BYTES;
    set_m0_rt(__builtin_amdgcn_readfirstlane(at));
    settle(t.sa_next);
    if constexpr (is_wgrad(MODE)) {
      static_for<NL>([&](auto i) { a_part(t, kt, i, IC<2>{}); });
    } else {
      static_for<HALF / 32>([&](auto g) {
        constexpr int i = 2 * decltype(g)::value;
        if (i == 0 || i < 2 * t.nv) { a_part(t, kt, IC<i>{}, IC<2>{}); a_part(t, kt, IC<i + 1>{}, IC<2>{}); }
      });
    }
    a_end(t, kt);
  };
  auto b_unit = [&](TileState& t, int kt) __attribute__((always_inline)) {
    const int slot = t.few ? kt : (2 * t.p0 + 2 * kt + 1) % NSLOT;
    set_m0_rt(__builtin_amdgcn_readfirstlane(lds_fill + slot * TILE_BYTES));
    settle(t.sb_next);
    static_for<NL>([&](auto i) { b_part(t, kt, i, IC<2>{}); });
    b_end(t, kt);
  };
  auto first_loads = [&](TileState& t) __attribute__((always_inline)) {
    if (t.nk <= 0) return;
    if constexpr (GATHER_A || GATHER_B) {
      // The tokens of steps 0, 1 and 2 are requested first, older than the loads of the other operand, and are here before
      // the epilogue starts: no register that a load has yet to write lives across it.  Rows past the expert's end, and
      // steps that do not exist, repeat its last row.
      int tk[3][NL];
      const int last = t.k_hi - t.k_lo - 1;
      settle(t.row_tok);
      static_for<3>([&](auto s_tag) {
        constexpr int s = decltype(s_tag)::value;
        static_for<NL>([&](auto i_tag) {
          constexpr int i = decltype(i_tag)::value;
          int r = s * BK + kn_load_row(i, lane);
          if (r > last) r = last;
          tk[s][i] = load_i32<0>(static_cast<uint32_t>(r) * 4u, t.row_tok);
        });
      });
      if constexpr (GATHER_B) a_unit(t, 0); else b_unit(t, 0);
      wait_vm<NL>();                            // on every path, behind no branch: the compiler does not know of these loads
#pragma unroll
      for (int i = 0; i < 3 * NL; ++i) asm volatile("" : "+v"(tk[i / NL][i % NL]));
      if (t.nk > 1) { if constexpr (GATHER_B) a_unit(t, 1); else b_unit(t, 1); }
      apply_tok(t, tk[0]);
      if constexpr (GATHER_B) b_unit(t, 0); else a_unit(t, 0);
      apply_tok(t, tk[1]);
#pragma unroll
      for (int i = 0; i < NL; ++i) t.tokn[i] = tk[2][i];
      if (t.nk > 1) { if constexpr (GATHER_B) b_unit(t, 1); else a_unit(t, 1); }
    } else {
      b_unit(t, 0);
      a_unit(t, 0);
      if (t.nk > 1) {
        if (!is_dgrad_h(MODE) || t.few) b_unit(t, 1);
        a_unit(t, 1);
      }
    }
  };
  auto last_first_loads = [&](TileState& t) __attribute__((always_inline)) {
    if constexpr (is_dgrad_h(MODE)) { if (t.nk > 1 && !t.few) b_unit(t, 1); }
  };
  auto main_loop = [&](TileState& t, auto nv_tag) __attribute__((always_inline)) {
    if (t.nk <= 0) return;
    if constexpr (!A_KN) {
#pragma unroll
      for (int st = 0; st < TL::SETS; ++st) {
        fa_base[st][0] += (t.r0 - fa_r0) * 32;
        fa_base[st][1] += (t.r0 - fa_r0) * 32;
      }
      fa_r0 = t.r0;
    }
    const int p0 = t.p0, nmain = t.nmain;
    // The tile's first loads are awaited; those of step 1 may stay in flight (the last of a gathered operand only: both
    // steps of the other one come first).  Stores of the epilogue before are in flight too; as loads complete in order
    // among themselves, the waits here and in the steps hold wherever the stores lie between them.
    constexpr int NV = decltype(nv_tag)::value;
    if (t.nk <= 1) wait_vm<0>(); else if (GATHER_A || GATHER_B) wait_vm<NL>(); else wait_vm<a_loads(NV) + NL>();
    wg_barrier();
    // ---- first fragments: sub-step 0 of step 0, from the slots of phase p0
    constexpr int NREADS = 2 * NV * A_OPS_PER_BLK + NB * B_OPS_PER_BLK;
    auto first_reads = [&](auto phase_tag) __attribute__((always_inline)) {
      constexpr int P = decltype(phase_tag)::value;
      static_for<NREADS>([&](auto op) { read_op(IC<slot_of_a(P)>{}, IC<slot_of_b(P)>{}, IC<0>{}, IC<0>{}, nv_tag, op); });
    };
    switch (p0) {
      case 0: first_reads(IC<0>{}); break;
      case 1: first_reads(IC<1>{}); break;
      case 2: first_reads(IC<2>{}); break;
      case 3: first_reads(IC<3>{}); break;
      default: first_reads(IC<4>{}); break;
    }
    lds_wait<0>();
    asm volatile("s_nop 7" ::: "memory");   // the accumulators were cleared by vector-ALU writes: keep the first MFMA clear of them
    // ---- the steps that load, in rounds of the five phases (the first round starts at p0)
    int kt = 0;
    int skip = p0;
    while (kt < nmain) {
      if (skip <= 0) { step(t, kt, IC<0>{}, IC<2>{}, nv_tag, IC<0>{}); ++kt; }
      if (skip <= 1) { step(t, kt, IC<1>{}, IC<2>{}, nv_tag, IC<0>{}); ++kt; }
      if (skip <= 2) { step(t, kt, IC<2>{}, IC<2>{}, nv_tag, IC<0>{}); ++kt; }
      if (skip <= 3) { step(t, kt, IC<3>{}, IC<2>{}, nv_tag, IC<0>{}); ++kt; }
      step(t, kt, IC<4>{}, IC<2>{}, nv_tag, IC<0>{}); ++kt;
      skip = 0;
    }
    // ---- the last three steps
    if (t.nk >= 3) step(t, t.nk - 3, IC<0>{}, IC<2>{}, nv_tag, IC<is_wgrad(MODE) ? 1 : 0>{});
    if (t.nk >= 2) step(t, t.nk - 2, IC<1>{}, IC<1>{}, nv_tag, IC<0>{});
    step(t, t.nk - 1, IC<2>{}, IC<0>{}, nv_tag, IC<0>{});
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");   // the last MFMAs have written before the accumulators are read
  };
  // The main loop of a small tile that holds all of an expert's at most 64 rows, in a list with no more tiles than workgroups.  It
  // shares its weights with nobody, has little to multiply, and what it waits for is the latency of memory: in the ring above a
  // step's B tile is requested one step before it is awaited; the rows that are not there make room for FEW_RING steps of B and A,
  // all but one of them in flight.  The loop is kept plain (slots are computed, fragments are read in front of the products
  // that use them): there is time for it.
  // Not for what is left of an expert after whole tiles, nor in tiles of 256: those share their weights with the expert's other
  // tiles, and taking more than their part of the memory's bandwidth slows the others down (2048 tokens, d 2048, f 1024, 64
  // experts, forward and backward: 901 -> 921 us when they had such a ring too).  Nor in longer lists, which wait for bandwidth
  // rather than latency (501 tokens of the same layer, forward: 192 -> 197 us on one card, 212 -> 202 us on another).
  // Without / with, us: forward of 597 tokens, d 2240, f 192, 41 experts, 1 per token 57.8 / 50.2; of 146 tokens, d 256, f 1216, 33
  // experts, 6 per token 42.3 / 40.5; forward and backward of 453 tokens, d 3072, f 128, 3 of 38 experts 100 / 96.8.
  auto few_rows_loop = [&](TileState& t) __attribute__((always_inline)) {
    constexpr int STEP_LOADS = 2 + NL;
    constexpr int NREADS = 2 + NB * B_OPS_PER_BLK;       // per 32-deep sub-step
    const int i16 = lane & 15;
    // row 32 i + 8 w + s of the tile lies at LDS row 8 (2 w + i) + s (see the loads; i is 0 or 1)
    const uint32_t a_lane = lds0 + FEW_RING * TILE_BYTES + (i16 >> 3) * 2048 + (lane & 7) * 128 + t.r0 * 32;
    const uint32_t a_sub0 = a_lane + (((lane >> 4) + (lane & 7)) & 7) * 16, a_sub1 = a_lane + ((4 + (lane >> 4) + (lane & 7)) & 7) * 16;
    asm volatile("s_nop 7" ::: "memory");   // the accumulators were cleared by vector-ALU writes
    int cur = 0, nxt = 2;                   // slots of step kt and of step kt + 2
#pragma clang loop unroll(disable)
    for (int kt = 0; kt < t.nk; ++kt) {
      asm volatile("" : "+s"(kt));          // one copy of the body: two would keep the accumulators in different registers
      // this step's tiles are here (requests complete in order) ...
      if (kt + 1 < t.nk) wait_vm<STEP_LOADS>(); else wait_vm<0>();
      wg_barrier();                         // ... those of the other waves too, and every wave is done with step kt - 1, whose slot
      if (kt + 2 < t.nk) {                  // is requested anew
        set_m0_rt(__builtin_amdgcn_readfirstlane(lds_fill + nxt * TILE_BYTES));
        settle(t.sb_next);
        static_for<NL>([&](auto i) { b_part(t, kt + 2, i, IC<0>{}); });
        b_end(t, kt + 2);
        set_m0_rt(__builtin_amdgcn_readfirstlane(few_a + nxt * FEW_A_BYTES));
        settle(t.sa_next);
        static_for<2>([&](auto i) { a_part(t, kt + 2, i, IC<0>{}); });
        a_end(t, kt + 2);
      }
      uint32_t a_at[2] = {a_sub0 + cur * FEW_A_BYTES, a_sub1 + cur * FEW_A_BYTES}, b_at[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) b_at[x] = fb_base[0][x] + cur * TILE_BYTES;
      static_for<2>([&](auto s_tag) {
        constexpr int SUB = decltype(s_tag)::value;
        static_for<2>([&](auto b_tag) {
          constexpr int blk = decltype(b_tag)::value;
          fa[SUB][blk].v = lds_read_b128<blk * 4096>(a_at[SUB]);
        });
        static_for<NB>([&](auto b_tag) {
          constexpr int blk = decltype(b_tag)::value;
          if constexpr (B_KN) {
            static_for<2>([&](auto h_tag) {
              constexpr int half = decltype(h_tag)::value;
              fb[SUB][blk].h[half] = lds_read_tr_b64<SUB * 32 * TL::KN_ROW + half * 4 * TL::KN_ROW + (blk & 1) * 32>(b_at[blk >> 1]);
            });
          } else {
            fb[SUB][blk].v = lds_read_b128<blk * 2048>(b_at[SUB]);
          }
        });
      });
      static_for<2>([&](auto s_tag) {
        constexpr int SUB = decltype(s_tag)::value;
        lds_wait<SUB == 0 ? NREADS : 0>();      // the reads of the other sub-step may be under way
        static_for<2>([&](auto i) { static_for<NB>([&](auto j) { mma(IC<SUB>{}, i, j); }); });
      });
      cur = cur + 1 == FEW_RING ? 0 : cur + 1;
      nxt = nxt + 1 == FEW_RING ? 0 : nxt + 1;
      // the last MFMAs have written before the accumulators are read, or moved, which the compiler may do where paths join and
      // without a wait, since it does not know the statements above for what they are
      asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");
    }
  };
  // one copy of the loop per number of live 32-row groups
  auto run_main = [&](TileState& t) __attribute__((always_inline)) {
    if constexpr (is_wgrad(MODE)) {
      main_loop(t, IC<HALF / 32>{});
    } else if constexpr (S == 128) {
      if (t.few) few_rows_loop(t); else if (t.nv == 2) main_loop(t, IC<2>{}); else main_loop(t, IC<1>{});
    } else {
      switch (t.nv) {
        case 4: main_loop(t, IC<4>{}); break;
        case 3: main_loop(t, IC<3>{}); break;
        case 2: main_loop(t, IC<2>{}); break;
        default: main_loop(t, IC<1>{}); break;
      }
    }
  };
  // ---------------- epilogue -----------------------------------------------------
  // acc[i][j][c] is the wave's element (row, col) with row = 16 i + (lane & 15) and col = 16 j + 4 (lane / 16) + c.
  // The wave stages its bf16 rows of S bytes in LDS of its own (its share of a ring slot; 16-byte pieces
  // swizzled by the row), a few rows at a time, and stores 16 bytes per lane in full row segments.
  // The accumulators are read out of the accumulation registers at the point of use, by hand: left to the
  // compiler they are moved (and spilled) in bulk where the copies of the main loop join.
  auto accq = [&](auto i_tag, auto j_tag) __attribute__((always_inline)) -> f32x4_t {
    constexpr int i = decltype(i_tag)::value, j = decltype(j_tag)::value;
    f32x4_t v;
    float x;
    const float c0 = acc[i][j][0], c1 = acc[i][j][1], c2 = acc[i][j][2], c3 = acc[i][j][3];
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x) : "a"(c0));  v[0] = x;
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x) : "a"(c1));  v[1] = x;
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x) : "a"(c2));  v[2] = x;
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x) : "a"(c3));  v[3] = x;
    return v;
  };
  // GATE_UP with gate weights folded into h, DGRAD_H_GATE: the weights of the lane's NB rows, requested
  // right behind the main loop and awaited before the next tile's first loads are requested.
  float wv[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) wv[i] = 1.f;
  auto fetch_row_weights = [&](const TileState& t, const float* rw) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      int r = t.m0 + t.r0 + i * 16 + (lane & 15);  if (r > t.m_end - 1) r = t.m_end - 1;
      wv[i] = rw[r];
    }
    asm volatile("" ::: "memory");            // requested here, not where they are used
  };

  // what the epilogue needs of a tile whose successor is set up already (and its first loads in flight: slot, and for the
  // SwiGLU derivative slot2, is what they leave free)
  struct Finished { int e, m0, n0, r0, m_wave, slot, slot2; bool second; };
  auto epilogue = [&](const Finished& t) __attribute__((always_inline)) {
    const ArgPtr ae = reload_args<ARG>();     // the epilogue reads its arguments afresh
    int tid = tid0;                           // laundered as in setup_tile
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
    const int m_end = t.m_wave, n0 = t.n0;                               // end of the wave's valid rows
    const int grow0 = t.m0 + t.r0;                                       // wave's first output row
    const int gcol0 = n0 + wn * (MODE == GATE_UP ? S / 4 : HALF);        // wave's first output column
    constexpr int RB = S, RP = S / 16;          // bytes and 16-byte pieces of a staged row of all the wave's columns
    char* stage = lds + t.slot * TILE_BYTES + wave * TL::SHARE;
    // address of the 8 bytes of columns 4 lq .. + 3 of 16-column block `blk` in staged row `row`
    auto quad_addr = [&](int row, int blk) __attribute__((always_inline)) -> char* {
      return stage + row * RB + (((2 * blk + (lq >> 1)) ^ (row & (RP - 1))) << 4) + (lq & 1) * 8;
    };
    auto put_quad = [&](int row, int blk, const f32x4_t& v) __attribute__((always_inline)) {
      u32x2 o;
      o.x = pack_bf16(v[0], v[1]);
      o.y = pack_bf16(v[2], v[3]);
      *reinterpret_cast<u32x2*>(quad_addr(row, blk)) = o;
    };
    // Rows are stored (and g, u loaded) through buffer resources that end with the wave's last valid row: what lies past it
    // is dropped (reads as zero) by the hardware's range check, and a lane whose columns do not exist carries an offset
    // past every end (the row is part of the lane's offset, which is what the check looks at).  So the whole epilogue is
    // straight-line code, ragged or not.
    const int ncol = ae->N;
    int rows = m_end - grow0;
    rows = rows < 0 ? 0 : (rows > HALF ? HALF : rows);
    auto rows_of = [&](const void* base, int ld_bytes) __attribute__((always_inline)) {
      const char* first = scalarize(static_cast<const char*>(base) + static_cast<size_t>(grow0) * ld_bytes);
      return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(first), 0, __builtin_amdgcn_readfirstlane(rows * ld_bytes), 0x00020000);
    };
    typedef decltype(rows_of(nullptr, 0)) Rsrc;
    // as unsigned 2^31: not before the end of 128 rows of any width for which the loads' 32-bit lane offsets suffice, and
    // still past it with the row of a part added
    constexpr int PAST = INT_MIN;
    // PASSES staged passes of 64 / PIECES rows of RB bytes each (16-byte pieces swizzled by row & (RB / 16 - 1), region at
    // `base`), the PIECES pieces from PIECE0 on of each row: read into registers, and stored from there (first row
    // `first`, counted from the wave's first) to columns col0 + 8 piece.  NT: the output is not read again soon (g and u: not
    // before the backward pass; dWg and dWu: not by this layer at all), so its stores are marked non-temporal and leave
    // the caches to what the next kernels read (measured: 0.4-0.6 % of the step, most of it in the kernels that follow).
    auto read_staged = [&](u32x4* v, const char* base, auto rb_tag, auto passes_tag, auto piece0_tag, auto pieces_tag)
        __attribute__((always_inline)) {
      constexpr int RB = decltype(rb_tag)::value, PASSES = decltype(passes_tag)::value, PIECES = decltype(pieces_tag)::value;
      constexpr int RPP = 64 / PIECES, SWZ = RB / 16 - 1;
#pragma unroll
      for (int k = 0; k < PASSES; ++k) {
        const int row = k * RPP + lane / PIECES;
        v[k] = *reinterpret_cast<const u32x4*>(base + row * RB + (((decltype(piece0_tag)::value + lane % PIECES) ^ (row & SWZ)) << 4));
      }
    };
    auto store_rows = [&](auto nt_tag, const u32x4* v, Rsrc out, int first, auto passes_tag, auto pieces_tag)
        __attribute__((always_inline)) {
      constexpr int PASSES = decltype(passes_tag)::value, PIECES = decltype(pieces_tag)::value, RPP = 64 / PIECES;
      const int gc = gcol0 + lane % PIECES * 8;
      const int off = gc < ncol ? (lane / PIECES * ncol + gc) * 2 : PAST;
#pragma unroll
      for (int k = 0; k < PASSES; ++k)
        __builtin_amdgcn_raw_buffer_store_b128(v[k], out, off + (first + k * RPP) * ncol * 2, 0, decltype(nt_tag)::value ? 2 : 0);
    };

    // A wave with HALF - 32 rows or fewer takes a second copy, which tests in front of every part whether it has a row: the tests
    // end the overlap, but the parts left out are worth more.
    // Measured against masked stores issued part by part: gate_up 470 -> 459 us and the launch of dgrad_h 575 -> 560 us at
    // 65536 rows, d 2048, f 1024, 64 experts; 17 -> 13 and 25 -> 17 us where experts have 56 rows (d 128, f 512).
    // In every form a part's rows are read back from LDS as soon as they are staged and stored behind the arithmetic of the
    // part after it: with one wave per SIMD nothing else covers the round trip through LDS.
    if constexpr (MODE == GATE_UP) {
      // The first half of the blocks are g, the other half the same columns of u.  Parts of 16 rows: g in the first and u in
      // the second half of the staged rows, h = silu(g) * u (from the fp32 accumulators, times the row's gate weight if
      // the caller folds the weights into h) in rows of half their length behind them.
      const bool weighted = ae->row_weight != nullptr;
      constexpr int HP = RP / 2, GP = 16 * HP / 64;   // pieces of a row of g, u or h; passes of 64 pieces over 16 rows
      char* hstage = stage + 16 * RB;
      const Rsrc go = rows_of(ae->O0, ncol * 2), uo = rows_of(ae->O1, ncol * 2), ho = rows_of(ae->O2, ncol * 2);
      u32x4 v[3 * GP];
      auto store_part = [&](int part) __attribute__((always_inline)) {
        store_rows(IC<1>{}, v, go, part * 16, IC<GP>{}, IC<HP>{});
        store_rows(IC<1>{}, v + GP, uo, part * 16, IC<GP>{}, IC<HP>{});
        store_rows(IC<0>{}, v + 2 * GP, ho, part * 16, IC<GP>{}, IC<HP>{});
      };
      auto parts = [&](auto ragged_tag) __attribute__((always_inline)) {
      constexpr bool RAGGED = decltype(ragged_tag)::value != 0;
      static_for<NB>([&](auto i_tag) {
        constexpr int i = decltype(i_tag)::value;
        if constexpr (RAGGED) { if (i * 16 >= rows) return; }
        const int row = l16;
        const float w = weighted ? wv[i] : 1.f;
        static_for<NB / 2>([&](auto j_tag) {
          constexpr int j = decltype(j_tag)::value;
          const f32x4_t gv = accq(i_tag, IC<j>{});
          const f32x4_t uv = accq(i_tag, IC<j + NB / 2>{});
          put_quad(row, j, gv);
          put_quad(row, j + NB / 2, uv);
          u32x2 o;
          float h[4];
#pragma unroll
          for (int c = 0; c < 4; ++c) h[c] = silu_f(gv[c]) * uv[c] * w;
          o.x = pack_bf16(h[0], h[1]);
          o.y = pack_bf16(h[2], h[3]);
          *reinterpret_cast<u32x2*>(hstage + row * (RB / 2) + (((2 * j + (lq >> 1)) ^ (row & (HP - 1))) << 4) + (lq & 1) * 8) = o;
        });
        __builtin_amdgcn_wave_barrier();
        if constexpr (!RAGGED && i > 0) store_part(i - 1);
        read_staged(v, stage, IC<RB>{}, IC<GP>{}, IC<0>{}, IC<HP>{});
        read_staged(v + GP, stage, IC<RB>{}, IC<GP>{}, IC<HP>{}, IC<HP>{});
        read_staged(v + 2 * GP, hstage, IC<RB / 2>{}, IC<GP>{}, IC<0>{}, IC<HP>{});
        __builtin_amdgcn_wave_barrier();
        if constexpr (RAGGED) store_part(i);
      });
      if constexpr (!RAGGED) store_part(NB - 1);
      };
      if (rows > HALF - 32) parts(IC<0>{}); else parts(IC<1>{});
    } else if constexpr (is_dgrad_h(MODE)) {
      // In parts of 16 rows, staged alternately in the wave's share of two ring slots: g rows in the first half, u rows in
      // the second half of the part's buffer, overwritten in place by dg and du.
      // DGRAD_H_GATE: the accumulators hold dh0 = dout[token] . Wd; the row's gate weight w turns them into
      // dh = w dh0, and the sum over a 64-column strip of dh0 * silu(g) * u is the strip's share of the
      // gradient of w (a lane holds 16 of the strip's columns of its row, lanes ^ 16, ^ 32 the others).
      constexpr bool GATE = (MODE == DGRAD_H_GATE);
      constexpr int GU_PASSES = 16 * RP / 64;   // 16 rows of RP pieces of 16 bytes, 64 per pass
      constexpr int GU_ROWS = 64 / RP;          // rows of a pass
      constexpr int UOFF = TL::SHARE / 2;
      const Rsrc gi = rows_of(ae->G, ncol * 2), ui = rows_of(ae->U, ncol * 2);
      const Rsrc dgo = rows_of(ae->O0, ncol * 2), duo = rows_of(ae->O1, ncol * 2);
      u32x4 pg[GU_PASSES], pu[GU_PASSES];
      const int gu_off = gcol0 + lane % RP * 8 < ncol ? (lane / RP * ncol + gcol0 + lane % RP * 8) * 2 : PAST;
      auto gu_load = [&](int part) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < GU_PASSES; ++p) {
          pg[p] = __builtin_amdgcn_raw_buffer_load_b128(gi, gu_off + (part * 16 + p * GU_ROWS) * ncol * 2, 0, 0);
          pu[p] = __builtin_amdgcn_raw_buffer_load_b128(ui, gu_off + (part * 16 + p * GU_ROWS) * ncol * 2, 0, 0);
        }
      };
      auto gu_stage = [&](char* buf) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < GU_PASSES; ++p) {
          const int row = p * GU_ROWS + lane / RP, piece = lane % RP;
          const int so = row * RB + ((piece ^ (row & (RP - 1))) << 4);
          *reinterpret_cast<u32x4*>(buf + so) = pg[p];
          *reinterpret_cast<u32x4*>(buf + UOFF + so) = pu[p];
        }
      };
      char* const bufs[2] = {stage, lds + t.slot2 * TILE_BYTES + wave * TL::SHARE};
      int qoff[NB];                 // offsets of the lane's quads in a part's buffer: the same for every part
#pragma unroll
      for (int j = 0; j < NB; ++j) qoff[j] = static_cast<int>(quad_addr(l16, j) - stage);
      u32x4 v[2 * GU_PASSES];
      auto store_part = [&](int part) __attribute__((always_inline)) {
        store_rows(IC<0>{}, v, dgo, part * 16, IC<GU_PASSES>{}, IC<RP>{});
        store_rows(IC<0>{}, v + GU_PASSES, duo, part * 16, IC<GU_PASSES>{}, IC<RP>{});
      };
      constexpr int STRIPS = HALF / 64;         // 64-column strips of the wave's piece
      float dpart[NB][STRIPS];
      auto parts = [&](auto ragged_tag) __attribute__((always_inline)) {
      constexpr bool RAGGED = decltype(ragged_tag)::value != 0;
      gu_load(0);
      gu_stage(bufs[0]);
      gu_load(1);
      static_for<NB>([&](auto part_tag) {
        constexpr int part = decltype(part_tag)::value;
        if constexpr (RAGGED) { if (part * 16 >= rows) return; }
        char* const buf = bufs[part & 1];
        const float wrow = GATE ? wv[part] : 1.f;
        float dsum[STRIPS] = {};
        __builtin_amdgcn_wave_barrier();
        // the lane's g and u quads of the part, read in one go: the quads are overwritten in place below, so
        // reads issued one by one would each wait behind the previous quad's write
        u32x2 gqs[NB], uqs[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          gqs[j] = *reinterpret_cast<const u32x2*>(buf + qoff[j]);
          uqs[j] = *reinterpret_cast<const u32x2*>(buf + qoff[j] + UOFF);
        }
        static_for<NB>([&](auto j_tag) {
          constexpr int j = decltype(j_tag)::value;
          const f32x4_t dhv = accq(part_tag, j_tag);
          char* ga = buf + qoff[j];
          char* ua = ga + UOFF;
          const u32x2 gq = gqs[j];
          const u32x2 uq = uqs[j];
          const float g4[4] = {bf16lo(gq.x), bf16hi(gq.x), bf16lo(gq.y), bf16hi(gq.y)};
          const float u4[4] = {bf16lo(uq.x), bf16hi(uq.x), bf16lo(uq.y), bf16hi(uq.y)};
          float dg[4], du[4];
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const float sg = sigmoid_f(g4[c]);
            if constexpr (GATE) {
              const float dh0 = dhv[c];
              const float sl = g4[c] * sg;                 // silu(g)
              const float t0 = dh0 * u4[c];
              dsum[j >> 2] = __builtin_fmaf(t0, sl, dsum[j >> 2]);   // 4 blocks to a strip
              du[c] = (dh0 * wrow) * sl;
              dg[c] = (t0 * wrow) * (sg * __builtin_fmaf(g4[c], 1.0f - sg, 1.0f));
            } else {
              const float dh = dhv[c];
              const float x = dh * sg;                     // shared by both derivatives
              du[c] = x * g4[c];
              dg[c] = (x * u4[c]) * __builtin_fmaf(g4[c], 1.0f - sg, 1.0f);
            }
          }
          u32x2 o;
          o.x = pack_bf16(dg[0], dg[1]);  o.y = pack_bf16(dg[2], dg[3]);
          *reinterpret_cast<u32x2*>(ga) = o;
          o.x = pack_bf16(du[0], du[1]);  o.y = pack_bf16(du[2], du[3]);
          *reinterpret_cast<u32x2*>(ua) = o;
        });
        if constexpr (GATE) {
#pragma unroll
          for (int s2 = 0; s2 < STRIPS; ++s2) {
            float x = dsum[s2];
            x += __shfl_xor(x, 16, 64);
            x += __shfl_xor(x, 32, 64);
            dpart[part][s2] = x;
          }
        }
        __builtin_amdgcn_wave_barrier();
        if constexpr (part + 1 < NB) gu_stage(bufs[(part + 1) & 1]);   // awaits the loads of part + 1
        __builtin_amdgcn_wave_barrier();
        if constexpr (!RAGGED && part > 0) store_part(part - 1);
        read_staged(v, buf, IC<RB>{}, IC<GU_PASSES>{}, IC<0>{}, IC<RP>{});
        read_staged(v + GU_PASSES, buf + UOFF, IC<RB>{}, IC<GU_PASSES>{}, IC<0>{}, IC<RP>{});
        __builtin_amdgcn_wave_barrier();
        if constexpr (RAGGED) store_part(part);
        if constexpr (part + 2 < NB) gu_load(part + 2);
      });
      if constexpr (!RAGGED) store_part(NB - 1);
      };
      if (rows > HALF - 32) parts(IC<0>{}); else if (rows > 0) parts(IC<1>{});
      if constexpr (GATE) {
        // the strips' shares of the gate gradient, stored behind everything else
        const int strips = ncol >> 6;
        const Rsrc dpo = rows_of(ae->dgate_part, strips * 4);
#pragma unroll
        for (int s2 = 0; s2 < STRIPS; ++s2) {
          // a strip past the last column has no share
          const int off = lq == 0 && gcol0 + s2 * 64 < ncol ? (l16 * strips + (gcol0 >> 6) + s2) * 4 : PAST;
          static_for<NB>([&](auto part_tag) {
            constexpr int part = decltype(part_tag)::value;
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(dpart[part][s2]), dpo, off + part * 16 * strips * 4, 0, 0);
          });
        }
      }
    } else {
      uint16_t* out = t.second ? ae->O1 : ae->O0;
      if constexpr (is_wgrad(MODE)) out += static_cast<size_t>(t.e) * ae->M * ncol;
      const Rsrc oo = rows_of(out, ncol * 2);
      constexpr int PASSES = 32 * RP / 64;
      u32x4 v[PASSES];
      // parts of 32 rows
      auto store_part = [&](int part) __attribute__((always_inline)) {
        store_rows(IC<(MODE == WGRAD_GATHER) ? 1 : 0>{}, v, oo, part * 32, IC<PASSES>{}, IC<RP>{});
      };
      auto parts = [&](auto ragged_tag) __attribute__((always_inline)) {
      constexpr bool RAGGED = decltype(ragged_tag)::value != 0;
      static_for<HALF / 32>([&](auto part_tag) {
        constexpr int part = decltype(part_tag)::value;
        if constexpr (RAGGED) { if (part * 32 >= rows) return; }
        static_for<2>([&](auto i2_tag) {
          constexpr int i2 = decltype(i2_tag)::value;
          static_for<NB>([&](auto j_tag) { put_quad(i2 * 16 + l16, decltype(j_tag)::value, accq(IC<part * 2 + i2>{}, j_tag)); });
        });
        __builtin_amdgcn_wave_barrier();
        if constexpr (!RAGGED && part > 0) store_part(part - 1);
        read_staged(v, stage, IC<RB>{}, IC<PASSES>{}, IC<0>{}, IC<RP>{});
        __builtin_amdgcn_wave_barrier();
        if constexpr (RAGGED) store_part(part);
      });
      if constexpr (!RAGGED) store_part(HALF / 32 - 1);
      };
      if (rows > HALF - 32) parts(IC<0>{}); else parts(IC<1>{});
    }
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): this wave's staging reads are done
  };

  // ---------------- the tile loop ------------------------------------------------
  // A workgroup that always took the same place of an XCD's run would meet the same row tile of every expert whose
  // number of row tiles divides the run, the whole one or the ragged one; so the places move on by one each round
  // (inside a run, where runs are whole: the list stays covered once).
  int tile = first_tile;
  // Where experts have few row tiles (three or fewer on average) the launch waits for weights, and an expert with one row
  // tile needs far more of them per operation than one with many.  The runs are then taken from the two ends of the list in
  // turn, so that a round asks memory for two stretches of experts instead of one.  What they hold depends on the load: inside
  // a class the list is in index order.  Forward and backward pass, in us, list from the front / from both ends, zipf-like
  // load with the experts sorted by size, reversed, in two random orders, and an even load:
  //   64 experts, 2048 tokens, d 2048   949/909  994/980  965/956  983/961  959/942
  //   128 experts, 3000 tokens, d 1024  918/905  902/892  978/947  987/963  770/763
  //   96 experts, 4099 tokens, d 2048   1651/1607  1677/1687  1709/1702  1628/1657  1503/1501
  // (Listing the experts by their tile counts first changed this by -3 to +3 %, on average by nothing.)  Not with reductions
  // under 16 steps: there the experts that straddle two runs, fetched twice when the runs are far apart in time, weigh more
  // (down of 128 experts with 250 rows and 8 steps: 116 -> 124 us), nor with more row tiles (no difference).
  bool mix = false;
  if constexpr (!is_wgrad(MODE)) mix = a.K * (MODE == DGRAD_X ? 2 : 1) >= 16 * BK && total <= 3 * a.E * a.n_tiles;
  const int run = static_cast<int>(gridDim.x >> 3);
  const int whole_runs = total / run;
  int block = first_tile / run, place = first_tile - block * run;
  auto list_entry = [&]() __attribute__((always_inline)) {
    if (block >= whole_runs) return tile;
    return (mix ? ((block & 1) ? whole_runs - 1 - (block >> 1) : (block >> 1)) : block) * run + place;
  };
  if (tile < total) {
    TileState cur;
    setup_tile(list_entry(), cur);
    first_loads(cur);
    for (;;) {
      last_first_loads(cur);
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
      run_main(cur);
      wg_barrier();                             // every wave is done with the operand tiles
      bool weighted = (MODE == DGRAD_H_GATE);
      if constexpr (MODE == GATE_UP) weighted = a.row_weight != nullptr;
      if constexpr (MODE == GATE_UP || MODE == DGRAD_H_GATE) {
        if (weighted) fetch_row_weights(cur, a.row_weight);
      }
      Finished done{cur.e, cur.m0, cur.n0, cur.r0, cur.m_wave, 0, 4, cur.second};
      tile += gridDim.x;
      const bool more = tile < total;
      if (more) {
        block += 8;
        place = place + 1 == run ? 0 : place + 1;
        setup_tile(list_entry(), cur);
        done.slot = __builtin_amdgcn_readfirstlane(spare_slot(cur));
        if constexpr (is_dgrad_h(MODE)) done.slot2 = __builtin_amdgcn_readfirstlane(spare_slot2(cur));
      }
      if constexpr (MODE == GATE_UP || MODE == DGRAD_H_GATE) {
        // (a use that the compiler sees: left to the epilogue, its wait would cover the first loads too)
#pragma unroll
        for (int i = 0; i < NB; ++i) asm volatile("" : "+v"(wv[i]));
      }
      if (more) first_loads(cur);
      epilogue(done);
      // a wave stages in, and loads into, its own share of a slot only: no barrier between epilogue and later loads
      if (!more) break;
    }
  }
  return tile - total;
}

// The launch is persistent: gridDim.x workgroups (one per compute unit) walk the tile list.
// Workgroups are dealt to the 8 XCDs round-robin, so workgroup b takes position
// (b % 8) * (gridDim.x / 8) + b / 8 of every round: each XCD then works on a run of
// consecutive tiles (same expert, neighbouring panels) that share its L2.
__device__ __forceinline__ int first_list_position() {
  const int per_xcd = gridDim.x >> 3;
  return (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
}

template <int MODE, int S>
__global__ __launch_bounds__(GEMM_THREADS, Tile<S>::PER_CU) void grouped_gemm_kernel(GemmArgs a) {
  gemm_tile_list<MODE, S, 0>(a, first_list_position());
}

// Two products that do not depend on each other in one launch: the tile list of the second follows
// that of the first, so the workgroups that run out of tiles of the first go on with the second
// instead of idling until the next launch (one tail and one start-up instead of two).
template <int MODE_A, int MODE_B, int S>
__global__ __launch_bounds__(GEMM_THREADS, Tile<S>::PER_CU) void grouped_gemm_pair_kernel(GemmArgs a, GemmArgs b) {
  const int next = gemm_tile_list<MODE_A, S, 0>(a, first_list_position());
  gemm_tile_list<MODE_B, S, 1>(b, next);
}

// Per-device facts, looked up once per device: HIP keeps function attributes and the number of compute
// units per device, and a process may drive several.  Races between host threads are benign (both write
// the same values).
constexpr int MAX_DEVICES = 64;
int current_device() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); dev = 0; }
  return dev >= 0 && dev < MAX_DEVICES ? dev : 0;
}
// Workgroups of the persistent launch: as many per compute unit as the LDS allows (one or two),
// a multiple of 8 so that every XCD gets the same share, and no more than there can be tiles.
int compute_units() {
  static int cus_of[MAX_DEVICES] = {};
  const int dev = current_device();
  int cus = cus_of[dev];
  if (cus == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 8) {
      (void)hipGetLastError();
      n = 256;
    }
    cus = cus_of[dev] = n & ~7;
  }
  return cus;
}
template <int S> int persistent_grid(long long max_tiles) {
  const int most = Tile<S>::PER_CU * compute_units();
  long long g = (max_tiles + 7) & ~7ll;
  if (g > most) g = most;
  if (g < 8) g = 8;
  return static_cast<int>(g);
}
// Raises the kernel's dynamic-LDS limit on the current device, once per device.
template <typename K>
int configure_lds(K kernel, int bytes, bool (&done)[MAX_DEVICES]) {
  const int dev = current_device();
  if (done[dev]) return MOE_OK;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) !=
      hipSuccess) {
    (void)hipGetLastError();
    return MOE_ERR_LAUNCH;
  }
  done[dev] = true;
  return MOE_OK;
}

template <int MODE, int S>
int launch_gemm(const GemmArgs& a, long long max_tiles, hipStream_t s, const char* name) {
  const dim3 grid(persistent_grid<S>(max_tiles));
  static bool configured[MAX_DEVICES] = {};
  if (configure_lds(&grouped_gemm_kernel<MODE, S>, Tile<S>::LDS, configured) != MOE_OK) return MOE_ERR_LAUNCH;
  MOE_LAUNCH(name, (grouped_gemm_kernel<MODE, S>), grid, dim3(GEMM_THREADS), Tile<S>::LDS, s, a);
  return moe_check_launch();
}

template <int MODE_A, int MODE_B, int S>
int launch_gemm_pair(const GemmArgs& a, const GemmArgs& b, long long max_tiles, hipStream_t s, const char* name) {
  const dim3 grid(persistent_grid<S>(max_tiles));
  static bool configured[MAX_DEVICES] = {};
  if (configure_lds(&grouped_gemm_pair_kernel<MODE_A, MODE_B, S>, Tile<S>::LDS, configured) != MOE_OK) return MOE_ERR_LAUNCH;
  MOE_LAUNCH(name, (grouped_gemm_pair_kernel<MODE_A, MODE_B, S>), grid, dim3(GEMM_THREADS), Tile<S>::LDS, s, a, b);
  return moe_check_launch();
}

// The launches fill in what depends on the tile's edge: column tiles, row tiles and the bound on the tile list.
int ceil_div(int n, int by) { return (n + by - 1) / by; }
template <int MODE, int S>
long long count_tiles(GemmArgs& a, int R_cap) {
  if constexpr (is_wgrad(MODE)) {
    a.n_tiles = ceil_div(a.N, S);
    a.m_tiles_cap = ceil_div(a.M, S);         // row tiles of one expert's dW
    return static_cast<long long>(a.n_tiles) * a.m_tiles_cap * a.E * (a.A1 != nullptr ? 2 : 1);
  } else {
    a.n_tiles = ceil_div(a.N, MODE == GATE_UP ? S / 2 : S);
    a.m_tiles_cap = R_cap / S + a.E;
    return static_cast<long long>(a.n_tiles) * a.m_tiles_cap;
  }
}

// Which tile edge a launch takes: the one for which the model below expects less time.  Both give the same bits.
//
// 256: half the operand bytes per operation, and what long lists are quickest with.  128: two workgroups share a compute
// unit, so that one's waits and epilogue lie under the other's main loop; four times the tiles, so that a short list still
// reaches every compute unit; a quarter of the epilogue behind the last step of a reduction of a few; half the padding where
// experts have few rows or d, f are no multiple of 256.
//
// The model, in units of one K step of a 256-edge tile (1.4 us): a tile costs something fixed (start, epilogue) and something
// per step.  A launch takes its tiles' sum, spread over the places of the chip, plus one tile of the longest kind, since a list
// rarely ends evenly; a list alone in its launch also ends on whole rounds.  The row tiles are counted for an even load of
// the expected rows; RAGGED is what the last one of an expert counts for.  The constants are a fit to 7700 layers of 64 to 12000
// tokens, d and f 128 to 4096, 4 to 240 experts, all or a share of them local, even and zipf-like loads (four launches each, timed
// with both edges).  On 26900 others the edge chosen is on average 1.05 % slower than the better one (gate_up 0.8, down 0.7, dgrad_h with dWd 1.05, dgrad_x
// with dWg and dWu 1.6), always 256 17 % slower, always 128 4 %; constants fitted to these themselves reach 1.0 %.  In 4 % of the launches it is wrong by
// 10 % or more: under 100 rows per expert weight gradients of narrow layers, and a share of the
// experts that holds the large ones of a skewed load, whose rows are far more than expected.  (The constants before, a fit to 152 layers, are 1.23 % off
// on the same 26900, 10 % or more in 5 %; a layer's four launches together gain 2 to 7 % over them in one of twenty, lose 4 % in one of a hundred.)
// Some of them, 256 / 128 in us, gate_up, down, dgrad_h with dWd, dgrad_x with dWg and dWu:
//   256 tokens, d 128, f 256, 8 experts, 2 per token        11 / 9      10 / 8      16 / 11     13 / 10
//   248 tokens, d 320, f 320, 28 of 57 experts, 6           13 / 11     11 / 9      15 / 13     23 / 19
//   7380 tokens, d 512, f 1600, 19 of 39 experts, 2         44 / 58     42 / 34     77 / 57     97 / 89
//   2000 tokens, d 1024, f 512, 128 experts, 8              76 / 83     43 / 46     85 / 112   152 / 164
//   1500 tokens, d 2048, f 1024, 64 experts, 8             156 / 166    72 / 84    165 / 196   312 / 361
//   2048 tokens of the same layer                          163 / 204    91 / 110   222 / 245   350 / 422
//   8192 tokens of the same layer                          470 / 646   263 / 324   557 / 683   876 / 1214
template <int S> struct TileCost;
template <> struct TileCost<256> { static constexpr double FIXED = 5.2, WGRAD = 6.0, STEP = 1.0, SWIGLU_BWD = 16.0, RAGGED = 0.5; };
template <> struct TileCost<128> { static constexpr double FIXED = 2.7, WGRAD = 3.8, STEP = 0.75, SWIGLU_BWD = 9.0, RAGGED = 0.8; };
struct ListCost { double tiles, each; };
// rows: routed rows to expect
template <int MODE, int S>
ListCost list_cost(const GemmArgs& a, double rows) {
  const double r = rows / a.E;
  if (is_wgrad(MODE)) {
    const double steps = r / BK + 0.5 > 1.0 ? r / BK + 0.5 : 1.0;
    return {static_cast<double>(a.E) * ceil_div(a.M, S) * ceil_div(a.N, S) * (a.A1 != nullptr ? 2 : 1),
            TileCost<S>::WGRAD + 1.1 * TileCost<S>::STEP * steps};
  }
  const double row_tiles = a.E * (r < 1.0 ? r : 1.0) * (r / S + TileCost<S>::RAGGED > 1.0 ? r / S + TileCost<S>::RAGGED : 1.0);
  return {row_tiles * ceil_div(a.N, MODE == GATE_UP ? S / 2 : S),
          TileCost<S>::FIXED + (is_dgrad_h(MODE) ? TileCost<S>::SWIGLU_BWD : 0.0) +
              TileCost<S>::STEP * (a.K / BK) * (MODE == DGRAD_X ? 2 : 1)};
}
template <int S> double places() { return static_cast<double>(Tile<S>::PER_CU) * compute_units(); }
template <int S> double launch_cost(const ListCost& l) {
  const double rounds = l.tiles / places<S>();
  const long long whole = static_cast<long long>(rounds + 0.95);      // a twentieth of a round too many does not count
  return 0.6 * (0.9 * rounds * l.each + l.each) + 0.4 * (whole < 1 ? 1 : whole) * l.each;
}
template <int S> double launch_cost(const ListCost& l, const ListCost& m) {
  return 0.65 * (l.tiles * l.each + m.tiles * m.each) / places<S>() + (l.each > m.each ? l.each : m.each);
}

// edge: null, or in: the edge to take (0: the rule's), out: the edge taken
bool take_small(int* edge, double small, double large) {
  const bool is_small = edge != nullptr && *edge != 0 ? *edge == 128 : small < large;
  if (edge != nullptr) *edge = is_small ? 128 : 256;
  return is_small;
}
template <int MODE>
int run_gemm(GemmArgs& a, int R_cap, long long rows, hipStream_t s, const char* name, int* edge) {
  const double r = static_cast<double>(rows);
  if (take_small(edge, launch_cost<128>(list_cost<MODE, 128>(a, r)), launch_cost<256>(list_cost<MODE, 256>(a, r)))) {
    const long long tiles = count_tiles<MODE, 128>(a, R_cap);
    return launch_gemm<MODE, 128>(a, tiles, s, name);
  }
  const long long tiles = count_tiles<MODE, 256>(a, R_cap);
  return launch_gemm<MODE, 256>(a, tiles, s, name);
}
template <int MODE_A, int MODE_B>
int run_gemm_pair(GemmArgs& a, GemmArgs& b, int R_cap, long long rows, hipStream_t s, const char* name, int* edge) {
  const double r = static_cast<double>(rows);
  if (take_small(edge, launch_cost<128>(list_cost<MODE_A, 128>(a, r), list_cost<MODE_B, 128>(b, r)),
                 launch_cost<256>(list_cost<MODE_A, 256>(a, r), list_cost<MODE_B, 256>(b, r)))) {
    const long long tiles = count_tiles<MODE_A, 128>(a, R_cap) + count_tiles<MODE_B, 128>(b, R_cap);
    return launch_gemm_pair<MODE_A, MODE_B, 128>(a, b, tiles, s, name);
  }
  const long long tiles = count_tiles<MODE_A, 256>(a, R_cap) + count_tiles<MODE_B, 256>(b, R_cap);
  return launch_gemm_pair<MODE_A, MODE_B, 256>(a, b, tiles, s, name);
}
bool bad_edges(const int* edges) {
  if (edges == nullptr) return false;
  for (int i = 0; i < 2; ++i) if (edges[i] != 0 && edges[i] != 128 && edges[i] != 256) return true;
  return false;
}

bool bad_gemm_dims(int E, int R_cap, int d, int f) {
  return E <= 0 || E > MOE_MAX_EXPERTS || R_cap <= 0 || d <= 0 || f <= 0 || d % 64 != 0 || f % 64 != 0;
}

inline const uint16_t* U16(const moe_bf16* p) { return p; }

}  // namespace

extern "C" size_t moe_grouped_gemm_bwd_workspace_bytes(int R_cap, int f) {
  if (R_cap <= 0 || f <= 0) return 0;
  const size_t one = (static_cast<size_t>(R_cap) * f * sizeof(moe_bf16) + 255) & ~static_cast<size_t>(255);
  return 2 * one;
}

extern "C" size_t moe_workspace_bytes(int T, int E, int k, int d, int f) {
  if (T <= 0 || k <= 0 || E <= 0 || d <= 0 || f <= 0) return 0;
  const unsigned long long rows = static_cast<unsigned long long>(T) * static_cast<unsigned long long>(k);
  if (rows > 0x7FFFFFFFull) return 0;   // no call takes that many routed rows
  const int R_cap = static_cast<int>(rows);
  // the largest of every workspace any call may ask for on a layer of this shape
  const size_t sizes[] = {moe_permute_workspace_bytes(T, k, E), moe_grouped_gemm_bwd_workspace_bytes(R_cap, f),
                          moe_grouped_gemm_bwd_folded_workspace_bytes(R_cap, f), moe_router_bwd_workspace_bytes(T, d, E)};
  size_t m = 0;
  for (size_t v : sizes) m = v > m ? v : m;
  return m;
}

// xp grouped rows, or (row_token not null) the token rows themselves, gathered by the GEMM's loads
extern "C" int moe_gemm_fwd(const moe_bf16* xp, const int32_t* row_token, const float* row_weight, const int32_t* expert_offsets, const moe_bf16* Wg,
                 const moe_bf16* Wu, const moe_bf16* Wd, int E, int R_cap, long long rows, int most, int d, int f,
                 moe_bf16* g, moe_bf16* u, moe_bf16* h, moe_bf16* yp, void* stream, int* edges) {
  if (!xp || !expert_offsets || !Wg || !Wu || !Wd || !g || !u || !h || !yp) return MOE_ERR_INVALID;
  if (bad_gemm_dims(E, R_cap, d, f) || bad_edges(edges)) return MOE_ERR_INVALID;
  const void* ptrs[] = {xp, expert_offsets, Wg, Wu, Wd, g, u, h, yp};
  for (const void* p : ptrs) if (!moe_aligned16(p)) return MOE_ERR_INVALID;
  hipStream_t s = static_cast<hipStream_t>(stream);
  // Few rows for certain: the streaming kernels.  Few rows expected, but not for certain (a rank's share of the experts): both,
  // and on the device one of the two finds that the rows are not for it (see small_gemm.h).
  const int few = STREAM_ROWS * E;
  const bool tiled = edges != nullptr && (edges[0] != 0 || edges[1] != 0);
  const bool streamed = !tiled && (R_cap <= few || most <= STREAM_TOKENS), either = !tiled && !streamed && rows <= few;
  int rc = MOE_OK;
  StreamFwdArgs p{}, q{};
  if (streamed || either) {
    p.A = U16(xp); p.row_token = row_token; p.row_weight = row_weight; p.offsets = expert_offsets;
    p.B0 = U16(Wg); p.B1 = U16(Wu); p.O0 = g; p.O1 = u; p.O2 = h; p.E = E; p.K = d; p.N = f;
    q.A = U16(h); q.offsets = expert_offsets; q.B0 = U16(Wd); q.O0 = yp; q.E = E; q.K = f; q.N = d;
    p.max_rows = q.max_rows = either ? few : R_cap;
    if ((rc = moe_stream_gate_up(p, rows, s)) != MOE_OK) return rc;
    if (streamed) return moe_stream_down(q, rows, s);
  }
  GemmArgs a{};
  a.offsets = expert_offsets; a.E = E; a.row_token = row_token; a.row_weight = row_weight;
  // gate | up with the SwiGLU epilogue
  a.A0 = U16(xp); a.B0 = U16(Wg); a.B1 = U16(Wu); a.O0 = g; a.O1 = u; a.O2 = h;
  a.K = d; a.N = f;
  a.stream_rows = either ? few : 0;
  rc = run_gemm<GATE_UP>(a, R_cap, rows, s, "gemm_gate_up", edges);
  if (rc != MOE_OK) return rc;
  // down
  if (either && (rc = moe_stream_down(q, rows, s)) != MOE_OK) return rc;
  GemmArgs b{};
  b.offsets = expert_offsets; b.E = E;
  b.A0 = U16(h); b.B0 = U16(Wd); b.O0 = yp;
  b.K = f; b.N = d;
  b.stream_rows = a.stream_rows;
  return run_gemm<DOWN>(b, R_cap, rows, s, "gemm_down", edges != nullptr ? edges + 1 : nullptr);
}

namespace {
// byte offsets of gathered rows are 32-bit lane offsets from the start of x (T*width*2 bytes just under 4 GiB at most)
bool bad_gather(const moe_bf16* x, int T, const int32_t* row_token, int width) {
  return !x || !row_token || T <= 0 || !moe_aligned16(row_token) ||
         static_cast<unsigned long long>(T) * width * sizeof(moe_bf16) > 0xFFFFFFFFull - 65536;   // lane offsets carry a small bias on top
}
}  // namespace

// x, row_token: rows gathered; row_weight (or null): gate weights folded into h.  No expert has more rows than
// there are tokens, since a token's experts are distinct.
int moe_gemm_fwd_gather(const moe_bf16* x, int T, const int32_t* row_token, const float* row_weight, const int32_t* expert_offsets,
                        const moe_bf16* Wg, const moe_bf16* Wu, const moe_bf16* Wd, int E, int R_cap, long long rows, int d,
                        int f, moe_bf16* g, moe_bf16* u, moe_bf16* h, moe_bf16* yp, void* stream) {
  if (bad_gather(x, T, row_token, d)) return MOE_ERR_INVALID;
  return moe_gemm_fwd(x, row_token, row_weight, expert_offsets, Wg, Wu, Wd, E, R_cap, rows, T, d, f, g, u, h, yp, stream);
}

extern "C" int moe_grouped_gemm_fwd(const moe_bf16* xp, const int32_t* expert_offsets, const moe_bf16* Wg,
                                    const moe_bf16* Wu, const moe_bf16* Wd, int E, int R_cap, int d, int f,
                                    moe_bf16* g, moe_bf16* u, moe_bf16* h, moe_bf16* yp, void* stream) {
  return moe_gemm_fwd(xp, nullptr, nullptr, expert_offsets, Wg, Wu, Wd, E, R_cap, R_cap, R_cap, d, f, g, u, h, yp, stream);
}

extern "C" int moe_grouped_gemm_fwd_gather(const moe_bf16* x, int T, const int32_t* row_token,
                                           const int32_t* expert_offsets, const moe_bf16* Wg, const moe_bf16* Wu,
                                           const moe_bf16* Wd, int E, int R_cap, int d, int f, moe_bf16* g,
                                           moe_bf16* u, moe_bf16* h, moe_bf16* yp, void* stream) {
  return moe_gemm_fwd_gather(x, T, row_token, nullptr, expert_offsets, Wg, Wu, Wd, E, R_cap, R_cap, d, f, g, u, h, yp, stream);
}

extern "C" int moe_grouped_gemm_fwd_folded(const moe_bf16* x, int T, const int32_t* row_token, const float* row_weight,
                                           const int32_t* expert_offsets, const moe_bf16* Wg, const moe_bf16* Wu,
                                           const moe_bf16* Wd, int E, int R_cap, int d, int f, moe_bf16* g,
                                           moe_bf16* u, moe_bf16* hw, moe_bf16* ypw, void* stream) {
  if (!row_weight || !moe_aligned16(row_weight)) return MOE_ERR_INVALID;
  return moe_gemm_fwd_gather(x, T, row_token, row_weight, expert_offsets, Wg, Wu, Wd, E, R_cap, R_cap, d, f, g, u, hw, ypw,
                             stream);
}

// xp grouped rows, or (row_token not null) the token rows themselves, gathered by the loads of the
// two weight-gradient products that read them
extern "C" int moe_gemm_bwd(const moe_bf16* dyp, const moe_bf16* xp, int T, const int32_t* row_token, const moe_bf16* g, const moe_bf16* u,
                 const moe_bf16* h, const int32_t* expert_offsets, const moe_bf16* Wg, const moe_bf16* Wu,
                 const moe_bf16* Wd, int E, int R_cap, long long rows, int d, int f, moe_bf16* dxp, moe_bf16* dWg,
                 moe_bf16* dWu, moe_bf16* dWd, void* ws, size_t ws_bytes, void* stream, int* edges) {
  if ((row_token != nullptr && bad_gather(xp, T, row_token, d)) || bad_edges(edges)) return MOE_ERR_INVALID;
  if (!dyp || !xp || !g || !u || !h || !expert_offsets || !Wg || !Wu || !Wd || !dxp || !dWg || !dWu || !dWd || !ws)
    return MOE_ERR_INVALID;
  if (bad_gemm_dims(E, R_cap, d, f)) return MOE_ERR_INVALID;
  const void* ptrs[] = {dyp, xp, g, u, h, expert_offsets, Wg, Wu, Wd, dxp, dWg, dWu, dWd, ws};
  for (const void* p : ptrs) if (!moe_aligned16(p)) return MOE_ERR_INVALID;
  if (ws_bytes < moe_grouped_gemm_bwd_workspace_bytes(R_cap, f)) return MOE_ERR_WORKSPACE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  uint16_t* dg = static_cast<uint16_t*>(ws);
  uint16_t* du = reinterpret_cast<uint16_t*>(static_cast<char*>(ws) + moe_grouped_gemm_bwd_workspace_bytes(R_cap, f) / 2);

  // Two launches of two independent products each (the second list of a launch takes over the workgroups
  // that the first leaves idle at its end).
  // dh = dyp . Wd, then the SwiGLU derivative -> dg, du (first: its tiles are the long ones) ; dWd = dyp^T h
  GemmArgs wd{};
  wd.offsets = expert_offsets; wd.E = E;
  wd.A0 = U16(dyp); wd.B0 = U16(h); wd.O0 = dWd; wd.M = d; wd.N = f;
  GemmArgs a{};
  a.offsets = expert_offsets; a.E = E;
  a.A0 = U16(dyp); a.B0 = U16(Wd); a.G = U16(g); a.U = U16(u); a.O0 = dg; a.O1 = du;
  a.K = d; a.N = f;
  int rc = run_gemm_pair<DGRAD_H, WGRAD>(a, wd, R_cap, rows, s, "gemm_dgrad_h+wgrad_down", edges);
  if (rc != MOE_OK) return rc;
  // dxp = dg . Wg + du . Wu ; dWg = dg^T xp and dWu = du^T xp (one list: both read the same rows of xp)
  GemmArgs w{};
  w.offsets = expert_offsets; w.E = E; w.row_token = row_token;
  w.A0 = dg; w.A1 = du; w.B0 = U16(xp); w.O0 = dWg; w.O1 = dWu; w.M = f; w.N = d;
  GemmArgs b{};
  b.offsets = expert_offsets; b.E = E;
  b.A0 = dg; b.A1 = du; b.B0 = U16(Wg); b.B1 = U16(Wu); b.O0 = dxp;
  b.K = f; b.N = d;
  // dgrad_x first: its tiles are the long ones, the weight gradients' many short tiles fill its tail
  int* edge = edges != nullptr ? edges + 1 : nullptr;
  if (row_token != nullptr) return run_gemm_pair<DGRAD_X, WGRAD_GATHER>(b, w, R_cap, rows, s, "gemm_wgrad_gate_up+dgrad_x", edge);
  return run_gemm_pair<DGRAD_X, WGRAD>(b, w, R_cap, rows, s, "gemm_wgrad_gate_up+dgrad_x", edge);
}

extern "C" int moe_grouped_gemm_bwd(const moe_bf16* dyp, const moe_bf16* xp, const moe_bf16* g, const moe_bf16* u,
                                    const moe_bf16* h, const int32_t* expert_offsets, const moe_bf16* Wg,
                                    const moe_bf16* Wu, const moe_bf16* Wd, int E, int R_cap, int d, int f,
                                    moe_bf16* dxp, moe_bf16* dWg, moe_bf16* dWu, moe_bf16* dWd, void* ws,
                                    size_t ws_bytes, void* stream) {
  return moe_gemm_bwd(dyp, xp, 0, nullptr, g, u, h, expert_offsets, Wg, Wu, Wd, E, R_cap, R_cap, d, f, dxp, dWg, dWu, dWd,
                      ws, ws_bytes, stream);
}

extern "C" int moe_grouped_gemm_bwd_gather(const moe_bf16* dyp, const moe_bf16* x, int T, const int32_t* row_token,
                                           const moe_bf16* g, const moe_bf16* u, const moe_bf16* h,
                                           const int32_t* expert_offsets, const moe_bf16* Wg, const moe_bf16* Wu,
                                           const moe_bf16* Wd, int E, int R_cap, int d, int f, moe_bf16* dxp,
                                           moe_bf16* dWg, moe_bf16* dWu, moe_bf16* dWd, void* ws, size_t ws_bytes,
                                           void* stream) {
  if (row_token == nullptr) return MOE_ERR_INVALID;
  return moe_gemm_bwd(dyp, x, T, row_token, g, u, h, expert_offsets, Wg, Wu, Wd, E, R_cap, R_cap, d, f, dxp, dWg, dWu, dWd,
                      ws, ws_bytes, stream);
}

// ---------------------------------------------------------------------------------------------
// Backward of a forward pass that folded the gate weights into h (moe_grouped_gemm_fwd_folded).
namespace {
// dgate[t, i] = sum over the column strips of the row's partial dot products (0 for a slot without a local row)
__global__ __launch_bounds__(256) void dgate_finish_kernel(const float* __restrict__ part, int strips,
                                                           const int32_t* __restrict__ slot_row, int n,
                                                           float* __restrict__ dgate) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= n) return;
  const int row = slot_row[idx];
  float sum = 0.f;
  if (row >= 0) {
    const float* p = part + static_cast<size_t>(row) * strips;
    for (int c = 0; c < strips; ++c) sum += p[c];
  }
  dgate[idx] = sum;
}

size_t folded_part_bytes(int R_cap, int f) {
  return (static_cast<size_t>(f / 64) * R_cap * sizeof(float) + 255) & ~static_cast<size_t>(255);
}
}  // namespace

extern "C" size_t moe_grouped_gemm_bwd_folded_workspace_bytes(int R_cap, int f) {
  if (R_cap <= 0 || f <= 0) return 0;
  return moe_grouped_gemm_bwd_workspace_bytes(R_cap, f) + folded_part_bytes(R_cap, f);
}

const float* moe_folded_part(const void* ws, int R_cap, int f) {
  return reinterpret_cast<const float*>(static_cast<const char*>(ws) + moe_grouped_gemm_bwd_workspace_bytes(R_cap, f));
}

extern "C" int moe_gemm_bwd_folded(const moe_bf16* dout, const moe_bf16* x, int T, int k,
                                           const int32_t* row_token, const float* row_weight, const int32_t* slot_row,
                                           const moe_bf16* g, const moe_bf16* u, const moe_bf16* hw,
                                           const int32_t* expert_offsets, const moe_bf16* Wg, const moe_bf16* Wu,
                                           const moe_bf16* Wd, int E, int R_cap, long long rows, int d, int f, moe_bf16* dxp,
                                           moe_bf16* dWg, moe_bf16* dWu, moe_bf16* dWd, float* dgate, void* ws,
                                           size_t ws_bytes, void* stream, int* edges) {
  if (!dout || !g || !u || !hw || !expert_offsets || !Wg || !Wu || !Wd || !dxp || !dWg || !dWu || !dWd || !ws || !row_weight || !slot_row || k <= 0)
    return MOE_ERR_INVALID;
  if (bad_gemm_dims(E, R_cap, d, f) || bad_gather(x, T, row_token, d) || bad_gather(dout, T, row_token, d) || bad_edges(edges))
    return MOE_ERR_INVALID;
  const void* ptrs[] = {dout, x, g, u, hw, expert_offsets, Wg, Wu, Wd, dxp, dWg, dWu, dWd, dgate, ws, row_weight, slot_row};
  for (const void* p : ptrs) if (!moe_aligned16(p)) return MOE_ERR_INVALID;
  if (ws_bytes < moe_grouped_gemm_bwd_folded_workspace_bytes(R_cap, f)) return MOE_ERR_WORKSPACE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const size_t one = moe_grouped_gemm_bwd_workspace_bytes(R_cap, f) / 2;
  uint16_t* dg = static_cast<uint16_t*>(ws);
  uint16_t* du = reinterpret_cast<uint16_t*>(static_cast<char*>(ws) + one);
  float* part = const_cast<float*>(moe_folded_part(ws, R_cap, f));

  // Two launches of two independent products each (the second list of a launch takes over the workgroups
  // that the first leaves idle at its end).
  // dh0 = dout[token] . Wd; dh = w dh0 -> dg, du; partial dot products of dh0 with h for the gate gradient
  // (first: its tiles are the long ones);
  // dWd = (w dout[token])^T h = dout[token]^T hw: rows of dout gathered by the loads of the A operand
  GemmArgs wd{};
  wd.offsets = expert_offsets; wd.E = E; wd.row_token = row_token;
  wd.A0 = U16(dout); wd.B0 = U16(hw); wd.O0 = dWd; wd.M = d; wd.N = f;
  GemmArgs a{};
  a.offsets = expert_offsets; a.E = E; a.row_token = row_token; a.row_weight = row_weight;
  a.dgate_part = part;
  a.A0 = U16(dout); a.B0 = U16(Wd); a.G = U16(g); a.U = U16(u); a.O0 = dg; a.O1 = du;
  a.K = d; a.N = f;
  int rc = run_gemm_pair<DGRAD_H_GATE, WGRAD_GATHER_A>(a, wd, R_cap, rows, s, "gemm_dgrad_h+wgrad_down", edges);
  if (rc != MOE_OK) return rc;
  if (dgate != nullptr) {
    const int n = T * k;
    MOE_LAUNCH("dgate_finish", dgate_finish_kernel, dim3((n + 255) / 256), dim3(256), 0, s, static_cast<const float*>(part),
               f / 64, slot_row, n, dgate);
  }
  // dWg = dg^T x[token] and dWu = du^T x[token] (one list: both read the same gathered rows of x), then
  // dxp = dg . Wg + du . Wu
  GemmArgs w{};
  w.offsets = expert_offsets; w.E = E; w.row_token = row_token;
  w.A0 = dg; w.A1 = du; w.B0 = U16(x); w.O0 = dWg; w.O1 = dWu; w.M = f; w.N = d;
  GemmArgs b{};
  b.offsets = expert_offsets; b.E = E;
  b.A0 = dg; b.A1 = du; b.B0 = U16(Wg); b.B1 = U16(Wu); b.O0 = dxp;
  b.K = f; b.N = d;
  // dgrad_x first: its tiles are the long ones, the weight gradients' many short tiles fill its tail.  (The other
  // order used to pay off through dxp still lying in the last-level cache when moe_permute_bwd read it; since that
  // kernel streams its rows with non-temporal loads it no longer depends on that.)
  return run_gemm_pair<DGRAD_X, WGRAD_GATHER>(b, w, R_cap, rows, s, "gemm_wgrad_gate_up+dgrad_x",
                                              edges != nullptr ? edges + 1 : nullptr);
}

extern "C" int moe_grouped_gemm_bwd_folded(const moe_bf16* dout, const moe_bf16* x, int T, int k,
                                           const int32_t* row_token, const float* row_weight, const int32_t* slot_row,
                                           const moe_bf16* g, const moe_bf16* u, const moe_bf16* hw,
                                           const int32_t* expert_offsets, const moe_bf16* Wg, const moe_bf16* Wu,
                                           const moe_bf16* Wd, int E, int R_cap, int d, int f, moe_bf16* dxp,
                                           moe_bf16* dWg, moe_bf16* dWu, moe_bf16* dWd, float* dgate, void* ws,
                                           size_t ws_bytes, void* stream) {
  if (!dgate) return MOE_ERR_INVALID;
  return moe_gemm_bwd_folded(dout, x, T, k, row_token, row_weight, slot_row, g, u, hw, expert_offsets, Wg, Wu, Wd, E, R_cap,
                             R_cap, d, f, dxp, dWg, dWu, dWd, dgate, ws, ws_bytes, stream);
}
