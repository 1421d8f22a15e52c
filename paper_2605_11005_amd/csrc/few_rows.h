// The experts' forward with few rows per weight matrix: a tile of it, for the kernels of expert_small.hip and of
// expert_bf16.hip.
#pragma once
#include "common.h"
#include "stream_rule.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int COLS = 128;                 // columns of a block (UP: 64 of W1 and the same 64 of W3)
constexpr int ROWS = 64;                  // rows of an expert block at most
constexpr int KP = 32;                    // depth of a piece
constexpr int NW_TILES = 4;                // wavefronts of a block that also runs the 256x256 tiles

struct SArgs {
  const bf16_t* A; long lda;
  const bf16_t* B0; const bf16_t* B1; long ldb, b_es;
  bf16_t* C0; bf16_t* C1; bf16_t* C2;     // UP: h1, h3 (both or neither), a; DOWN: o in C0
  float* F;                               // RL, RW
  long ldc;
  const int32_t* off;                     // UP, DOWN
  int rows, e_cnt, N, K;
  long xstep;                             // RW: elements from a row's piece to its next piece
  int n_experts;                          // RW: rows are (plane, expert), expert fastest
  int cached;                             // UP, DOWN: cached_experts
  int range;                              // RL, RW: pieces of the contraction per range (grid z); range z's sums go to F + z * rows * N
                                          // narrow_router: rows per block; UP, DOWN: most tiles that are halved
};

// Loads go through a buffer descriptor: a wave-uniform base and a 32-bit byte offset per lane (64-bit addresses per lane limit
// a CU's address path, see lds_load16 in common.h).  A descriptor of length
// zero makes a load return zeros without touching memory: pieces past the end of a wavefront's share are issued that way,
// which keeps the number of loads, and so the wait counts, the same for every piece.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t descriptor(const bf16_t* base, bool in) {
  uint64_t b = (uint64_t)base;
  int bytes = in ? 0x7FFFFFFF : 0;
  asm("" : "+s"(b), "+s"(bytes));         // both are wave-uniform: keep them in scalar registers
  return __builtin_amdgcn_make_buffer_rsrc((void*)b, 0, bytes, 0x00027000);
}

// A wavefront's piece of a weight matrix as loaded: a lane holds an 8 x 8 block, 16 bytes of each of eight rows.
struct Piece {
  u32x4 w[8];
  // row: bytes per weight row; voff: this lane's offset
  template <int FIRST, int END, bool STREAM = false>
  __device__ __forceinline__ void load(const bf16_t* base, bool in, int row, int voff) {      // rows FIRST .. END - 1 of the eight
    constexpr int NT = STREAM ? 2 : 0;      // "nt": the line is used once
    const __amdgpu_buffer_rsrc_t d = descriptor(base, in);
#pragma unroll
    for (int r = FIRST; r < END; ++r) w[r] = __builtin_amdgcn_raw_buffer_load_b128(d, voff, r * row, NT);
  }
  __device__ __forceinline__ bf16x8 operand(int j) const {      // column j of the block, its eight k
    u32x4 f;
#pragma unroll
    for (int q = 0; q < 4; ++q)           // k elements 2q, 2q+1
      f[q] = __builtin_amdgcn_perm(w[2 * q + 1][j >> 1], w[2 * q][j >> 1], (j & 1) ? 0x07060302u : 0x05040100u);
    return __builtin_bit_cast(bf16x8, f);
  }
};

// Which of the 512 places (16 bytes: eight k of one column) of 32 k by 128 columns in LDS holds k chunk g of column c: 16
// columns and one chunk fill 256 bytes, and the XOR keeps both the 16 columns of a fragment (consecutive) and the 16 lanes of
// a store (columns 8 apart, in UP over two chunks) on different banks.
__device__ __forceinline__ int place(int c, int g) { return 16 * (4 * (c >> 4) + g) + ((c & 15) ^ (c >> 4) ^ ((g & 1) << 2)); }

// UP, DOWN: up to 16 * TG rows of one expert against 32 * NW columns (UP: 16 * NW of either matrix).  The NW wavefronts share the
// loads, in rounds of 128 k: with four of them wavefront w fetches in DOWN 32 k of the 128 columns, in UP 64 k of the 64 columns of
// matrix w % 2; with two it is 64 k and 128 k of half as many columns.  It hands the operands over through LDS, with its share of
// the rows' k.  Each wavefront then multiplies its own 32 columns (UP: 16 of either matrix) through the
// round's steps in ascending order, so that an output is one chain of sums over ascending k.  It is the chain of the 256x256
// tiles: a 16x16x32 instruction gives the bits of two 32x32x16 ones, in either order of the operands.  The forward's results
// therefore do not depend on which of the two kernels a call takes, which the caller's capacity decides.
// Two LDS buffers: a round's operands are stored before the round in front of it is multiplied, one barrier per round.
// Forward of both GEMMs, d = 4096, f = 1536, 16 experts of which four have rows (4, 2, 1 and 1): 46 us where UP loads 8 bytes
// per lane from both matrices, 42 with 16 bytes from one, 39 with the loads that refill the registers issued in two parts
// beside the LDS reads of the multiplication, 38 as it is now: one block per CU (96 KB of LDS see to it) with two rounds on
// their way.  More are no faster: 32 experts of 1 row, d = 7168, f = 2048, take 489 / 493 / 497 us with two / three / four
// rounds, 513 us with three and two blocks per CU.
constexpr int STEPS = 4;                   // of 32 k, per round
template <int NW> constexpr int STEP_PLACES = KP * 32 * NW / 8;
template <int NW> constexpr int WEIGHT_PLACES = STEPS * STEP_PLACES<NW>;
constexpr int ROW_PLACES = STEPS * ROWS / 16 * WAVE;
template <bool DUAL, int TG, int NW, bool STREAM>
__device__ __forceinline__ void expert_tile(const SArgs& p, u32x4* lds, int e, int row0, int row_end, int n0, int tid) {
  constexpr int DEPTH = 2, XS = STEPS / NW;           // XS: steps of the rows per wavefront
  constexpr int CHUNKS = (DUAL ? 2 : 4) * NW;         // of 8 columns, in a row of a wavefront's piece
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, g = lane >> 4;
  // weights: lane (ci, kg) loads columns 8 ci .. 8 ci + 7 of rows 8 kg .. 8 kg + 7
  const int ci = lane % CHUNKS, kg = lane / CHUNKS;
  const int wk0 = DUAL ? (NW == 4 ? wave & 2 : 0) : XS * wave;        // first step of this wavefront's piece in a round
  const bf16_t* b = (DUAL && (wave & 1) ? p.B1 : p.B0) + (size_t)e * p.b_es + n0;
  const bf16_t* xrow = p.A + (size_t)row0 * p.lda;
  // columns and rows past the end repeat the last ones
  const int wcol = 2 * min(8 * ci, p.N - n0 - 8);
  int xoff[TG];
#pragma unroll
  for (int t = 0; t < TG; ++t) xoff[t] = 2 * (min(16 * t + i, row_end - row0 - 1) * (int)p.lda + 8 * g);
  const int steps = p.K / KP, rounds = (steps + STEPS - 1) / STEPS;       // of 32 k; of 128 k
  Piece w[DEPTH];
  u32x4 x[DEPTH][XS][TG];
  auto load = [&](auto slot, int round, auto half) {
    constexpr int S = decltype(slot)::value, H = decltype(half)::value;
    const int wk = STEPS * round + wk0;           // (steps is even: of a round there are four, two or none)
    // rows past the contraction repeat its last ones (their steps are not multiplied)
    const int woff = min(8 * kg, max(8, KP * (steps - wk)) - 8) * 2 * (int)p.ldb + wcol;
    w[S].template load<4 * H, 4 * H + 4, STREAM>(b + (wk < steps ? (long)wk * KP : 0) * p.ldb, wk < steps, 2 * (int)p.ldb, woff);
    if (H) {
#pragma unroll
      for (int q = 0; q < XS; ++q) {
        const int xk = STEPS * round + XS * wave + q;
        const __amdgpu_buffer_rsrc_t dx = descriptor(xrow + (xk < steps ? xk * KP : 0), xk < steps);
#pragma unroll
        for (int t = 0; t < TG; ++t) x[S][q][t] = __builtin_amdgcn_raw_buffer_load_b128(dx, xoff[t], 0, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);    // loads stay in order: waiting for one round must not wait for the next
  };
  u32x4* const xlds = lds + 2 * WEIGHT_PLACES<NW>;
  auto publish = [&](auto slot, int round) {
    constexpr int S = decltype(slot)::value;
    u32x4* buf = lds + (round & 1) * WEIGHT_PLACES<NW> + (wk0 + (kg >> 2)) * STEP_PLACES<NW>;
#pragma unroll
    for (int j = 0; j < 8; ++j)           // (in UP the second matrix's columns are kept behind the first one's)
      buf[place((DUAL ? 16 * NW * (wave & 1) : 0) + 8 * ci + j, kg & 3)] = __builtin_bit_cast(u32x4, w[S].operand(j));
#pragma unroll
    for (int q = 0; q < XS; ++q)
#pragma unroll
      for (int t = 0; t < TG; ++t) xlds[(round & 1) * ROW_PLACES + ((XS * wave + q) * TG + t) * WAVE + lane] = x[S][q][t];
    __builtin_amdgcn_sched_barrier(0);
  };
  f32x4 acc[2][TG];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int t = 0; t < TG; ++t) acc[c][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int col0 = DUAL ? 16 * wave : 32 * wave, col1 = DUAL ? 16 * NW + col0 : col0 + 16;
  bf16x8 f[2][2], r[2][TG];
  auto read = [&](int round, int q0) {    // operands of steps q0, q0 + 1 of a round
    const u32x4* buf = lds + (round & 1) * WEIGHT_PLACES<NW>;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      f[q][0] = __builtin_bit_cast(bf16x8, buf[(q0 + q) * STEP_PLACES<NW> + place(col0 + i, g)]);
      f[q][1] = __builtin_bit_cast(bf16x8, buf[(q0 + q) * STEP_PLACES<NW> + place(col1 + i, g)]);
#pragma unroll
      for (int t = 0; t < TG; ++t) r[q][t] = __builtin_bit_cast(bf16x8, xlds[(round & 1) * ROW_PLACES + ((q0 + q) * TG + t) * WAVE + lane]);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto multiply = [&]() {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int t = 0; t < TG; ++t)
#pragma unroll
        for (int c = 0; c < 2; ++c) acc[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[q][c], r[q][t], acc[c][t], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  // one round: slot `next` holds the one after it (zeros after the last), and is refilled
  auto step = [&](auto next, int round, bool refill) {
    publish(next, round + 1);
    read(round, 0);
    if (refill) load(next, round + 1 + DEPTH, Int<0>{});
    multiply();
    // the last round has four steps or two, and multiplying the others' zeros could turn a -0 into +0
    const bool full = steps - STEPS * round >= STEPS;
    if (full) read(round, 2);
    if (refill) load(next, round + 1 + DEPTH, Int<1>{});
    if (full) multiply();
    __syncthreads();
  };
  static_for<DEPTH>([&](auto s) {
    load(s, decltype(s)::value, Int<0>{});
    load(s, decltype(s)::value, Int<1>{});
  });
  publish(Int<0>{}, 0);
  load(Int<0>{}, DEPTH, Int<0>{});
  load(Int<0>{}, DEPTH, Int<1>{});
  __syncthreads();
  int round = 0;
  for (; round + DEPTH <= rounds; round += DEPTH)
    static_for<DEPTH>([&](auto s) { step(Int<(decltype(s)::value + 1) % DEPTH>{}, round + decltype(s)::value, true); });
  static_for<DEPTH - 1>([&](auto s) {     // what is left is on its way
    constexpr int S = decltype(s)::value;
    if (round + S < rounds) step(Int<S + 1>{}, round + S, false);
  });
  // element r of acc[c][t] is row 16t + i, column 4g + r of the wavefront's c-th 16 columns
#pragma unroll
  for (int t = 0; t < TG; ++t) {
    const int row = row0 + 16 * t + i;
    if (row >= row_end) continue;
    const f32x4 u = acc[0][t], v = acc[1][t];
    const u32x2 o0 = {pack_bf16x2(u[0], u[1]), pack_bf16x2(u[2], u[3])}, o1 = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
    const size_t at = (size_t)row * p.ldc + n0 + 4 * g;
    if (DUAL) {
      const u32x2 a = {pack_bf16x2(silu_f(u[0]) * v[0], silu_f(u[1]) * v[1]), pack_bf16x2(silu_f(u[2]) * v[2], silu_f(u[3]) * v[3])};
      if (p.C0) {
        *reinterpret_cast<u32x2*>(p.C0 + at + 16 * wave) = o0;
        *reinterpret_cast<u32x2*>(p.C1 + at + 16 * wave) = o1;
      }
      *reinterpret_cast<u32x2*>(p.C2 + at + 16 * wave) = a;
    } else if (n0 + 32 * wave < p.N) {    // N % 64 == 0: a wavefront's 32 columns are all in or all out
      *reinterpret_cast<u32x2*>(p.C0 + at + 32 * wave) = o0;
      *reinterpret_cast<u32x2*>(p.C0 + at + 32 * wave + 16) = o1;
    }
  }
}

// Tile b of a launch over all experts; false: the list is shorter.  MAY_STREAM: the experts may not fit the Infinity Cache (stream_rule.h).
template <int NW> constexpr int FEW_ROWS_PLACES = 2 * (WEIGHT_PLACES<NW> + ROW_PLACES);      // LDS, 16 bytes each
template <bool DUAL, int NW, bool STREAM>
__device__ __forceinline__ void sized_tile(const SArgs& p, u32x4* lds, int e, int row0, int row_end, int n0, int tid) {
  const int rows = row_end - row0;
  if (rows <= 16) expert_tile<DUAL, 1, NW, STREAM>(p, lds, e, row0, row_end, n0, tid);
  else if (rows <= 32) expert_tile<DUAL, 2, NW, STREAM>(p, lds, e, row0, row_end, n0, tid);
  else expert_tile<DUAL, 4, NW, STREAM>(p, lds, e, row0, row_end, n0, tid);
}
template <bool DUAL, int NW, bool MAY_STREAM>
__device__ __forceinline__ bool few_rows_tile(const SArgs& p, const RaggedTiles<ROWS>& list, u32x4* lds, int b) {
  constexpr int WIDTH = (DUAL ? 16 : 32) * NW;
  const int tid = threadIdx.x;
  int e, mt, nt;
  if (!list.tile((p.N + WIDTH - 1) / WIDTH, b, e, mt, nt)) return false;
  const int first = p.off[e], end = p.off[e + 1], row0 = first + mt * ROWS, row_end = min(end, row0 + ROWS);
  if (MAY_STREAM && stream_weights(list.active, p.cached, end - first, ROWS)) sized_tile<DUAL, NW, true>(p, lds, e, row0, row_end, nt * WIDTH, tid);
  else sized_tile<DUAL, NW, false>(p, lds, e, row0, row_end, nt * WIDTH, tid);
  return true;
}

}  // namespace
