// bf16 products with few rows per weight matrix: the experts' forward in a decode step, and the router's logits.
//
//   UP     h1|h3 = xp [W1|W3] -> a = silu(h1) h3     per expert, up to 64 rows at a time
//   DOWN   o     = a W2
//   RL     logits = x Wr (fp32)                       one "expert" of T rows
//   RW     dWr = x^T dlogits (fp32 partial sums)      x streams in the weights' place, the contraction runs over the tokens
//                                                     and the rows are the experts (launch_router_dw_small)
//
// What bounds it: reading the weights once (a row of a decode step multiplies each of them once or a few times), so the
// kernel is a stream of weights with the matrix instruction at its end.  256x256 tiles leave most of the chip idle here (four
// active experts of width 1536 are 48 of them) and carry the weights through LDS; this kernel has
//   * blocks of 64+64 (UP) or 128 columns whose eight wavefronts share the contraction: wavefront w takes the 32-deep pieces
//     w, w+8, ..; the eight partial results are added in LDS in ascending order;
//   * weights that go from memory to registers in 16-byte pieces of whole rows (256 bytes per row and wavefront) and are
//     transposed there: lane (i, g) loads columns 8i..8i+7 of rows 8g..8g+7 of a piece, which is an 8 x 8 block, and 32 byte
//     permutes turn it into the operands of eight 16x16x32 matrix instructions, the j-th of which computes columns 8i+j;
//   * two to four pieces (8 KB each) in flight per wavefront.
// The weights are the instruction's first operand and the rows its second, so that 16 rows cost one instruction per eight
// columns and lane.
#include "common.h"
#include "kernels.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

enum { UP, DOWN, RL, RW };

constexpr int COLS = 128;                 // columns of a block (UP: 64 of W1 and the same 64 of W3)
constexpr int ROWS = 64;                  // rows of a block at most
constexpr int KP = 32;                    // depth of a piece
constexpr int RPITCH = COLS + 4;          // partial results in LDS: [wavefront][16 rows][RPITCH]
constexpr int NW_EXPERT = 4, NW_ROUTER = 8;      // wavefronts per block

struct SArgs {
  const bf16_t* A; long lda;
  const bf16_t* B0; const bf16_t* B1; long ldb, b_es;
  bf16_t* C0; bf16_t* C1; bf16_t* C2;     // UP: h1, h3 (both or neither), a; DOWN: o in C0
  float* F;                               // RL
  long ldc;
  const int32_t* off;                     // NULL (RL): one expert of `rows` rows
  int rows, e_cnt, N, K;
  long xstep;                             // elements from a row's piece to its next piece
  int n_experts;                          // RW: rows are (plane, expert), expert fastest
  int range;                              // RL, RW: pieces of the contraction per range (grid z); range z's sums go to F + z * rows * N
};

// Loads go through a buffer descriptor: a wave-uniform base and a 32-bit byte offset per lane.  With 64-bit addresses per
// lane a CU's address path limits it to about 27 bytes per cycle, half of what this form reaches.  A descriptor of length
// zero makes a load return zeros without touching memory: pieces past the end of a wavefront's share are issued that way,
// which keeps the number of loads, and so the wait counts, the same for every piece.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t descriptor(const bf16_t* base, bool in) {
  uint64_t b = (uint64_t)base;
  int bytes = in ? 0x7FFFFFFF : 0;
  asm("" : "+s"(b), "+s"(bytes));         // both are wave-uniform: keep them in scalar registers
  return __builtin_amdgcn_make_buffer_rsrc((void*)b, 0, bytes, 0x00027000);
}

// Weights of one piece, 32 rows of 128 columns, as loaded, and the operand of matrix instruction j made from them.
// row: bytes per weight row; voff: this lane's offset
struct PieceWide {                        // one matrix: lane (i, g) holds columns 8i..8i+7 of rows 8g..8g+7
  u32x4 w[8];
  __device__ __forceinline__ void load(const bf16_t* b0, const bf16_t*, bool in, int row, int voff) {
    const __amdgpu_buffer_rsrc_t d = descriptor(b0, in);
#pragma unroll
    for (int r = 0; r < 8; ++r) w[r] = __builtin_amdgcn_raw_buffer_load_b128(d, voff, r * row, 0);
  }
  __device__ __forceinline__ bf16x8 operand(int j) const {
    u32x4 f;
#pragma unroll
    for (int q = 0; q < 4; ++q)           // k elements 2q, 2q+1 of column j
      f[q] = __builtin_amdgcn_perm(w[2 * q + 1][j >> 1], w[2 * q][j >> 1], (j & 1) ? 0x07060302u : 0x05040100u);
    return __builtin_bit_cast(bf16x8, f);
  }
};
struct PieceDual {                        // 64 columns of each of two matrices: lane (i, g) holds columns 4i..4i+3 of both
  u32x2 w[2][8];
  __device__ __forceinline__ void load(const bf16_t* b0, const bf16_t* b1, bool in, int row, int voff) {
    const __amdgpu_buffer_rsrc_t d0 = descriptor(b0, in), d1 = descriptor(b1, in);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      w[0][r] = __builtin_amdgcn_raw_buffer_load_b64(d0, voff, r * row, 0);
      w[1][r] = __builtin_amdgcn_raw_buffer_load_b64(d1, voff, r * row, 0);
    }
  }
  __device__ __forceinline__ bf16x8 operand(int j) const {      // j = 0..3: first matrix, 4..7: second
    u32x4 f;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      f[q] = __builtin_amdgcn_perm(w[j >> 2][2 * q + 1][(j >> 1) & 1], w[j >> 2][2 * q][(j >> 1) & 1], (j & 1) ? 0x07060302u : 0x05040100u);
    return __builtin_bit_cast(bf16x8, f);
  }
};

template <bool DUAL> struct PickPiece { typedef PieceWide type; };
template <> struct PickPiece<true> { typedef PieceDual type; };

template <int MODE, int TG, int NW>
__device__ __forceinline__ void tile(const SArgs& p, float* red, int e, int row0, int row_end, int n0, int first, int pieces,
                                     int tid) {
  constexpr bool DUAL = MODE == UP;
  constexpr int DEPTH = TG == 1 ? 4 : (TG == 2 ? 3 : 2);        // pieces in flight
  typedef typename PickPiece<DUAL>::type Piece;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, g = lane >> 4;
  f32x4 acc[TG][8];
#pragma unroll
  for (int t = 0; t < TG; ++t)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  {
    const bf16_t* b0 = p.B0 + (size_t)e * p.b_es + n0;
    const bf16_t* b1 = DUAL ? p.B1 + (size_t)e * p.b_es + n0 : b0;
    const bf16_t* xrow = p.A + (size_t)row0 * p.lda;
    // columns and rows past the end repeat the last ones
    const int woff = 2 * (8 * g * (int)p.ldb + (DUAL ? 4 * i : min(8 * i, p.N - n0 - 8)));
    int xoff[TG];
#pragma unroll
    for (int t = 0; t < TG; ++t) xoff[t] = 2 * (min(16 * t + i, row_end - row0 - 1) * (int)p.lda + 8 * g);
    const int n = (pieces - wave + NW - 1) / NW;                // pieces of this wavefront
    Piece w[DEPTH];
    bf16x8 x[DEPTH][TG];
    auto load = [&](auto slot, int idx) {
      constexpr int S = decltype(slot)::value;
      const bool in = idx < n;
      const long piece = in ? first + wave + NW * idx : 0;
      const long k = MODE == RW ? min(piece * KP, (long)p.K - KP) : piece * KP;      // RW: the last piece ends at the last token
      w[S].load(b0 + k * p.ldb, b1 + k * p.ldb, in, 2 * (int)p.ldb, woff);
      const __amdgpu_buffer_rsrc_t dx = descriptor(xrow + piece * p.xstep, in);
#pragma unroll
      for (int t = 0; t < TG; ++t) x[S][t] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(dx, xoff[t], 0, 0));
      __builtin_amdgcn_sched_barrier(0);  // pieces stay in order: waiting for one must not wait for the next
    };
    static_for<DEPTH>([&](auto s) { load(s, decltype(s)::value); });
    for (int idx = 0; idx < n; idx += DEPTH)
      static_for<DEPTH>([&](auto s) {
        constexpr int S = decltype(s)::value;
        if (idx + S < n) {
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const bf16x8 f = w[S].operand(j);
#pragma unroll
            for (int t = 0; t < TG; ++t) acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, x[S][t], acc[t][j], 0, 0, 0);
          }
        }
        load(s, idx + DEPTH + S);
      });
  }
  // Add the partial results up, 16 rows at a time.  Element r of acc[t][j] belongs to row 16t + i and lane group 4g + r of
  // the loads: column 8 * (4g + r) + j, in UP column 4 * (4g + r) + j % 4 of matrix j / 4 (kept 64 columns further on).
  constexpr int PER = 16 * COLS / (NW * WAVE);                  // columns per thread
#pragma unroll
  for (int t = 0; t < TG; ++t) {
    if (t > 0) __syncthreads();
    float* mine = red + (wave * 16 + i) * RPITCH;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        *reinterpret_cast<f32x4*>(mine + (DUAL ? 64 * h + 4 * (4 * g + r) : 8 * (4 * g + r) + 4 * h)) =
            f32x4{acc[t][4 * h][r], acc[t][4 * h + 1][r], acc[t][4 * h + 2][r], acc[t][4 * h + 3][r]};
    __syncthreads();
    if (MODE == RW) {                                           // [column][expert], one plane after the other; rows fastest
      const int r = tid & 15, row = row0 + 16 * t + r;
      if (row < row_end) {
        const int plane = row / p.n_experts;
        float* out = p.F + (size_t)plane * p.N * p.n_experts + (row - plane * p.n_experts);
        for (int c = tid >> 4; c < COLS && n0 + c < p.N; c += NW * WAVE / 16) {
          float v = 0.f;
#pragma unroll
          for (int wv = 0; wv < NW; ++wv) v += red[(wv * 16 + r) * RPITCH + c];
          out[(size_t)(n0 + c) * p.n_experts] = v;
        }
      }
      continue;
    }
    const int rr = tid / (COLS / PER), c = tid % (COLS / PER);  // row of the group, column group
    const int row = row0 + 16 * t + rr;
    // this thread's columns: PER / 2 from each half of a row (UP: h1 | h3), or PER in a row
    float v[2][PER / 2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float* q = red + rr * RPITCH + (DUAL ? 64 * h + PER / 2 * c : PER * c + PER / 2 * h);
#pragma unroll
      for (int k = 0; k < PER / 2; ++k) v[h][k] = 0.f;
#pragma unroll
      for (int wv = 0; wv < NW; ++wv)
#pragma unroll
        for (int k = 0; k < PER / 2; ++k) v[h][k] += q[wv * 16 * RPITCH + k];
    }
    const int col = n0 + (DUAL ? PER / 2 : PER) * c;
    if (row >= row_end || col >= p.N) continue;
    const size_t idx = (size_t)row * p.ldc + col;
    if (MODE == RL) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int k = 0; k < PER / 2; ++k) p.F[idx + PER / 2 * h + k] = v[h][k];
    } else {
      uint32_t o[2][PER / 4], a[PER / 4];
#pragma unroll
      for (int k = 0; k < PER / 4; ++k) {
        o[0][k] = pack_bf16x2(v[0][2 * k], v[0][2 * k + 1]);
        o[1][k] = pack_bf16x2(v[1][2 * k], v[1][2 * k + 1]);
        if (DUAL) a[k] = pack_bf16x2(silu_f(v[0][2 * k]) * v[1][2 * k], silu_f(v[0][2 * k + 1]) * v[1][2 * k + 1]);
      }
#pragma unroll
      for (int k = 0; k < PER / 4; ++k) {
        if (DUAL) {
          if (p.C0) {
            reinterpret_cast<uint32_t*>(p.C0 + idx)[k] = o[0][k];
            reinterpret_cast<uint32_t*>(p.C1 + idx)[k] = o[1][k];
          }
          reinterpret_cast<uint32_t*>(p.C2 + idx)[k] = a[k];
        } else {
          reinterpret_cast<uint32_t*>(p.C0 + idx)[k] = o[0][k];
          reinterpret_cast<uint32_t*>(p.C0 + idx)[PER / 4 + k] = o[1][k];
        }
      }
    }
  }
}

template <int MODE>
__global__ __launch_bounds__(NW_EXPERT * WAVE, 2) void small_rows(SArgs p) {
  __shared__ __align__(16) float red[NW_EXPERT * 16 * RPITCH];
  const int tid = threadIdx.x;
  int e, mt, nt;
  if (!ragged_tile<ROWS>(p.off, p.e_cnt, (p.N + (MODE == UP ? 63 : COLS - 1)) / (MODE == UP ? 64 : COLS), blockIdx.x, tid & 63, e, mt, nt)) return;
  const int row0 = p.off[e] + mt * ROWS, row_end = min(p.off[e + 1], row0 + ROWS);
  const int n0 = nt * (MODE == UP ? 64 : COLS);
  const int rows = row_end - row0;
  if (rows <= 16) tile<MODE, 1, NW_EXPERT>(p, red, e, row0, row_end, n0, 0, p.K / KP, tid);
  else if (rows <= 32) tile<MODE, 2, NW_EXPERT>(p, red, e, row0, row_end, n0, 0, p.K / KP, tid);
  else tile<MODE, 4, NW_EXPERT>(p, red, e, row0, row_end, n0, 0, p.K / KP, tid);
}

// grid = (row blocks of 16 * TG, column blocks, ranges of the contraction)
template <int MODE, int TG>
__global__ __launch_bounds__(NW_ROUTER * WAVE) void small_rows_router(SArgs p) {
  __shared__ __align__(16) float red[NW_ROUTER * 16 * RPITCH];
  const int row0 = blockIdx.x * 16 * TG, first = blockIdx.z * p.range;
  p.F += (size_t)blockIdx.z * p.rows * p.N;
  tile<MODE, TG, NW_ROUTER>(p, red, 0, row0, min(p.rows, row0 + 16 * TG), blockIdx.y * COLS, first,
                            min(p.range, (p.K + KP - 1) / KP - first), threadIdx.x);
}

template <int MODE>
int launch_small(const SArgs& p, int cap, int prof_id, hipStream_t s) {
  const long long cols = MODE == UP ? p.N / 64 : (p.N + COLS - 1) / COLS;
  const long long blocks = (((long long)cap / ROWS + (cap < p.e_cnt ? cap : p.e_cnt)) * cols + 7) / 8 * 8;
  if (blocks >= (1ll << 31)) return MOE_EUNSUPPORTED;
  ProfScope prof(prof_id, s);
  hipLaunchKernelGGL(small_rows<MODE>, dim3((unsigned)blocks), dim3(NW_EXPERT * WAVE), 0, s, p);
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}

}  // namespace

int launch_expert_fwd_small(const void* xp, int cap, int d, int f, int e_cnt, const int32_t* offsets, const void* w1,
                            const void* w3, const void* w2, void* h1, void* h3, void* a, void* o, hipStream_t s) {
  SArgs u = {};
  u.A = (const bf16_t*)xp; u.lda = d;
  u.B0 = (const bf16_t*)w1; u.B1 = (const bf16_t*)w3; u.ldb = f; u.b_es = (long)d * f;
  u.C0 = (bf16_t*)h1; u.C1 = (bf16_t*)h3; u.C2 = (bf16_t*)a; u.ldc = f; u.xstep = KP;
  u.off = offsets; u.e_cnt = e_cnt; u.N = f; u.K = d;
  int rc = launch_small<UP>(u, cap, MOE_K_UP, s);
  if (rc) return rc;
  SArgs w = {};
  w.A = (const bf16_t*)a; w.lda = f;
  w.B0 = (const bf16_t*)w2; w.ldb = d; w.b_es = (long)f * d;
  w.C0 = (bf16_t*)o; w.ldc = d; w.xstep = KP;
  w.off = offsets; w.e_cnt = e_cnt; w.N = d; w.K = f;
  return launch_small<DOWN>(w, cap, MOE_K_DOWN, s);
}

// partials: room for max_ranges * T * E floats.  Returns the number of ranges through `ranges`: 1 = the logits are
// complete, else the partial sums in `partials` are still to be added up.
int launch_router_fwd_small(const void* x, const void* wr, int T, int d, int E, float* logits, float* partials, int max_ranges,
                            int* ranges, hipStream_t s) {
  SArgs p = {};
  p.A = (const bf16_t*)x; p.lda = d;
  p.B0 = (const bf16_t*)wr; p.ldb = E;
  p.ldc = E; p.rows = T; p.e_cnt = 1; p.N = E; p.K = d; p.xstep = KP;
  const int cols = (E + COLS - 1) / COLS, cus = device_cu_count(), pieces = d / KP;
  // as many rows per block as still leave a block for every CU: the weights are read once per block
  const int tg = (long long)(T + 63) / 64 * cols >= cus ? 4 : ((long long)(T + 31) / 32 * cols >= cus ? 2 : 1);
  const int row_blocks = (T + 16 * tg - 1) / (16 * tg);
  // A CU takes about 65 GB/s of weights, so a handful of blocks is cut along the contraction (at least two pieces per
  // wavefront); the second launch that adds the ranges up pays from three ranges on.
  int n = cus / (cols * row_blocks);
  if (n > max_ranges) n = max_ranges;
  if (n > pieces / (2 * NW_ROUTER)) n = pieces / (2 * NW_ROUTER);
  if (n < 3) n = 1;
  p.range = (pieces + n - 1) / n;
  n = (pieces + p.range - 1) / p.range;
  p.F = n > 1 ? partials : logits;
  *ranges = n;
  const dim3 grid(row_blocks, cols, n), block(NW_ROUTER * WAVE);
  ProfScope prof(MOE_K_ROUTER_FWD, s);
  if (tg == 4) hipLaunchKernelGGL((small_rows_router<RL, 4>), grid, block, 0, s, p);
  else if (tg == 2) hipLaunchKernelGGL((small_rows_router<RL, 2>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((small_rows_router<RL, 1>), grid, block, 0, s, p);
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}

// dlogits as router_dw_operand lays them out: [pieces][planes * E][32].  Partial sums go to partials[ranges * planes][d][E]
// (range by range, plane by plane); at most max_sums of them.  T >= 32.
int launch_router_dw_small(const void* x, const void* dl_pieces, int planes, int T, int d, int E, float* partials, int max_sums,
                           int* sums, hipStream_t s) {
  SArgs p = {};
  p.A = (const bf16_t*)dl_pieces; p.lda = KP; p.rows = planes * E; p.xstep = (long)planes * E * KP; p.n_experts = E;
  p.B0 = (const bf16_t*)x; p.ldb = d;
  p.F = partials; p.N = d; p.K = T;
  const int cols = (d + COLS - 1) / COLS, pieces = (T + KP - 1) / KP;
  const int tg = p.rows <= 16 ? 1 : (p.rows <= 32 ? 2 : 4);
  const int row_blocks = (p.rows + 16 * tg - 1) / (16 * tg);
  // a block for every CU, but at least two pieces per wavefront and no more sums than there is room for
  int n = device_cu_count() / (cols * row_blocks);
  if (n > max_sums / planes) n = max_sums / planes;
  if (n > pieces / (2 * NW_ROUTER)) n = pieces / (2 * NW_ROUTER);
  if (n < 1) n = 1;
  p.range = (pieces + n - 1) / n;
  n = (pieces + p.range - 1) / p.range;
  *sums = n * planes;
  const dim3 grid(row_blocks, cols, n), block(NW_ROUTER * WAVE);
  ProfScope prof(MOE_K_ROUTER_DW, s);
  if (tg == 4) hipLaunchKernelGGL((small_rows_router<RW, 4>), grid, block, 0, s, p);
  else if (tg == 2) hipLaunchKernelGGL((small_rows_router<RW, 2>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((small_rows_router<RW, 1>), grid, block, 0, s, p);
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}
