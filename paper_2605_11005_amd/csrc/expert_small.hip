// bf16 products with few rows per weight matrix: the experts' forward in a decode step, and the router's logits.
//
//   UP     h1|h3 = xp [W1|W3] -> a = silu(h1) h3     per expert, up to 64 rows at a time
//   DOWN   o     = a W2
//   RL     logits = x Wr (fp32)                       one "expert" of T rows
//   RW     dWr = x^T dlogits (fp32 partial sums)      x streams in the weights' place, the contraction runs over the tokens
//                                                     and the rows are the experts (launch_router_dw_small)
//
// What bounds it: reading the weights once (a row of a decode step multiplies each of them once or a few times), so the
// kernels are a stream of weights with the matrix instruction at its end.  256x256 tiles leave most of the chip idle here
// (four active experts of width 1536 are 48 of them) and fetch a whole tile's rows for the few that are there.  Blocks cover
// 128 columns (UP: 64 of either matrix), and the weights go from memory to registers in 16-byte pieces and are transposed
// there: a lane loads eight columns of eight rows, and 32 byte permutes turn the 8 x 8 block into the operands of eight
// 16x16x32 matrix instructions.  The weights are the instruction's first operand and the rows its second, so that 16 rows
// cost one instruction per 16 columns and 32 k.
//   * UP, DOWN: four wavefronts that share the loads and multiply 32 columns each, every output one chain of sums over
//     ascending k (expert_tile);
//   * RL, RW: eight wavefronts that share the contraction, wavefront w the 32-deep pieces w, w + 8, .., two to four of them in flight; the
//     eight partial results are added in LDS in ascending order (router_logits, router_tile);
//   * RL with 8 to 56 experts: eight wavefronts with an eighth of the contraction each, eight sums per output (narrow_router).
#include "few_rows.h"
#include "kernels.h"

namespace {

enum { UP, DOWN };

constexpr int NW_ROUTER = 8;              // wavefronts per block
constexpr int RPITCH = COLS + 4;          // partial results in LDS: [wavefront][16 rows][RPITCH]

// RW: up to 16 * TG rows against COLS columns.  Wavefront w multiplies the pieces w, w + NW, .. of all columns, and the
// partial results are added in LDS in ascending order of the wavefronts.
template <int TG>
__device__ __forceinline__ void router_tile(const SArgs& p, float* red, int row0, int row_end, int n0, int first, int pieces, int tid) {
  constexpr int NW = NW_ROUTER;
  constexpr int DEPTH = TG == 1 ? 4 : (TG == 2 ? 3 : 2);        // pieces in flight
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, g = lane >> 4;
  f32x4 acc[TG][8];
#pragma unroll
  for (int t = 0; t < TG; ++t)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  {
    const bf16_t* b0 = p.B0 + n0;
    const bf16_t* xrow = p.A + (size_t)row0 * p.lda;
    // columns and rows past the end repeat the last ones
    const int woff = 2 * (8 * g * (int)p.ldb + min(8 * i, p.N - n0 - 8));
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
      const long k = min(piece * KP, (long)p.K - KP);               // the last piece ends at the last token
      w[S].template load<0, 8>(b0 + k * p.ldb, in, 2 * (int)p.ldb, woff);
      const __amdgpu_buffer_rsrc_t dx = descriptor(xrow + piece * p.xstep, in);
#pragma unroll
      for (int t = 0; t < TG; ++t) x[S][t] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(dx, xoff[t], 0, 0));
      __builtin_amdgcn_sched_barrier(0);  // pieces stay in order: waiting for one must not wait for the next
    };
    static_for<DEPTH>([&](auto s) { load(s, decltype(s)::value); });
    auto multiply = [&](auto slot) {
      constexpr int S = decltype(slot)::value;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const bf16x8 f = w[S].operand(j);
#pragma unroll
        for (int t = 0; t < TG; ++t) acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, x[S][t], acc[t][j], 0, 0, 0);
      }
    };
    int idx = 0;
    for (; idx + DEPTH < n; idx += DEPTH)
      static_for<DEPTH>([&](auto s) {
        multiply(s);
        load(s, idx + DEPTH + decltype(s)::value);
      });
    static_for<DEPTH>([&](auto s) {       // the last ones are on their way
      if (idx + decltype(s)::value < n) multiply(s);
    });
  }
  // Add the partial results up, 16 rows at a time.  Element r of acc[t][j] belongs to row 16t + i and lane group 4g + r of
  // the loads: column 8 * (4g + r) + j.
#pragma unroll
  for (int t = 0; t < TG; ++t) {
    if (t > 0) __syncthreads();
    float* mine = red + (wave * 16 + i) * RPITCH;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        *reinterpret_cast<f32x4*>(mine + 8 * (4 * g + r) + 4 * h) =
            f32x4{acc[t][4 * h][r], acc[t][4 * h + 1][r], acc[t][4 * h + 2][r], acc[t][4 * h + 3][r]};
    __syncthreads();
    const int r = tid & 15, row = row0 + 16 * t + r;            // [column][expert], one plane after the other; rows fastest
    if (row >= row_end) continue;
    const int plane = row / p.n_experts;
    float* out = p.F + (size_t)plane * p.N * p.n_experts + (row - plane * p.n_experts);
    for (int c = tid >> 4; c < COLS && n0 + c < p.N; c += NW * WAVE / 16) {
      float v = 0.f;
#pragma unroll
      for (int wv = 0; wv < NW; ++wv) v += red[(wv * 16 + r) * RPITCH + c];
      out[(size_t)(n0 + c) * p.n_experts] = v;
    }
  }
}

// RL: 16 * TG tokens against 16 * CL experts.  Wavefront w multiplies the pieces w, w + NW, .. of 32 k in one chain, and the partial
// results are added in LDS in ascending order of the wavefronts, so that neither TG nor CL changes a bit.  (Relative error of the logits,
// T, d, E: 2047, 2880, 128 11.8e-8; 1000, 7168, 256 18.0e-8; 300, 7168, 512 in three ranges 11.4e-8.)
// What bounds it is how a CU fetches x and the weights, at 60 to 85 GB/s.  Operands of x loaded where the instruction wants them, 16
// tokens by 64 bytes, touch a line with every lane of 16 and ask memory for half lines, so LDS turns them round:
//   * 16 tokens: four lanes load a token's 64 bytes, and a wavefront hands them over to itself;
//   * 32 and 64 tokens: wavefronts 2r and 2r + 1, whose pieces are the halves of the same 128 bytes, load whole lines of half of the tokens
//     each, for a barrier per piece (24.7 us for 26.4 without, T = 9001, d = 2880, E = 128; with 16 tokens 7.5 for 7.2, T = 4, 4096, 128).
// And nothing is asked for past the end: eight pieces of void loads were 1.5 us.  Calls in a captured graph, us, operands loaded
// directly by blocks of 128 experts / this:
//   T = 2047, d = 2880, E = 128 17.9 / 11.0    4096, 2048, 64 11.6 / 9.1    9001, 2880, 128 30.0 / 24.7     16384, 2048, 128 24.5 / 21.8
//   T = 128, d = 4096, E = 128 10.4 / 7.6      4, 4096, 128 8.9 / 6.3       4096, 7168, 256 43.8 / 37.2     8192, 4096, 64 25.6 / 19.9
template <int CL>
struct RouterPiece {                      // 32 k of the weights: a lane holds CL columns of eight rows
  typedef unsigned int vec __attribute__((ext_vector_type(CL / 2)));
  vec w[8];
  __device__ __forceinline__ void load(const bf16_t* base, bool in, int row, int voff) {
    const __amdgpu_buffer_rsrc_t d = descriptor(base, in);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      if constexpr (CL == 8) w[r] = __builtin_amdgcn_raw_buffer_load_b128(d, voff, r * row, 0);
      else w[r] = __builtin_amdgcn_raw_buffer_load_b64(d, voff, r * row, 0);
    }
  }
  __device__ __forceinline__ bf16x8 operand(int j) const {      // column j of the lane's, its eight k
    u32x4 f;
#pragma unroll
    for (int q = 0; q < 4; ++q) f[q] = __builtin_amdgcn_perm(w[2 * q + 1][j >> 1], w[2 * q][j >> 1], (j & 1) ? 0x07060302u : 0x05040100u);
    return __builtin_bit_cast(bf16x8, f);
  }
};

template <int TG, int CL>
__global__ __launch_bounds__(NW_ROUTER * WAVE) void router_logits(SArgs p) {
  constexpr int NW = NW_ROUTER, WIDTH = 16 * CL, PITCH = WIDTH + 4;
  constexpr bool SHARED = TG > 1;                               // two wavefronts load lines of x together
  // pieces in flight: more gain nothing (16 by 64: two 6.3 us, four 7.1, T = 4, d = 4096, E = 128; 32 by 128: two 24.0, three 25.1, T = 5000)
  constexpr int DEPTH = TG == 1 ? (CL == 8 ? 4 : 2) : (CL == 8 ? 2 : (TG == 2 ? 4 : 3));
  constexpr int BUFFER = NW * 64 * TG;                          // 16-byte places of a piece of all wavefronts
  constexpr int X_PLACES = SHARED ? 2 * BUFFER : BUFFER, SUM_PLACES = NW * 16 * PITCH / 4;
  __shared__ u32x4 lds[X_PLACES > SUM_PLACES ? X_PLACES : SUM_PLACES];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, g = lane >> 4, odd = wave & 1;
  const int row0 = blockIdx.x * 16 * TG, rows = min(p.rows - row0, 16 * TG), n0 = blockIdx.y * WIDTH;
  const int first = blockIdx.z * p.range, pieces = min(p.range, p.K / KP - first);
  const int n = (pieces - wave + NW - 1) / NW;                  // pieces of this wavefront
  const int steps = SHARED ? (pieces + NW - 1) / NW : n;        // SHARED: the same in all of them
  f32x4 acc[TG][CL];
#pragma unroll
  for (int t = 0; t < TG; ++t)
#pragma unroll
    for (int j = 0; j < CL; ++j) acc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  {
    const bf16_t* const b0 = p.B0 + n0;
    const bf16_t* const xrow = p.A + (size_t)row0 * p.lda;
    const int woff = 2 * (8 * g * (int)p.ldb + min(CL * i, p.N - n0 - CL));       // columns past the end repeat the last ones
    const int xoff = SHARED ? 2 * ((8 * odd + (lane >> 3)) * (int)p.lda + 8 * (lane & 7)) : 2 * ((lane >> 2) * (int)p.lda + 8 * (lane & 3));
    RouterPiece<CL> w[DEPTH];
    u32x4 x[DEPTH][TG];
    // Rows past the end are zeros: the descriptor ends there.  (SHARED: behind an odd number of pieces a line's second half is what
    // follows in memory, which its wavefront does not multiply.)
    auto load_x = [&](auto slot, int idx) {
      const int piece = NW * idx + (SHARED ? wave - odd : wave);
      const bool in = piece < pieces;
      const int k = in ? KP * (first + piece) : 0;
      uint64_t base = (uint64_t)(xrow + k);
      int bytes = in ? 2 * (rows * (int)p.lda - k) : 0, sixteen = 32 * (int)p.lda;
      asm("" : "+s"(base), "+s"(bytes), "+s"(sixteen));         // (the offsets are formed again each time: no registers are kept for them)
      const __amdgpu_buffer_rsrc_t d = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00027000);
#pragma unroll
      for (int t = 0; t < TG; ++t) x[decltype(slot)::value][t] = __builtin_amdgcn_raw_buffer_load_b128(d, xoff + t * sixteen, 0, 0);
      __builtin_amdgcn_sched_barrier(0);  // loads stay in order: waiting for one must not wait for the next
    };
    auto load_w = [&](auto slot, int idx) {
      const bool in = idx < n;
      const long k = in ? KP * (first + wave + NW * idx) : 0;
      w[decltype(slot)::value].load(b0 + k * p.ldb, in, 2 * (int)p.ldb, woff);
      __builtin_amdgcn_sched_barrier(0);
    };
    // token r's chunk c (eight k): the chunks of a token and the same chunk of eight tokens are on different banks
    const auto at = [](int r, int c) { return SHARED ? 8 * r + (c ^ (r & 7)) : 4 * r + (c ^ ((r >> 1) & 3)); };
    auto step = [&](auto slot, int idx, auto more) {
      constexpr int S = decltype(slot)::value;
      constexpr bool MORE = decltype(more)::value;
      u32x4* const mine = lds + (SHARED ? (idx & 1) * BUFFER + (wave >> 1) * 128 * TG : wave * 64 * TG);
#pragma unroll
      for (int t = 0; t < TG; ++t)
        mine[SHARED ? at(16 * t + 8 * odd + (lane >> 3), lane & 7) : at(16 * t + (lane >> 2), lane & 3)] = x[S][t];
      if constexpr (MORE) load_x(slot, idx + DEPTH);
      if constexpr (SHARED) __syncthreads();              // (two buffers: the next piece is written while this one is read)
      else __builtin_amdgcn_wave_barrier();               // LDS serves a wavefront's accesses in order
      if (!SHARED || idx < n) {
        bf16x8 f[TG];
#pragma unroll
        for (int t = 0; t < TG; ++t) f[t] = __builtin_bit_cast(bf16x8, mine[at(16 * t + i, SHARED ? 4 * odd + g : g)]);
#pragma unroll
        for (int j = 0; j < CL; ++j) {
          const bf16x8 c = w[S].operand(j);
#pragma unroll
          for (int t = 0; t < TG; ++t) acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(c, f[t], acc[t][j], 0, 0, 0);
        }
      }
      if constexpr (MORE) load_w(slot, idx + DEPTH);
      if constexpr (!SHARED) __builtin_amdgcn_wave_barrier();
    };
    static_for<DEPTH>([&](auto s) {
      load_x(s, decltype(s)::value);
      load_w(s, decltype(s)::value);
    });
    int idx = 0;
    for (; idx + DEPTH < steps; idx += DEPTH) static_for<DEPTH>([&](auto s) { step(s, idx + decltype(s)::value, Int<1>{}); });
    static_for<DEPTH>([&](auto s) {       // the last ones are on their way
      if (idx + decltype(s)::value < steps) step(s, idx + decltype(s)::value, Int<0>{});
    });
  }
  // Element r of acc[t][j] belongs to token 16t + i and lane group 4g + r of the loads: column CL * (4g + r) + j.
  float* const red = reinterpret_cast<float*>(lds);             // [wavefront][16 tokens][PITCH]
  float* const out = p.F + ((size_t)blockIdx.z * p.rows + row0) * p.N;
  constexpr int PER = 16 * WIDTH / (NW * WAVE);                 // columns per thread
  const int rr = tid / (WIDTH / PER), cc = PER * (tid % (WIDTH / PER));
#pragma unroll
  for (int t = 0; t < TG; ++t) {
    __syncthreads();
    float* const mine = red + (wave * 16 + i) * PITCH;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int h = 0; h < CL / 4; ++h)
        *reinterpret_cast<f32x4*>(mine + CL * (4 * g + r) + 4 * h) =
            f32x4{acc[t][4 * h][r], acc[t][4 * h + 1][r], acc[t][4 * h + 2][r], acc[t][4 * h + 3][r]};
    __syncthreads();
    float v[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) v[k] = 0.f;
#pragma unroll
    for (int wv = 0; wv < NW; ++wv)
#pragma unroll
      for (int k = 0; k < PER; ++k) v[k] += red[(wv * 16 + rr) * PITCH + cc + k];
    if (16 * t + rr >= rows || n0 + cc >= p.N) continue;
#pragma unroll
    for (int k = 0; k < PER; ++k) out[(size_t)(16 * t + rr) * p.N + n0 + cc + k] = v[k];
  }
}

// RL with fewer than 64 experts (E % 8 == 0).  Before there was a matrix-core kernel for them, a block of 256 threads took a
// token and added its products up in 256 chains and a tree, and the error of that is the measure here: a chain of matrix
// instructions, whose sums are not rounded to nearest, is up to 2.2 times further off (relative error of the logits at
// d = 512 / 2048 / 7168: 6.2 / 7.3 / 8.3e-8 with the block per token, 7.1 / 10.3 / 18e-8 with chains of d / 256 instructions
// and their eight results added in turn).  So every instruction starts from zero, its result goes to one of eight fp32
// sums per output by an ordinary addition, and these and the wavefronts' results are added in pairs: 6.1 / 7.2 / 8.1e-8.
// Wavefront w multiplies the w-th eighth of the contraction whatever T is: a token's logits do not depend on the batch.
// Loads: the 128 columns of router_tile would be up to 16 times the same ones.  A wavefront's piece is 8 KB of whole rows,
// 512 / G k of 8 G columns (G = 2, 4 or 8, from E / 8 on); a lane's 8 x 8 block is transposed in registers and goes to the
// lanes that want it through the wavefront's own LDS.
constexpr int SUMS = 8;
template <int TG, int G, int NG>          // NG: groups of 16 columns
__global__ __launch_bounds__(NW_ROUTER * WAVE) void narrow_router(SArgs p) {
  constexpr int NW = NW_ROUTER, STEPS = 16 / G;                 // steps of 32 k in a piece
  constexpr int SB = G == 2 ? 8 : 4;                            // steps whose rows are loaded at a time; two batches in flight
  constexpr int SLOTS = SB > STEPS ? SB / STEPS : 1;            // pieces that start in a batch
  constexpr int PLACES = 512;
  __shared__ u32x4 lds[NW * PLACES];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, g = lane >> 4, E = p.N;
  const int row0 = blockIdx.x * p.range, row_end = min(p.rows, row0 + p.range);      // up to 16 * TG rows
  const int units = p.K / 64, per = (units + NW - 1) / NW;
  const int first = 64 * min(wave * per, units), steps = 2 * (min((wave + 1) * per, units) - first / 64);
  u32x4* mine = lds + wave * PLACES;
  // place of k chunk kg (8 k) of column c in a piece: the 16 lanes of a store (columns 8 apart, chunks in turn) and of a fragment
  // (columns in turn) are on different banks
  const auto place = [](int c, int kg) {
    const int x = G == 2 ? kg : (G == 4 ? (c >> 4 & 1) | kg << 1 : (c >> 4 & 3) | kg << 2);
    return kg * 8 * G + (c & ~7) + ((c ^ x) & 7);
  };
  const int ci = lane % G, kg = lane / G;                       // weights: this lane's eight columns and eight k
  const int wcol = min(8 * ci, E - 8);                          // columns past the end repeat the last ones
  int xoff[TG];
#pragma unroll
  for (int t = 0; t < TG; ++t) xoff[t] = 2 * (min(16 * t + i, row_end - row0 - 1) * (int)p.lda + 8 * g);
  Piece w[SLOTS];
  auto load_w = [&](auto slot, int step) {      // the piece that starts at a step; chunks past the end repeat the last one
    const bool in = step < steps;
    const int last = in ? 4 * min(steps - step, STEPS) - 1 : 0;
    w[decltype(slot)::value].template load<0, 8>(p.B0 + (in ? (size_t)(first + step * KP) * E : 0), in, 2 * E, 2 * (8 * min(kg, last) * E + wcol));
    __builtin_amdgcn_sched_barrier(0);
  };
  u32x4 x[2][SB][TG];
  auto load_x = [&](auto set, int step) {
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int q = 0; q < SB; ++q) {
      const bool in = step + q < steps;
      const __amdgpu_buffer_rsrc_t d = descriptor(p.A + (size_t)row0 * p.lda + (in ? first + (step + q) * KP : 0), in);
#pragma unroll
      for (int t = 0; t < TG; ++t) x[S][q][t] = __builtin_amdgcn_raw_buffer_load_b128(d, xoff[t], 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 sum[NG][TG][SUMS];
#pragma unroll
  for (int n = 0; n < NG; ++n)
#pragma unroll
    for (int t = 0; t < TG; ++t)
#pragma unroll
      for (int k = 0; k < SUMS; ++k) sum[n][t][k] = zero;
  auto batch = [&](auto set, int step) {
    constexpr int S = decltype(set)::value;
    static_for<SB>([&](auto index) {
      constexpr int q = decltype(index)::value;
      if (step + q >= steps) return;
      if (q % STEPS == 0 && (step + q) % STEPS == 0) {
        constexpr int slot = q / STEPS;
#pragma unroll
        for (int j = 0; j < 8; ++j) mine[place(8 * ci + j, kg)] = __builtin_bit_cast(u32x4, w[slot].operand(j));
        __builtin_amdgcn_wave_barrier();  // LDS serves a wavefront's accesses in order
        load_w(Int<slot>{}, step + q + SLOTS * STEPS);
      }
#pragma unroll
      for (int n = 0; n < NG; ++n) {
        const bf16x8 f = __builtin_bit_cast(bf16x8, mine[place(16 * n + i, 4 * ((step + q) % STEPS) + g)]);
#pragma unroll
        for (int t = 0; t < TG; ++t)
          sum[n][t][(S * SB + q) % SUMS] += __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, __builtin_bit_cast(bf16x8, x[S][q][t]), zero, 0, 0, 0);
      }
      __builtin_amdgcn_wave_barrier();
    });
  };
  static_for<SLOTS>([&](auto slot) { load_w(slot, decltype(slot)::value * STEPS); });
  load_x(Int<0>{}, 0);
  for (int step = 0; step < steps; step += 2 * SB) {
    load_x(Int<1>{}, step + SB);
    batch(Int<0>{}, step);
    load_x(Int<0>{}, step + 2 * SB);
    batch(Int<1>{}, step + SB);
  }
  // element r of a sum is row 16t + i, column 16n + 4g + r; a wavefront's results at [row][4 columns] of its LDS
#pragma unroll
  for (int n = 0; n < NG; ++n)
#pragma unroll
    for (int t = 0; t < TG; ++t) {
#pragma unroll
      for (int half = SUMS / 2; half > 0; half /= 2)
#pragma unroll
        for (int k = 0; k < half; ++k) sum[n][t][k] += sum[n][t][k + half];
      mine[(16 * t + i) * 4 * NG + 4 * n + g] = __builtin_bit_cast(u32x4, sum[n][t][0]);
    }
  __syncthreads();
  const int row = row0 + tid / (4 * NG), col = 4 * (tid % (4 * NG));
  if (tid >= 64 * TG * NG || row >= row_end || col >= E) return;
  f32x4 v[NW];
#pragma unroll
  for (int wv = 0; wv < NW; ++wv) v[wv] = __builtin_bit_cast(f32x4, lds[wv * PLACES + tid]);
#pragma unroll
  for (int half = NW / 2; half > 0; half /= 2)
#pragma unroll
    for (int wv = 0; wv < half; ++wv) v[wv] += v[wv + half];
  *reinterpret_cast<f32x4*>(p.F + (size_t)row * E + col) = v[0];
}

// A CU alone reads 50 to 85 GB/s however many loads are on their way, so tiles for at most a quarter of the CUs (p.range) are
// halved: two wavefronts with 64 columns (UP: 32 of either matrix) each, the other two leave.  Once there are more halves than CUs
// they cost: they read 64 bytes of a row (UP) and more blocks read the same rows.  Experts of one row each, whole / halved tiles,
// us, weights in the Infinity Cache (and fetched from memory):
//   UP    d = 4096, f = 1536    48 tiles  28 / 22 (47 / 43)   96  29 / 24 (50 / 47)    144  (62 / 77)           192  (78 / 86)
//   UP    d = 7168, f = 2048    64 tiles  41 / 35 (70 / 67)   128  64 / 62 (99 / 99)   160  (113 / 131)         192  (125 / 131)
//   DOWN  d = 4096, f = 1536    64 tiles  12 / 10 (17 / 14)   128  13 / 14 (24 / 23)   160  (28 / 30)           256  (35 / 35)
//   DOWN  d = 7168, f = 2048    56 tiles  14 / 12 (21 / 17)   112  15 / 15 (28 / 26)   168  18 / 23 (36 / 40)   224  24 / 28 (32 / 36)
//   DOWN  d = 4096, f = 14336   64 tiles  89 / 66 (90 / 66)   128  100 / 83 (101 / 83) 160  (110 / 133)         256  (162 / 173)
// Halves win while every one of them has a CU to itself, so the line could lie at half the CUs; at a quarter they win throughout.
constexpr int NW_HALF = NW_TILES / 2;
template <int MODE> constexpr int TILE_COLS = (MODE == UP ? 16 : 32) * NW_TILES;
template <int MODE, bool MAY_STREAM>
__global__ __launch_bounds__(NW_TILES * WAVE) void small_rows(SArgs p) {
  __shared__ u32x4 lds[FEW_ROWS_PLACES<NW_TILES>];
  const int n_cols = (p.N + TILE_COLS<MODE> - 1) / TILE_COLS<MODE>;
  const RaggedTiles<ROWS> list(p.off, p.e_cnt, threadIdx.x & 63);
  if (list.total * n_cols > p.range) few_rows_tile<MODE == UP, NW_TILES, MAY_STREAM>(p, list, lds, blockIdx.x);
  else if (threadIdx.x < NW_HALF * WAVE) few_rows_tile<MODE == UP, NW_HALF, MAY_STREAM>(p, list, lds, blockIdx.x);
}

// grid = (row blocks of 16 * TG, column blocks, ranges of the contraction)
template <int TG>
__global__ __launch_bounds__(NW_ROUTER * WAVE) void router_dw_few(SArgs p) {
  __shared__ __align__(16) float red[NW_ROUTER * 16 * RPITCH];
  const int row0 = blockIdx.x * 16 * TG, first = blockIdx.z * p.range;
  p.F += (size_t)blockIdx.z * p.rows * p.N;
  router_tile<TG>(p, red, row0, min(p.rows, row0 + 16 * TG), blockIdx.y * COLS, first,
                  min(p.range, (p.K + KP - 1) / KP - first), threadIdx.x);
}

template <int MODE>
int launch_small(SArgs p, int cap, int prof_id, hipStream_t s) {
  p.range = device_cu_count() / 4;
  const long long bound = ((long long)cap / ROWS + (cap < p.e_cnt ? cap : p.e_cnt)) * ((p.N + TILE_COLS<MODE> - 1) / TILE_COLS<MODE>);
  const long long halves = 2 * (bound < p.range ? bound : p.range);
  const long long blocks = ((bound > halves ? bound : halves) + 7) / 8 * 8;
  if (blocks >= (1ll << 31)) return MOE_EUNSUPPORTED;
  ProfScope prof(prof_id, s);
  // Layers that fit the Infinity Cache as a whole never stream: without that half of the code up and down projection take 0.05 to 0.35 us
  // less (d = 4160, f = 704, one row 23.6 -> 23.3 us; 4224, 3968, 2 experts of 9 rows 45.0 -> 44.7; 2048, 768, 16 of 40 36.0 -> 35.8).
  const dim3 grid((unsigned)blocks), block(NW_TILES * WAVE);
  if (p.e_cnt > p.cached) hipLaunchKernelGGL((small_rows<MODE, true>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((small_rows<MODE, false>), grid, block, 0, s, p);
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}

}  // namespace

int launch_expert_fwd_small(const void* xp, int cap, int d, int f, int e_cnt, const int32_t* offsets, const void* w1,
                            const void* w3, const void* w2, void* h1, void* h3, void* a, void* o, hipStream_t s) {
  SArgs u = {};
  u.A = (const bf16_t*)xp; u.lda = d;
  u.B0 = (const bf16_t*)w1; u.B1 = (const bf16_t*)w3; u.ldb = f; u.b_es = (long)d * f;
  u.C0 = (bf16_t*)h1; u.C1 = (bf16_t*)h3; u.C2 = (bf16_t*)a; u.ldc = f;
  u.off = offsets; u.e_cnt = e_cnt; u.N = f; u.K = d; u.cached = cached_experts(d, f);
  int rc = launch_small<UP>(u, cap, MOE_K_UP, s);
  if (rc) return rc;
  SArgs w = {};
  w.A = (const bf16_t*)a; w.lda = f;
  w.B0 = (const bf16_t*)w2; w.ldb = d; w.b_es = (long)f * d;
  w.C0 = (bf16_t*)o; w.ldc = d;
  w.off = offsets; w.e_cnt = e_cnt; w.N = d; w.K = f; w.cached = u.cached;
  return launch_small<DOWN>(w, cap, MOE_K_DOWN, s);
}

// logits of 8 to 56 experts, E % 8 == 0
int launch_router_fwd_narrow(const void* x, const void* wr, int T, int d, int E, float* logits, hipStream_t s) {
  SArgs p = {};
  p.A = (const bf16_t*)x; p.lda = d;
  p.B0 = (const bf16_t*)wr;
  p.F = logits; p.rows = T; p.N = E; p.K = d;
  // As few rows per block as make at most one block per CU, up to 32 (16 for more than 16 experts: the sums take the registers).
  // Block per token / the 128 columns of router_tile / this, us, d = 4096:
  //   E = 8:   T = 1 5.7 / 12.1 / 5.8      T = 300 7.9 / 14.9 / 6.6     T = 4096 45 / 15.6 / 9.5     T = 16384 179 / 28.5 / 32.6
  //   E = 24:  T = 1 13.8 / 12.1 / 6.3     T = 300 20.0 / 14.8 / 7.1    T = 4096 178 / 15.3 / 9.8    T = 16384 695 / 28.2 / 33.1
  //   E = 56:  T = 1 30.0 / 12.0 / 12.5    T = 300 47.2 / 14.7 / 13.9   T = 4096 438 / 15.5 / 18.5   T = 16384 1723 / 28.4 / 64.9
  const int cus = device_cu_count(), most = E <= 16 ? 32 : 16;
  p.range = 1;
  while (p.range < most && (T + p.range - 1) / p.range > cus) p.range *= 2;
  const dim3 grid((T + p.range - 1) / p.range), block(NW_ROUTER * WAVE);
  ProfScope prof(MOE_K_ROUTER_FWD, s);
  if (p.range > 16) hipLaunchKernelGGL((narrow_router<2, 2, 1>), grid, block, 0, s, p);
  else if (E <= 16) hipLaunchKernelGGL((narrow_router<1, 2, 1>), grid, block, 0, s, p);
  else if (E <= 32) hipLaunchKernelGGL((narrow_router<1, 4, 2>), grid, block, 0, s, p);
  else if (E <= 48) hipLaunchKernelGGL((narrow_router<1, 8, 3>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((narrow_router<1, 8, 4>), grid, block, 0, s, p);
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}

// partials: room for max_ranges * T * E floats.  Returns the number of ranges through `ranges`: 1 = the logits are
// complete, else the partial sums in `partials` are still to be added up.
int launch_router_fwd_small(const void* x, const void* wr, int T, int d, int E, float* logits, float* partials, int max_ranges,
                            int* ranges, hipStream_t s) {
  SArgs p = {};
  p.A = (const bf16_t*)x; p.lda = d;
  p.B0 = (const bf16_t*)wr; p.ldb = E;
  p.rows = T; p.N = E; p.K = d;
  const int cus = device_cu_count(), pieces = d / KP;
  // A handful of blocks cannot draw the weights fast enough, so the contraction is cut, at two pieces or more per wavefront; the second
  // launch, which adds the ranges up, pays from three ranges on.  Where it is cut decides the bits, so it follows from blocks of 128
  // experts, by as few tokens as make at most one block per CU, whatever the blocks are.
  const int cut_cols = (E + COLS - 1) / COLS;
  const int cut_rows = (long long)(T + 15) / 16 * cut_cols <= cus ? 16 : ((long long)(T + 31) / 32 * cut_cols <= cus ? 32 : 64);
  int n = cus / (cut_cols * ((T + cut_rows - 1) / cut_rows));
  if (n > max_ranges) n = max_ranges;
  if (n > pieces / (2 * NW_ROUTER)) n = pieces / (2 * NW_ROUTER);
  if (n < 3) n = 1;
  p.range = (pieces + n - 1) / n;
  n = (pieces + p.range - 1) / p.range;
  p.F = n > 1 ? partials : logits;
  *ranges = n;
  // Tokens (16 tg) and experts (16 cl) of a block: the first of the list with at most one block per CU; a second round of blocks nearly
  // doubles the time.  32 by 64 comes before 16 by 128 where the experts fill blocks of 128: it asks for a third less per block; where
  // they do not, the half empty blocks of 128 ask for less.
  // 16 x 64 / 32 x 64 / 16 x 128 / 64 x 64 / 32 x 128 / 64 x 128, us:
  //   E = 128   T = 2047, d = 2880 11.0 / 13.4 / 15.5 / 17.4 / 17.6 / -    3000, 2048 13.1 / 11.0 / 11.6 / 14.1 / 13.2 / -
  //             T = 4096, d = 4096 23 / 17.1 / 19.8 / 22.4 / 22.2 / -      5000, 4096 - / 31 / - / 25.1 / 24.1 / 29.5
  //             T = 8000, d = 2880 - / 26 / - / 20.7 / 19.8 / 24.2         9001, 2880 - / 35 / - / 33 / 35 / 24.6
  //   E = 192   T = 1500, d = 4096 21.7 / 17.5 / 16.2 / 22.5 / 18.3 / -    3000, 2048 16.7 / 18.0 / 15.4 / 14.7 / 11.7 / -
  //   E = 72    T = 3500, d = 2048 13.8 / 11.3 / 9.8 / 14.7 / 11.4 / -     7000, 2048 - / 19.6 / - / 17.2 / 12.3 / 16.1
  //   E = 64    T = 8192, d = 4096 - / 19.9 / - / 26.1 / 20.3 / 26.5       16384, 2048 - / 23.0 / - / 19.1 / 23.6 / 19.8
  static constexpr struct { int tg, cl; bool full; } shapes[] = {{1, 4, false}, {2, 4, true}, {1, 8, false}, {2, 4, false}, {2, 8, false}, {4, 4, false}, {4, 8, false}};
  int tg = 0, cl = 0, cols = 0, row_blocks = 0;
  for (const auto& b : shapes) {
    if (b.full && E % COLS) continue;
    tg = b.tg, cl = b.cl;
    cols = (E + 16 * cl - 1) / (16 * cl), row_blocks = (T + 16 * tg - 1) / (16 * tg);
    if ((long long)row_blocks * cols * n <= cus) break;
  }
  const dim3 grid(row_blocks, cols, n), block(NW_ROUTER * WAVE);
  ProfScope prof(MOE_K_ROUTER_FWD, s);
  if (tg == 1 && cl == 4) hipLaunchKernelGGL((router_logits<1, 4>), grid, block, 0, s, p);
  else if (tg == 1) hipLaunchKernelGGL((router_logits<1, 8>), grid, block, 0, s, p);
  else if (tg == 2 && cl == 4) hipLaunchKernelGGL((router_logits<2, 4>), grid, block, 0, s, p);
  else if (tg == 2) hipLaunchKernelGGL((router_logits<2, 8>), grid, block, 0, s, p);
  else if (cl == 4) hipLaunchKernelGGL((router_logits<4, 4>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((router_logits<4, 8>), grid, block, 0, s, p);
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}

// dlogits as router_dl_operands lays them out: [pieces][planes * E][32].  Partial sums go to partials[ranges * planes][d][E]
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
  if (tg == 4) hipLaunchKernelGGL((router_dw_few<4>), grid, block, 0, s, p);
  else if (tg == 2) hipLaunchKernelGGL((router_dw_few<2>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((router_dw_few<1>), grid, block, 0, s, p);
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}
