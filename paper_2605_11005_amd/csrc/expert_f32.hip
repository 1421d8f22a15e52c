// fp32 expert FFNs on the matrix cores: every operand as three bf16 terms, whose products are summed in fp32.  The bf16 path is in
// expert_bf16.hip.
//
// One kernel template covers the six GEMM shapes of the layer, with the activation in the epilogue:
//   UP     h1|h3 = xp [W1|W3]   ragged M, weights n-contiguous, two outputs of one tile -> a = silu(h1) h3
//   DOWN   o     = a W2         ragged M, weights n-contiguous
//   DA     dA    = d_o W2^T     ragged M, weights k-contiguous, SwiGLU backward -> dH1, dH3 (and a if it was not kept)
//   DX     dxp   = dH1 W1^T + dH3 W3^T   ragged M, K in two segments
//   WG     dW2   = a^T d_o      ragged K (the expert's rows)
//   WGD    dW1|dW3 = xp^T [dH1|dH3]      ragged K, two outputs of one tile
//
// The fp32 matrix instruction does 256 FLOP per cycle and CU, the bf16 one sixteen times that, so six bf16 products take 3/8 of
// the time.  Three terms hold all 24 bits of a number.  The three products of terms that are left out are up to 2^-24.0 of a product of
// operands (x = y = 1.0039), 2^-27.4 in the root mean square; two more of them would make that 2^-33 and training steps 5 to 10 %
// longer.  Sixteen products are added per rounding instead of two: against 64 bits the outputs are off by half of what the fp32
// instruction gave (1.3e-7 for 2.9e-7 for h1 at d = 520, 3.3e-7 for 6.7e-7 for the worst gradient; twelve shapes, none of them further
// off).
//
// What bounds it now, all near 1000 cycles per k-tile of a dual tile: the operands' way to the CU (24 KB), LDS (36 KB written,
// 114 KB read), splitting the operands (about 175 vector instructions) and the matrix pipe (768).  Only other blocks' waves fill
// the gaps, hence a small tile, 64x64 by four wavefronts of 32x32 each, one LDS buffer and registers for three (dual) or four
// blocks per CU (two buffers where two blocks per CU or fewer are all there are: launch()), and two k-tiles of 32 on their way in
// registers while a third is multiplied.  3000 rows over 16 experts, d = 520, f = 776, forward + backward on one card: 107 + 215 us
// with the fp32 instruction, 90 + 175 as it is.  Tried, on another card and before the operands were scaled, against 79 + 160:
// two LDS buffers and two blocks per CU 87 + 176; splitting between the matrix instructions of one wavefront, which takes more
// registers, 104 + 181; tiles of 128x64 95 + 199 (better only for a thousand rows and more per expert: 145 for 176 at 3000, d = f =
// 1024).
#include "common.h"
#include "kernels.h"

namespace {

constexpr int TM = 64, TN = 64, TK = 32, NT = 256;
typedef float f32x16 __attribute__((ext_vector_type(16)));

enum { UP, DOWN, DA, DX, WG, WGD };

// An fp32 matrix instruction contracts two values of k, one per half of the wavefront.  Which two is free as long as both
// operands agree: in groups of eight steps the lower half takes k = 0..7 and the upper one k = 8..15 of a group of 16, so
// that a lane of a k-contiguous operand reads consecutive words (16 bytes serve four steps).
// Pitches: [64 rows][k] at 36 words -- 16 lanes reading 16 bytes each hit 64 banks; [k][64 columns] at 68 -- rows eight
// apart, read together by the two halves, are 32 banks apart.
constexpr int PITCH_KC = 36, PITCH_MN = 68;
constexpr int HALF = TK / 4;      // steps whose fragments are held at a time: half of a k-tile

// Loads go through a buffer descriptor that begins at the k-tile and ends with the operand's last valid element: a lane's offset in a
// tile never changes, so that a k-tile's addresses are a few 32-bit scalar instructions instead of two 64-bit multiplications per
// load on the vector unit, which the splitting keeps busy.  Training steps (T, d, f, experts, k), us: 1500, 520, 776, 16, 2 256 -> 247; 2579, 592,
// 880, 12, 2 470 -> 452; 1128, 452, 880, 32, 4 380 -> 366; 265, 712, 144, 4, 1 115 -> 113; 256, 128, 256, 8, 2 84.4 -> 83.6.  (With 64-bit
// scalar bounds, whose comparisons are vector instructions, the small ones took 1 to 2 % longer than before.)
// Past the end of the contraction a load of an operand whose columns are contiguous returns zeros; one whose k is contiguous returns what
// follows in memory up to the tile's last valid element, the next rows' beginnings, also in the k-tiles past the last one.  So mask() and
// keep() make that part zero on the way to LDS (the k-tiles past the last one are not multiplied); rows and columns past the end repeat the last
// ones (their products are never stored).  32 bits hold 64 rows: the entry points take d and f up to 4.2 million in fp32.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_descriptor(const float* base, int words) {
  uint64_t b = (uint64_t)base;
  int bytes = 4 * max(0, words);
  asm("" : "+s"(b), "+s"(bytes));         // both are wave-uniform: keep them in scalar registers
  return __builtin_amdgcn_make_buffer_rsrc((void*)b, 0, bytes, 0x00027000);
}
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 tile_load(__amdgpu_buffer_rsrc_t d, int voff) {
  return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(d, voff, 0, 0));
}
// a pointer that is the same in all lanes, in scalar registers
__device__ __forceinline__ const float* uniform(const float* q) {
  const uint64_t u = (uint64_t)q;
  return (const float*)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(u >> 32)) << 32) |
                        (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u));
}

__device__ __forceinline__ float4 keep(float4 v, bool in) {
  return make_float4(in ? v.x : 0.f, in ? v.y : 0.f, in ? v.z : 0.f, in ? v.w : 0.f);
}

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
// Weight gradients of up to this many rows are summed by the fp32 instruction.  Largest error of 400000 outputs in units of 2^-24 sum
// |products| (rms), fp32 instruction / terms, Gaussian operands: one row 1.00 / 1.54 (0.425 / 0.435; a product is rounded
// correctly, the terms leave out up to 2^-24 of it), two 1.89 / 2.70 (0.516 / 0.369), three 2.45 / 2.37 (0.490 / 0.328), eight 2.92
// / 1.92 (0.412 / 0.240), 64 3.07 / 1.83 (0.345 / 0.160).
constexpr int EXACT_ROWS = 2;
// SCALE x = h + m + l in bf16, each the rounded rest of the ones before it.  The scale brings the last bit of fp32's smallest
// number, 2^-149, among bf16's normal numbers, so that the three hold every x up to 2^96 exactly; products, and with them sums,
// are SCALE^2 times what they stand for.  Beyond 2^96 the first term is infinite and the second NaN, and so are the sums that it enters.
// (Without the scale numbers below 2^-109 lost bits and those below 2^-134 everything; it takes 0 to 2 % of a training step: 293 ->
// 300 us at T = 600, d = f = 1000, 8 experts, k = 2.)
constexpr float SCALE = 0x1p32f, UNSCALE = 0x1p-64f;
struct Split4 {
  uint2 h, m, l;
  __device__ __forceinline__ explicit Split4(float4 v) {
    v.x *= SCALE; v.y *= SCALE; v.z *= SCALE; v.w *= SCALE;
    h = make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
    v.x -= bf16lo(h.x); v.y -= bf16hi(h.x); v.z -= bf16lo(h.y); v.w -= bf16hi(h.y);
    m = make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
    v.x -= bf16lo(m.x); v.y -= bf16hi(m.x); v.z -= bf16lo(m.y); v.w -= bf16hi(m.y);
    l = make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
  }
};
// The three terms of an operand's k-tile lie one behind the other, 4 KB each.
constexpr int PLANE_BYTES = 64 * TK * 2;
__device__ __forceinline__ void store_planes(char* s, int off, float4 v) {
  const Split4 t(v);
  *reinterpret_cast<uint2*>(s + off) = t.h;
  *reinterpret_cast<uint2*>(s + PLANE_BYTES + off) = t.m;
  *reinterpret_cast<uint2*>(s + 2 * PLANE_BYTES + off) = t.l;
}

// k-contiguous operand: rows [0, rows) of a matrix with leading dimension ld; k in [0, K), K % 4 == 0
struct OperKC {
  static constexpr int WORDS = 64 * PITCH_KC;
  // plane: [64 rows][4 chunks of 8 k], chunk' = chunk ^ ((row>>2)&3): 16 lanes reading 16 bytes each hit 64 banks
  __device__ __forceinline__ void store_split(const float4* v, char* s, int tid) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int idx = tid + NT * i, r = idx >> 3, q = idx & 7;
      store_planes(s, r * 64 + (((q >> 1) ^ ((r >> 2) & 3)) << 4) + (q & 1) * 8, v[i]);
    }
  }
  __device__ __forceinline__ void mask(float4* v, int k0, int tid) const {       // zeros past the end of the contraction
#pragma unroll
    for (int i = 0; i < 2; ++i) v[i] = keep(v[i], k0 + 4 * ((tid + NT * i) & 7) < K);
  }
  // pos0: first of the wavefront's 32 rows or columns; k-step t of 16
  static __device__ __forceinline__ bf16x8 split_frag(const char* plane, int pos0, int lane, int t) {
    const int r = pos0 + (lane & 31);
    return *reinterpret_cast<const bf16x8*>(plane + r * 64 + (((2 * t + (lane >> 5)) ^ ((r >> 2) & 3)) << 4));
  }
  const float* base;
  long ld;
  int rows, K, voff[2];
  int left;                // of the contraction
  __device__ __forceinline__ void setup(const float* base_, long ld_, int rows_, int K_, int tid) {
    base = uniform(base_);
    ld = ld_;
    K = K_;
    rows = __builtin_amdgcn_readfirstlane(min(rows_, TM));
    left = K;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int idx = tid + NT * i;
      voff[i] = 4 * (min(idx >> 3, rows - 1) * (int)ld + 4 * (idx & 7));
    }
  }
  __device__ __forceinline__ void load(float4* v) {      // k-tiles in order
    const __amdgpu_buffer_rsrc_t d = tile_descriptor(base, (rows - 1) * (int)ld + left);
    base += TK;
    left -= TK;
#pragma unroll
    for (int i = 0; i < 2; ++i) v[i] = tile_load(d, voff[i]);
  }
  __device__ __forceinline__ void store(const float4* v, float* s, int k0, int tid) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int idx = tid + NT * i;
      *reinterpret_cast<float4*>(s + (idx >> 3) * PITCH_KC + 4 * (idx & 7)) = keep(v[i], k0 + 4 * (idx & 7) < K);
    }
  }
  // fragments of steps [HALF * h, HALF * (h + 1)); pos: row or column of this lane in the tile, up: upper half of the wavefront
  static __device__ __forceinline__ void frags(float* f, const float* s, int pos, int up, int h) {
#pragma unroll
    for (int q = 0; q < HALF / 4; ++q) {
      const float4 w = *reinterpret_cast<const float4*>(s + pos * PITCH_KC + 16 * h + 8 * up + 4 * q);
      f[4 * q] = w.x; f[4 * q + 1] = w.y; f[4 * q + 2] = w.z; f[4 * q + 3] = w.w;
    }
  }
};

// operand whose rows or columns are contiguous: base points at k = 0, tile column 0; cols columns are valid (cols % 4 == 0)
struct OperMN {
  static constexpr int WORDS = TK * PITCH_MN;
  // plane: [32 k][8 chunks of 8 columns], chunk' = chunk ^ (4*((k>>1)&1)), read by the transposing LDS reads
  __device__ __forceinline__ void store_split(const float4* v, char* s, int tid) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int idx = tid + NT * i, k = idx >> 4, c = idx & 15;
      store_planes(s, k * 128 + (((c >> 1) ^ (4 * ((k >> 1) & 1))) << 4) + (c & 1) * 8, v[i]);
    }
  }
  __device__ __forceinline__ void mask(float4* v, int k0, int tid) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) v[i] = keep(v[i], k0 + ((tid + NT * i) >> 4) < K);
  }
  static __device__ __forceinline__ bf16x8 split_frag(const char* plane, int pos0, int lane, int t) {
    const int i = lane & 15, g = lane >> 4;
    const int k = 8 * (g >> 1) + (i >> 2), n = pos0 + 16 * (g & 1) + 4 * (i & 3);
    const char* p = plane + t * 2048 + k * 128 + (((n >> 3) ^ (4 * ((k >> 1) & 1))) << 4) + ((n & 4) << 1);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p + 512));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
  const float* base;
  long ld;
  int cols, K, voff[2];
  int left;                // of the contraction
  __device__ __forceinline__ void setup(const float* base_, long ld_, int cols_, int K_, int tid) {
    base = uniform(base_);
    ld = ld_;
    cols = cols_;
    K = __builtin_amdgcn_readfirstlane(K_);
    left = K;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int idx = tid + NT * i;
      voff[i] = 4 * ((idx >> 4) * (int)ld + min(4 * (idx & 15), cols - 4));
    }
  }
  __device__ __forceinline__ void load(float4* v) {      // k-tiles in order
    const __amdgpu_buffer_rsrc_t d = tile_descriptor(base, (min(left, TK) - 1) * (int)ld + cols);
    base += TK * ld;
    left -= TK;
#pragma unroll
    for (int i = 0; i < 2; ++i) v[i] = tile_load(d, voff[i]);
  }
  __device__ __forceinline__ void store(const float4* v, float* s, int k0, int tid) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int idx = tid + NT * i;
      *reinterpret_cast<float4*>(s + (idx >> 4) * PITCH_MN + 4 * (idx & 15)) = keep(v[i], k0 + (idx >> 4) < K);
    }
  }
  static __device__ __forceinline__ void frags(float* f, const float* s, int pos, int up, int h) {
#pragma unroll
    for (int q = 0; q < HALF; ++q) f[q] = s[(16 * h + 8 * up + q) * PITCH_MN + pos];
  }
};

template <bool C, typename A, typename B> struct Pick { typedef A type; };
template <typename A, typename B> struct Pick<false, A, B> { typedef B type; };

struct Args {
  const float* A[2];        // [1]: second K segment of DX
  const float* B[2];        // [1]: second output of a dual tile / second K segment of DX
  long lda, ldb, b_es;      // b_es: expert stride of B (0: row-indexed)
  float* C[3];
  const float* H[2];        // DA: h1, h3
  long ldc, c_es;           // c_es: expert stride of C (0: row-indexed)
  int M, N, K;              // M: WG / WGD, K: ragged-M shapes (per segment)
  const int32_t* off;
  int e_cnt, beta;
};

// LDS of one k-tile: the three bf16 terms of each operand, or the operands themselves
template <int MODE> struct Traits {
  static constexpr bool RAGGED_K = MODE == WG || MODE == WGD;
  static constexpr bool DUAL = MODE == UP || MODE == WGD;
  static constexpr int NB = DUAL ? 2 : 1;
  typedef typename Pick<RAGGED_K, OperMN, OperKC>::type OperA;
  typedef typename Pick<MODE == DA || MODE == DX, OperKC, OperMN>::type OperB;
  static constexpr int SPLIT_BYTES = (1 + NB) * 3 * PLANE_BYTES, PLAIN_BYTES = (OperA::WORDS + NB * OperB::WORDS) * 4;
  static constexpr int BUFFER = SPLIT_BYTES > PLAIN_BYTES ? SPLIT_BYTES : PLAIN_BYTES;
  static constexpr int BLOCKS = DUAL ? 3 : 4;      // per CU, with one LDS buffer
};

// Block `block` of one GEMM, a 1-D list of tiles: RaggedTiles' for the ragged-M shapes, the same with a fixed number of row tiles
// per expert for the ragged-K ones.
// BUFS: LDS buffers, two in launches of few blocks (use_two()).
template <int MODE, int BUFS>
__device__ __forceinline__ void gemm_tile(const Args& p, int block, char* lds) {
  using TR = Traits<MODE>;
  constexpr bool RAGGED_K = TR::RAGGED_K, DUAL = TR::DUAL;
  constexpr int NB = TR::NB, BUFFER = TR::BUFFER;
  typedef typename TR::OperA OperA;
  typedef typename TR::OperB OperB;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_tiles = (p.N + TN - 1) / TN, m_tiles = (p.M + TM - 1) / TM;
  int e, mt, nt, row0, row_end, K;                       // output rows [row0, row_end)
  if (RAGGED_K) {
    const int total = p.e_cnt * m_tiles * n_tiles, share = (total + 7) / 8;
    const int tile = (block % 8) * share + block / 8;
    if (block / 8 >= share || tile >= total) return;
    e = tile / (m_tiles * n_tiles);
    mt = (tile - e * m_tiles * n_tiles) / n_tiles;
    nt = tile % n_tiles;
    row0 = mt * TM;
    row_end = p.M;
    K = p.off[e + 1] - p.off[e];
  } else {
    if (!RaggedTiles<TM>(p.off, p.e_cnt, lane).tile(n_tiles, block, e, mt, nt)) return;
    row0 = p.off[e] + mt * TM;
    row_end = p.off[e + 1];
    K = p.K;
  }
  const int col0 = nt * TN;

  OperA a;
  OperB b[NB];
  auto setup = [&](int seg) {
    if constexpr (RAGGED_K) {
      const size_t first = p.off[e];
      a.setup(p.A[0] + first * p.lda + row0, p.lda, p.M - row0, K, tid);
#pragma unroll
      for (int i = 0; i < NB; ++i) b[i].setup(p.B[i] + first * p.ldb + col0, p.ldb, p.N - col0, K, tid);
    } else {
      a.setup(p.A[seg] + (size_t)row0 * p.lda, p.lda, row_end - row0, K, tid);
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const float* w = p.B[DUAL ? i : seg] + (size_t)e * p.b_es;
        if constexpr (MODE == DA || MODE == DX) b[i].setup(w + (size_t)col0 * p.ldb, p.ldb, p.N - col0, K, tid);
        else b[i].setup(w + col0, p.ldb, p.N - col0, K, tid);
      }
    }
  };
  f32x16 acc[NB][2];         // two sums per output, added at the end

  const int wm = wave >> 1, wn = wave & 1;
  const int a_pos = wm * 32 + (lane & 31), b_pos = wn * 32 + (lane & 31), up = lane >> 5;
  const int nk1 = (K + TK - 1) / TK, nk = MODE == DX ? 2 * nk1 : nk1;
  const bool live = wm * 32 < row_end - row0;    // a wavefront without valid rows only moves data
  // SPLIT: on the bf16 matrix instruction, the operands as three terms each.  Six products: h h in one sum, h m, m h, h l, l h and
  // m m in the other; the three left out are below 2^-24 of the whole.  Else: on the fp32 matrix instruction, even and odd steps
  // in the two sums.
  auto sums = [&](auto split_tag) {
    constexpr bool SPLIT = decltype(split_tag)::value != 0;
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][0][r] = acc[i][1][r] = 0.f;
    // two k-tiles travel in registers while one is multiplied
    float4 va[2][2], vb[2][NB][2];
    const auto first_k = [&](int kt) { return (MODE == DX && kt >= nk1 ? kt - nk1 : kt) * TK; };
    auto fetch = [&](int kt, auto set) {
      constexpr int S = decltype(set)::value;
      if (MODE == DX && kt == nk1) setup(1);       // the second half of the k-tiles is the second segment
      a.load(va[S]);                               // (past the last one: never multiplied)
#pragma unroll
      for (int i = 0; i < NB; ++i) b[i].load(vb[S][i]);
    };
    auto publish = [&](int kt, auto set) {
      constexpr int S = decltype(set)::value;
      char* const to = lds + (BUFS == 2 ? S * BUFFER : 0);
      if constexpr (SPLIT) {
        if (first_k(kt) + TK > K) {
          a.mask(va[S], first_k(kt), tid);
#pragma unroll
          for (int i = 0; i < NB; ++i) b[i].mask(vb[S][i], first_k(kt), tid);
        }
        a.store_split(va[S], to, tid);
#pragma unroll
        for (int i = 0; i < NB; ++i) b[i].store_split(vb[S][i], to + (1 + i) * 3 * PLANE_BYTES, tid);
      } else {
        float* buf = reinterpret_cast<float*>(to);
        a.store(va[S], buf, first_k(kt), tid);
#pragma unroll
        for (int i = 0; i < NB; ++i) b[i].store(vb[S][i], buf + OperA::WORDS + i * OperB::WORDS, first_k(kt), tid);
      }
    };
    auto multiply = [&](auto set) {
      const char* const from = lds + (BUFS == 2 ? decltype(set)::value * BUFFER : 0);
      if (!live) return;
      if constexpr (SPLIT) {
#pragma unroll
        for (int t = 0; t < TK / 16; ++t) {
          bf16x8 fa[3], fb[NB][3];
#pragma unroll
          for (int q = 0; q < 3; ++q) {
            fa[q] = OperA::split_frag(from + q * PLANE_BYTES, wm * 32, lane, t);
#pragma unroll
            for (int i = 0; i < NB; ++i) fb[i][q] = OperB::split_frag(from + ((1 + i) * 3 + q) * PLANE_BYTES, wn * 32, lane, t);
          }
          const auto mfma = [&](int i, int c, int x, int y) { acc[i][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[x], fb[i][y], acc[i][c], 0, 0, 0); };
          // consecutive instructions add to different sums
#pragma unroll
          for (int i = 0; i < NB; ++i) { mfma(i, 1, 1, 1); mfma(i, 0, 0, 0); }
#pragma unroll
          for (int i = 0; i < NB; ++i) mfma(i, 1, 0, 2);
#pragma unroll
          for (int i = 0; i < NB; ++i) mfma(i, 1, 2, 0);
#pragma unroll
          for (int i = 0; i < NB; ++i) mfma(i, 1, 0, 1);
#pragma unroll
          for (int i = 0; i < NB; ++i) mfma(i, 1, 1, 0);
        }
      } else {
        const float* buf = reinterpret_cast<const float*>(from);
        float fa[2][HALF], fb[2][NB][HALF];
        auto read = [&](int h) {
          OperA::frags(fa[h], buf, a_pos, up, h);
#pragma unroll
          for (int i = 0; i < NB; ++i) OperB::frags(fb[h][i], buf + OperA::WORDS + i * OperB::WORDS, b_pos, up, h);
        };
        read(0);
        read(1);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int q = 0; q < HALF; ++q)
#pragma unroll
            for (int i = 0; i < NB; ++i)
              acc[i][q & 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[h][q], fb[h][i][q], acc[i][q & 1], 0, 0, 0);
      }
    };
    setup(0);
    if (nk > 0) {
      fetch(0, Int<0>{});
      fetch(1, Int<1>{});
    }
    if constexpr (BUFS == 2) {
      // one buffer is written while the other is multiplied; the barrier ends both
      if (nk > 0) publish(0, Int<0>{});
      __syncthreads();
      for (int kt = 0; kt + 1 < nk; kt += 2) {
        fetch(kt + 2, Int<0>{});
        multiply(Int<0>{});
        publish(kt + 1, Int<1>{});
        __syncthreads();
        fetch(kt + 3, Int<1>{});
        multiply(Int<1>{});
        publish(kt + 2, Int<0>{});
        __syncthreads();
      }
      if (nk & 1) multiply(Int<0>{});
    } else {
      // published, multiplied, and the buffer is free again
      auto step = [&](int kt, auto set) {
        publish(kt, set);
        __syncthreads();
        fetch(kt + 2, set);
        multiply(set);
        __syncthreads();
      };
      for (int kt = 0; kt < nk; kt += 2) {
        step(kt, Int<0>{});
        if (kt + 1 < nk) step(kt + 1, Int<1>{});
      }
    }
  };
  // The outputs of the accumulator elements in todo (bit r: element r).  Element 4g + i of a lane is row 8g + 4*(lane/32) + i,
  // column lane%32 of its wavefront's block.
  auto finish = [&](uint32_t todo, float scale) {
    const int col = col0 + wn * 32 + (lane & 31);
    if (col >= p.N) return;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      float h1[4], h3[4];
      const int r0 = row0 + wm * 32 + 8 * g + 4 * (lane >> 5);
      if (MODE == DA) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const size_t idx = (size_t)(r0 + i < row_end ? r0 + i : row_end - 1) * p.ldc + col;
          h1[i] = p.H[0][idx];
          h3[i] = p.H[1][idx];
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (r0 + i >= row_end || !(todo >> (4 * g + i) & 1)) continue;
        const size_t idx = (size_t)e * p.c_es + (size_t)(r0 + i) * p.ldc + col;
        const float x = (acc[0][0][4 * g + i] + acc[0][1][4 * g + i]) * scale;
        const float x3 = (acc[NB - 1][0][4 * g + i] + acc[NB - 1][1][4 * g + i]) * scale;      // second output of a dual tile
        if (MODE == UP) {
          if (p.C[0]) { p.C[0][idx] = x; p.C[1][idx] = x3; }
          p.C[2][idx] = (x / (1.0f + expf(-x))) * x3;
        } else if (MODE == DA) {
          const float z = h1[i], sg = 1.0f / (1.0f + expf(-z)), sl = z * sg;
          if (p.C[0]) p.C[0][idx] = sl * h3[i];      // not stored when the forward's copy is at hand
          p.C[1][idx] = x * h3[i] * (sg * (1.0f + z * (1.0f - sg)));
          p.C[2][idx] = x * sl;
        } else {
          p.C[0][idx] = p.beta ? p.C[0][idx] + x : x;
          if (DUAL) p.C[1][idx] = p.beta ? p.C[1][idx] + x3 : x3;
        }
      }
    }
  };
  // Outputs with an infinity, a NaN, a number beyond 2^96 or a sum beyond 2^64 in them have sums that are no numbers.  Those, and no
  // others of their tile, come from the operands as they are: what a row or column holds does not show in its neighbours' bits.
  // (With one in every tile the six GEMMs of 3000 rows, d = 520, f = 776, take 178 + 360 us for 90 + 175.)
  // So do all weight gradients of an expert with one or two rows, which the terms would not round as well (EXACT_ROWS).
  const bool exact = RAGGED_K && K <= EXACT_ROWS;
  uint32_t lost = exact ? 0xFFFFu : 0u;
  if (!exact) {
    sums(Int<1>{});
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      bool whole = true;
#pragma unroll
      for (int i = 0; i < NB; ++i) whole &= fabsf(acc[i][0][r] + acc[i][1][r]) <= 3.402823466e38f;
      lost |= whole ? 0u : 1u << r;
    }
  }
  const bool again = __syncthreads_or(lost != 0);
  finish(~lost, UNSCALE);
  if (again) {
    sums(Int<0>{});
    finish(lost, 1.f);
  }
}

template <int MODE, int BUFS>
__global__ __launch_bounds__(NT, BUFS == 2 ? 2 : Traits<MODE>::BLOCKS) void gemm_f32(Args p) {
  __shared__ __align__(16) char lds[BUFS * Traits<MODE>::BUFFER];
  gemm_tile<MODE, BUFS>(p, blockIdx.x, lds);
}

// Two GEMMs that do not depend on each other in one launch, one of them in blocks [0, first), the other behind it.
template <int M1, int M2, int BUFS>
__global__ __launch_bounds__(NT, BUFS == 2 ? 2 : (Traits<M1>::BLOCKS < Traits<M2>::BLOCKS ? Traits<M1>::BLOCKS : Traits<M2>::BLOCKS))
void gemm_f32_pair(Args p1, Args p2, int first, int m2_first) {
  __shared__ __align__(16) char lds[BUFS * (Traits<M1>::BUFFER > Traits<M2>::BUFFER ? Traits<M1>::BUFFER : Traits<M2>::BUFFER)];
  const bool in_first = (int)blockIdx.x < first;
  const int block = in_first ? blockIdx.x : blockIdx.x - first;
  if (in_first != (m2_first != 0)) gemm_tile<M1, BUFS>(p1, block, lds);
  else gemm_tile<M2, BUFS>(p2, block, lds);
}

// Two LDS buffers while at most two blocks share a CU: nothing else fills the gaps there.  The sums and their order are the same.
// Training step before the operands were scaled, us, one buffer / two up to 256 blocks / two up to 512 (T, d, f, experts, k): 100,
// 256, 512, 8, 2 107 / 99 / 97; 256, 1024, 512, 8, 1 170 / 152 / 151; 300, 400, 600, 16, 2 146 / 137 / 131; 600, 1000, 1000, 8, 2 300 /
// 300 / 293.  At 1500, 520, 776, 16, 2 (800 blocks and more) two buffers for all take 87 + 176 for 79 + 160 in the six GEMMs.
inline bool use_two(long long blocks) { return blocks <= 2 * device_cu_count(); }

// m_tiles: bound on the row tiles of all experts
inline long long tile_blocks(const Args& p, long long m_tiles) { return (m_tiles * ((p.N + TN - 1) / TN) + 7) / 8 * 8; }

template <int MODE>
int launch(const Args& p, long long m_tiles, hipStream_t s) {
  const long long blocks = tile_blocks(p, m_tiles);
  if (blocks >= (1ll << 31)) return MOE_EUNSUPPORTED;
  const auto kernel = use_two(blocks) ? gemm_f32<MODE, 2> : gemm_f32<MODE, 1>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(NT), 0, s, p);
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}

template <int M1, int M2>
int launch_pair(const Args& p1, long long m_tiles1, const Args& p2, long long m_tiles2, bool m2_first, hipStream_t s) {
  const long long n1 = tile_blocks(p1, m_tiles1), n2 = tile_blocks(p2, m_tiles2), blocks = n1 + n2;
  if (blocks >= (1ll << 31)) {
    const int rc = launch<M1>(p1, m_tiles1, s);
    return rc ? rc : launch<M2>(p2, m_tiles2, s);
  }
  const auto kernel = use_two(blocks) ? gemm_f32_pair<M1, M2, 2> : gemm_f32_pair<M1, M2, 1>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(NT), 0, s, p1, p2, (int)(m2_first ? n2 : n1), m2_first ? 1 : 0);
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}

}  // namespace

int launch_expert_fwd_f32(const float* xp, int cap, int d, int f, int e_cnt, const int32_t* offsets,
                          const float* w1, const float* w3, const float* w2, float* h1, float* h3,
                          float* o, float* a, hipStream_t s) {
  if (cap == 0 || e_cnt == 0) return MOE_OK;
  const long long mtb = ((long long)cap + TM - 1) / TM + e_cnt;
  Args u = {};
  u.A[0] = xp; u.lda = d; u.B[0] = w1; u.B[1] = w3; u.ldb = f; u.b_es = (long)d * f;
  u.C[0] = h1; u.C[1] = h3; u.C[2] = a; u.ldc = f; u.N = f; u.K = d; u.off = offsets; u.e_cnt = e_cnt;
  int rc = launch<UP>(u, mtb, s);
  if (rc) return rc;
  Args w = {};
  w.A[0] = a; w.lda = f; w.B[0] = w2; w.ldb = d; w.b_es = (long)f * d;
  w.C[0] = o; w.ldc = d; w.N = d; w.K = f; w.off = offsets; w.e_cnt = e_cnt;
  return launch<DOWN>(w, mtb, s);
}

int launch_expert_bwd_f32(const float* xp, const float* h1, const float* h3, const float* a_in, const float* d_o, int cap,
                          int d, int f, int e_cnt, const int32_t* offsets, const float* w1,
                          const float* w3, const float* w2, float* dxp, float* dw1, float* dw3,
                          float* dw2, int accumulate, float* ws, hipStream_t s) {
  if (e_cnt == 0) return MOE_OK;
  float* a = ws;
  float* dh1 = ws + (size_t)cap * f;
  float* dh3 = ws + 2 * (size_t)cap * f;
  int rc;
  const long long mtb = ((long long)cap + TM - 1) / TM + e_cnt;
  Args g = {};
  g.A[0] = d_o; g.lda = d; g.B[0] = w2; g.ldb = d; g.b_es = (long)f * d;
  g.C[0] = a_in ? nullptr : a; g.C[1] = dh1; g.C[2] = dh3; g.H[0] = h1; g.H[1] = h3; g.ldc = f;
  g.N = f; g.K = d; g.off = offsets; g.e_cnt = e_cnt;
  Args x = {};
  x.A[0] = dh1; x.A[1] = dh3; x.lda = f; x.B[0] = w1; x.B[1] = w3; x.ldb = f; x.b_es = (long)d * f;
  x.C[0] = dxp; x.ldc = d; x.N = d; x.K = f; x.off = offsets; x.e_cnt = e_cnt;
  // dW2 takes the activation the forward kept, if the caller passed it, else the one that dA recomputes
  Args w = {};
  w.A[0] = a_in ? a_in : a; w.lda = f; w.B[0] = d_o; w.ldb = d;
  w.C[0] = dw2; w.ldc = d; w.c_es = (long)f * d; w.M = f; w.N = d; w.off = offsets; w.e_cnt = e_cnt; w.beta = accumulate;
  Args v = {};
  v.A[0] = xp; v.lda = d; v.B[0] = dh1; v.B[1] = dh3; v.ldb = f;
  v.C[0] = dw1; v.C[1] = dw3; v.ldc = f; v.c_es = (long)d * f; v.M = d; v.N = f; v.off = offsets; v.e_cnt = e_cnt; v.beta = accumulate;
  // With the forward's activation dA and dW2 do not depend on each other, dX and dW1|dW3 never do: they share launches, the second
  // one's blocks filling the CUs that the first one's leave.  dX has one round of blocks or less even where the gradients have
  // several (T = 1500, d = 520, f = 776, 16 experts, k = 2: 568 and 1872 blocks for 768 places), and a small GEMM is little more
  // than its launch, its first loads and its last stores.  Training steps, us, four launches / two (T, d, f, experts, k): 1500, 520,
  // 776, 16, 2 292 / 265; 309, 736, 792, 32, 2 399 / 361; 261, 120, 992, 12, 4 176 / 157; 126, 336, 808, 8, 4 153 / 131.
  // The longer tiles come first: a gradient's contract the rows of an expert, of which the capacity tells the average, dA's d and dX's f
  // twice into one output.  Backward, us, four launches / dA and dX first / gradients first (d, f, experts, rows of each): 1024, 1024, 1, 3000
  // 340 / 350 / 297; 1024, 1024, 2, 3000 572 / 598 / 547; 1024, 1024, 1, 1000 143 / 110 / 119; 512, 512, 8, 2000 406 / 398 / 383; 512, 512, 8,
  // 500 127 / 113 / 113; 1024, 1024, 8, 400 344 / 325 / 346; 520, 776, 16, 190 176 / 152 / 160; 512, 256, 32, 3000 / (1 + e) 336 / 346 / 326.
  const auto gradients_first = [&](int contraction) { return 5ll * cap > 6ll * e_cnt * contraction; };
  const long long wt = (long long)e_cnt * ((f + TM - 1) / TM), vt = (long long)e_cnt * ((d + TM - 1) / TM);
  if (cap == 0) {
    if ((rc = launch<WG>(w, wt, s))) return rc;
    return launch<WGD>(v, vt, s);
  }
  if (a_in) {
    if ((rc = launch_pair<DA, WG>(g, mtb, w, wt, gradients_first(d), s))) return rc;
  } else {
    if ((rc = launch<DA>(g, mtb, s))) return rc;
    if ((rc = launch<WG>(w, wt, s))) return rc;
  }
  return launch_pair<DX, WGD>(x, mtb, v, vt, gradients_first(f), s);
}
