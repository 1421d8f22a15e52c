// The trainable gate around the expert layer: router GEMM, fused backward of combine (d_o and the
// gradient of the gate weights in one pass over dy), gradient through the gate weights to the
// logits, and the router's backward GEMMs.
//
// bf16 with d % 64 == 0 runs on the matrix cores:
//   logits           E % 8 == 0: expert_small.hip; many tokens of E % 64 == 0 the grouped-GEMM kernel of expert_bf16.hip (launch_router_fwd)
//   weight gradient  32, 64, 96, 128, 160, 192 and 256 experts: router_dw.hip where router_dw_ranges says so; else up to 128 experts (42
//                    where the dlogits stay fp32) expert_small.hip, other E % 64 == 0 the grouped GEMM (launch_router_bwd)
//   input gradient   32, 96, 160 and E % 64 == 0 experts up to 256: router_dx.hip; E % 64 == 0 beyond: the grouped GEMM
// Every other shape (fp32, odd expert counts) takes the plain kernels below, which accept any size.  The contraction over the tokens
// (dWr) is always split into ranges that depend on the sizes alone, whose fp32 sums are added in ascending order, so the result does
// not depend on scheduling.
#include "common.h"
#include "kernels.h"

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float ldf(const float* p, size_t i) { return p[i]; }
__device__ __forceinline__ float ldf(const bf16_t* p, size_t i) { return bf16_to_f32(p[i]); }
__device__ __forceinline__ void stf(float* p, size_t i, float v) { p[i] = v; }
__device__ __forceinline__ void stf(bf16_t* p, size_t i, float v) { p[i] = f32_to_bf16(v); }

__device__ __forceinline__ float wave_sum_f(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, WAVE);
  return v;
}

constexpr int TM = 64, TN = 64, TK = 16;

// C[r,n] (=|+=) sum_k A[r,k] * B[k*b_rs + n*b_cs], r in [0,M), n in [0,N); fp32 accumulation in
// ascending k.  grid = (N tiles, M tiles), 256 threads, 4x4 outputs per thread.
template <typename TA, typename TB, typename TC>
__global__ __launch_bounds__(256) void gemm_rows_valu(const TA* __restrict__ A, int lda, const TB* __restrict__ B,
                                                     long b_rs, long b_cs, TC* __restrict__ C, int ldc, int M,
                                                     int N, int K, int beta) {
  const int row0 = blockIdx.y * TM, col0 = blockIdx.x * TN;
  __shared__ float sa[TK][TM + 1], sb[TK][TN + 1];
  const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < K; k0 += TK) {
    for (int i = threadIdx.x; i < TM * TK; i += 256) {
      const int m = i / TK, kk = i % TK;
      const int r = row0 + m, kidx = k0 + kk;
      sa[kk][m] = (r < M && kidx < K) ? ldf(A, (size_t)r * lda + kidx) : 0.f;
    }
    for (int i = threadIdx.x; i < TN * TK; i += 256) {
      int n, kk;
      if (b_cs == 1) { n = i % TN; kk = i / TN; } else { kk = i % TK; n = i / TK; }
      const int c = col0 + n, kidx = k0 + kk;
      sb[kk][n] = (c < N && kidx < K) ? ldf(B, (size_t)kidx * b_rs + (size_t)c * b_cs) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < TK; ++kk) {
      float av[4], bv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) av[i] = sa[kk][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) bv[j] = sb[kk][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] += av[i] * bv[j];
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = row0 + ty * 4 + i;
    if (r >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = col0 + tx * 4 + j;
      if (c < N) {
        const size_t idx = (size_t)r * ldc + c;
        stf(C, idx, beta ? ldf(C, idx) + acc[i][j] : acc[i][j]);
      }
    }
  }
}

// partial[z][i][j] = sum over rows r of chunk z of P[r,i] * Q[r,j]; chunk z = [z*chunk, min((z+1)*chunk, rows)).
// grid = (N tiles, M tiles, chunks)
template <typename TP>
__global__ __launch_bounds__(256) void gemm_tn_valu(const TP* __restrict__ P, int ldp, const float* __restrict__ Q,
                                                   int ldq, float* __restrict__ partial, int M, int N, int rows,
                                                   int chunk) {
  const long long lo_l = (long long)blockIdx.z * chunk;
  const int lo = (int)(lo_l < rows ? lo_l : rows);
  const int hi = (int)(lo_l + chunk < rows ? lo_l + chunk : rows);
  const int i0 = blockIdx.y * TM, j0 = blockIdx.x * TN;
  __shared__ float sa[TK][TM + 1], sb[TK][TN + 1];
  const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
  float acc[4][4] = {};
  // The loads of a step are independent of each other and travel while the step before is multiplied: a chunk of a small batch
  // is a few steps, each of which waited eight times for memory (256 tokens, d = 128, E = 8: 15.3 us, now 9.7).
  float na[TM * TK / 256], nb[TN * TK / 256];
  const auto fetch = [&](int r0) {
#pragma unroll
    for (int q = 0; q < TM * TK / 256; ++q) {
      const int t = threadIdx.x + 256 * q, r = r0 + t / TM, i = i0 + t % TM;
      na[q] = (r < hi && i < M) ? ldf(P, (size_t)r * ldp + i) : 0.f;
    }
#pragma unroll
    for (int q = 0; q < TN * TK / 256; ++q) {
      const int t = threadIdx.x + 256 * q, r = r0 + t / TN, j = j0 + t % TN;
      nb[q] = (r < hi && j < N) ? Q[(size_t)r * ldq + j] : 0.f;
    }
  };
  fetch(lo);
  for (int r0 = lo; r0 < hi; r0 += TK) {
#pragma unroll
    for (int q = 0; q < TM * TK / 256; ++q) sa[(threadIdx.x + 256 * q) / TM][(threadIdx.x + 256 * q) % TM] = na[q];
#pragma unroll
    for (int q = 0; q < TN * TK / 256; ++q) sb[(threadIdx.x + 256 * q) / TN][(threadIdx.x + 256 * q) % TN] = nb[q];
    __syncthreads();
    fetch(r0 + TK);
#pragma unroll
    for (int kk = 0; kk < TK; ++kk) {
      float av[4], bv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) av[i] = sa[kk][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) bv[j] = sb[kk][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] += av[i] * bv[j];
    }
    __syncthreads();
  }
  float* out = partial + (size_t)blockIdx.z * M * N;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int ii = i0 + ty * 4 + i;
    if (ii >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int jj = j0 + tx * 4 + j;
      if (jj < N) out[(size_t)ii * N + jj] = acc[i][j];
    }
  }
}

// out[i] = (beta ? out[i] : 0) + partial[0][i] + partial[1][i] + ...   (ascending chunk order)
template <typename TOut>
__global__ void reduce_chunks(const float* __restrict__ partial, int chunks, size_t n, TOut* __restrict__ out,
                              int beta) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    float s = 0.f;
    for (int c = 0; c < chunks; ++c) s += partial[(size_t)c * n + i];
    stf(out, i, beta ? ldf(out, i) + s : s);
  }
}

// dx[t,c] (=|+=) sum_e dl[t,e] * Wr[c,e] for a small number of experts (the plain path's router term of dx):
// one thread per 4 consecutive columns c, whose 4*E weights are contiguous in memory; the token's
// dlogits row sits in LDS.  1-D grid: block = (token, group of 1024 columns), column group fastest.
template <typename TW>
__global__ __launch_bounds__(256) void router_dx_small_e(const float* __restrict__ dl, const TW* __restrict__ wr,
                                                        TW* __restrict__ dx, int d, int E, int beta, int col_groups) {
  __shared__ float row[MOE_MAX_EXPERTS];
  const int t = blockIdx.x / col_groups;
  const int cg = blockIdx.x - t * col_groups;
  for (int e = threadIdx.x; e < E; e += 256) row[e] = dl[(size_t)t * E + e];
  __syncthreads();
  const int c0 = (cg * 256 + threadIdx.x) * 4;
  if (c0 >= d) return;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (c0 + i >= d) break;
    const TW* w = wr + (size_t)(c0 + i) * E;
    float s = 0.f;
    for (int e = 0; e < E; ++e) s += row[e] * ldf(w, e);
    acc[i] = s;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (c0 + i >= d) break;
    const size_t idx = (size_t)t * d + c0 + i;
    stf(dx, idx, beta ? ldf(dx, idx) + acc[i] : acc[i]);
  }
}

// logits[t,e] = sum_c x[t,c] * Wr[c,e] for a small number of experts: one block per token, eight
// experts per pass (their weights are contiguous in a row of Wr), columns strided over the threads,
// sums reduced lanes -> wavefront -> block in a fixed order.
template <typename TX>
__global__ __launch_bounds__(256) void router_fwd_small_e(const TX* __restrict__ x, const TX* __restrict__ wr,
                                                         float* __restrict__ logits, int d, int E) {
  __shared__ float red[8][4];
  const int t = blockIdx.x, lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
  for (int e0 = 0; e0 < E; e0 += 8) {
    const int ne = E - e0 < 8 ? E - e0 : 8;
    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.f;
    if (sizeof(TX) == 2 && (E & 7) == 0 && (d & 7) == 0) {
      // bf16, whole groups of eight: 16-byte loads of eight columns of x and of each column's eight weights
      const uint16_t* xb = reinterpret_cast<const uint16_t*>(x);
      const uint16_t* wb = reinterpret_cast<const uint16_t*>(wr);
      for (int c8 = threadIdx.x * 8; c8 < d; c8 += 2048) {
        const uint4 xq = *reinterpret_cast<const uint4*>(xb + (size_t)t * d + c8);
        const uint32_t* xu = reinterpret_cast<const uint32_t*>(&xq);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float xv = (j & 1) ? bf16hi(xu[j >> 1]) : bf16lo(xu[j >> 1]);
          const uint4 wq = *reinterpret_cast<const uint4*>(wb + (size_t)(c8 + j) * E + e0);
          const uint32_t* wu = reinterpret_cast<const uint32_t*>(&wq);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            acc[2 * i] += xv * bf16lo(wu[i]);
            acc[2 * i + 1] += xv * bf16hi(wu[i]);
          }
        }
      }
    } else {
      for (int c = threadIdx.x; c < d; c += 256) {
        const float xv = ldf(x, (size_t)t * d + c);
        const TX* w = wr + (size_t)c * E + e0;
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (i < ne) acc[i] += xv * ldf(w, i);
      }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float v = wave_sum_f(acc[i]);
      if (lane == 0) red[i][wave] = v;
    }
    __syncthreads();
    if ((int)threadIdx.x < ne)
      logits[(size_t)t * E + e0 + threadIdx.x] = (red[threadIdx.x][0] + red[threadIdx.x][1]) + (red[threadIdx.x][2] + red[threadIdx.x][3]);
    __syncthreads();
  }
}

// dlogits as bf16, where only their rows are wanted; the first block clears the ticket counters of the product that follows
__global__ void round_to_bf16(const float* __restrict__ in, bf16_t* __restrict__ out, size_t n, int32_t* __restrict__ words, int n_words) {
  if (blockIdx.x == 0 && (int)threadIdx.x < n_words) words[threadIdx.x] = 0;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    out[i] = f32_to_bf16(in[i]);
}

// dlogits for the matrix-core products, one block per 32 tokens (a piece of the contraction over the tokens):
//   dlb     [T][E] bf16 (NULL: not wanted): operand of the input-gradient product
//   pieces  [piece][plane][E][32] bf16: operand of the weight-gradient product, tokens contiguous.
//           PLANES = 1: rounded once, the path whose dlogits are bf16.  PLANES = 3: three terms whose sum keeps all 24 bits,
//           for shapes whose dlogits stay fp32, times `scale`.  The last piece ends at the last token, with zeros for the tokens that the
//           piece before it has covered (T >= 32).
// The first block also clears the ticket counters of the product that follows (n_words; a launch of its own otherwise).
template <int PLANES>
__global__ __launch_bounds__(256) void router_dl_operands(const float* __restrict__ dl, int T, int E, bf16_t* __restrict__ dlb,
                                                         bf16_t* __restrict__ pieces, float scale, int32_t* __restrict__ words, int n_words) {
  __shared__ float tile[32][65];
  const int tid = threadIdx.x;
  if (blockIdx.x == 0 && tid < n_words) words[tid] = 0;
  const int t0 = blockIdx.x * 32, base = T - 32 < t0 ? T - 32 : t0;
  for (int e0 = 0; e0 < E; e0 += 64) {
    __syncthreads();
    for (int i = tid; i < 32 * 64; i += 256) {
      const int t = base + (i >> 6), e = e0 + (i & 63);
      float v = 0.f;
      if (t >= t0 && t < T && e < E) {
        v = dl[(size_t)t * E + e];
        if (dlb) dlb[(size_t)t * E + e] = f32_to_bf16(v);
      }
      tile[i >> 6][i & 63] = v;
    }
    __syncthreads();
    const int e = e0 + (tid >> 2), k = 8 * (tid & 3);
    if (e < E) {
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = tile[k + i][tid >> 2] * scale;
#pragma unroll
      for (int p = 0; p < PLANES; ++p) {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          w[i] = pack_bf16x2(v[2 * i], v[2 * i + 1]);
          v[2 * i] -= bf16lo(w[i]);
          v[2 * i + 1] -= bf16hi(w[i]);
        }
        *reinterpret_cast<uint4*>(pieces + (((size_t)blockIdx.x * PLANES + p) * E + e) * 32 + k) = make_uint4(w[0], w[1], w[2], w[3]);
      }
    }
  }
}

// The router term of dx for E = 8 or 16 experts: a thread keeps the weights of its eight columns in registers and walks
// `tokens` tokens (their dlogits are uniform: scalar loads), so that what is left is the read-modify-write of dx, eight
// tokens in flight.  With one block per token, which fetched the weights again for each, T = 16384, d = 4096, E = 8 took
// 172 us.
template <int E>
__global__ __launch_bounds__(256) void router_dx_columns(const float* __restrict__ dl, const bf16_t* __restrict__ wr,
                                                        bf16_t* __restrict__ dx, int T, int d, int beta, int tokens, int col_groups) {
  const int tg = blockIdx.x / col_groups;
  const int c0 = ((blockIdx.x - tg * col_groups) * 256 + threadIdx.x) * 8;
  if (c0 >= d) return;
  float w[8][E];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int e = 0; e < E; e += 8) {
      const uint4 q = *reinterpret_cast<const uint4*>(wr + (size_t)(c0 + i) * E + e);
      const uint32_t* u = reinterpret_cast<const uint32_t*>(&q);
#pragma unroll
      for (int j = 0; j < 4; ++j) { w[i][e + 2 * j] = bf16lo(u[j]); w[i][e + 2 * j + 1] = bf16hi(u[j]); }
    }
  constexpr int AHEAD = 8;
  const int t_end = min(T, (tg + 1) * tokens);
  for (int t0 = tg * tokens; t0 < t_end; t0 += AHEAD) {
    u32x4 old[AHEAD];
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) {
      old[k] = u32x4{0u, 0u, 0u, 0u};
      if (beta) old[k] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(dx + (size_t)min(t0 + k, t_end - 1) * d + c0));
    }
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) {
      if (t0 + k >= t_end) break;
      const float* row = dl + (size_t)(t0 + k) * E;
      float acc[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = 0.f;
#pragma unroll
      for (int e = 0; e < E; ++e)
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] += row[e] * w[i][e];
      u32x4 out;
#pragma unroll
      for (int i = 0; i < 4; ++i) out[i] = pack_bf16x2(bf16lo(old[k][i]) + acc[2 * i], bf16hi(old[k][i]) + acc[2 * i + 1]);
      __builtin_nontemporal_store(out, reinterpret_cast<u32x4*>(dx + (size_t)(t0 + k) * d + c0));
    }
  }
}

// ---- fused backward of combine ------------------------------------------------------------
// One block per token.  dy[t] is read once; for each local slot the matching row of o is read,
// its dot product with dy[t] is reduced (lanes -> wavefront -> block, fixed order) and the
// gate-scaled row of d_o is written.  Bytes: (U + 2R) * d * b.
template <bool BF16>
__device__ __forceinline__ float dot_vec(u32x4 a, u32x4 b) {
  if (BF16) {
    float s = bf16lo(a.x) * bf16lo(b.x);
    s += bf16hi(a.x) * bf16hi(b.x);
    s += bf16lo(a.y) * bf16lo(b.y); s += bf16hi(a.y) * bf16hi(b.y);
    s += bf16lo(a.z) * bf16lo(b.z); s += bf16hi(a.z) * bf16hi(b.z);
    s += bf16lo(a.w) * bf16lo(b.w); s += bf16hi(a.w) * bf16hi(b.w);
    return s;
  } else {
    float s = __uint_as_float(a.x) * __uint_as_float(b.x);
    s += __uint_as_float(a.y) * __uint_as_float(b.y);
    s += __uint_as_float(a.z) * __uint_as_float(b.z);
    s += __uint_as_float(a.w) * __uint_as_float(b.w);
    return s;
  }
}
template <bool BF16>
__device__ __forceinline__ u32x4 scale_vec2(u32x4 v, float sc) {
  u32x4 r;
  if (BF16) {
    r.x = pack_bf16x2(bf16lo(v.x) * sc, bf16hi(v.x) * sc);
    r.y = pack_bf16x2(bf16lo(v.y) * sc, bf16hi(v.y) * sc);
    r.z = pack_bf16x2(bf16lo(v.z) * sc, bf16hi(v.z) * sc);
    r.w = pack_bf16x2(bf16lo(v.w) * sc, bf16hi(v.w) * sc);
  } else {
    r.x = __float_as_uint(__uint_as_float(v.x) * sc);
    r.y = __float_as_uint(__uint_as_float(v.y) * sc);
    r.z = __float_as_uint(__uint_as_float(v.z) * sc);
    r.w = __float_as_uint(__uint_as_float(v.w) * sc);
  }
  return r;
}

constexpr int CB_MAX_WAVES = 16;

template <bool BF16>
__global__ __launch_bounds__(1024) void combine_bwd_rows(const u32x4* __restrict__ dy, const u32x4* __restrict__ o,
                                                        int row_vecs, int k, const int32_t* __restrict__ inv,
                                                        const float* __restrict__ topk_w, u32x4* __restrict__ d_o,
                                                        float* __restrict__ dgate) {
  __shared__ float red[MOE_MAX_TOPK * CB_MAX_WAVES];
  const int t = blockIdx.x, tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
  const int n_waves = blockDim.x / WAVE;
  const int32_t* irow = inv + (size_t)t * k;         // uniform address: scalar loads
  for (int i = tid; i < k * CB_MAX_WAVES; i += blockDim.x) red[i] = 0.f;
  __syncthreads();
  for (int c0 = 0; c0 < row_vecs; c0 += blockDim.x) {
    const int c = c0 + tid;
    const bool in = c < row_vecs;
    u32x4 v = {0u, 0u, 0u, 0u};
    bool loaded = false;
    for (int j = 0; j < k; ++j) {                     // ascending slot j; the branch is block-uniform
      const int row = irow[j];
      if (row < 0) continue;
      if (!loaded) {
        if (in) v = __builtin_nontemporal_load(dy + (size_t)t * row_vecs + c);
        loaded = true;
      }
      float part = 0.f;
      if (in) {
        const u32x4 ov = __builtin_nontemporal_load(o + (size_t)row * row_vecs + c);
        part = dot_vec<BF16>(v, ov);
        __builtin_nontemporal_store(scale_vec2<BF16>(v, topk_w[(size_t)t * k + j]), d_o + (size_t)row * row_vecs + c);
      }
      part = wave_sum_f(part);
      if (lane == 0) red[j * CB_MAX_WAVES + wave] += part;   // each wavefront owns its column
    }
  }
  __syncthreads();
  if (tid < k) {
    float s = 0.f;
    for (int w = 0; w < n_waves; ++w) s += red[tid * CB_MAX_WAVES + w];
    dgate[(size_t)t * k + tid] = s;
  }
}

// ---- gradient through the gate weights ----------------------------------------------------
// One wavefront per token; lane j < k holds slot j (its expert, logit and dgate); each lane owns
// the logit positions lane + 64*i and writes them with one coalesced store.
template <int VPL>
__global__ __launch_bounds__(256) void gate_bwd_kernel(const float* __restrict__ logits,
                                                      const int32_t* __restrict__ topk_idx,
                                                      const float* __restrict__ dgate, int T, int E, int k, int mode,
                                                      float* __restrict__ dlogits) {
  const int lane = lane_id();
  const int wave = threadIdx.x / WAVE;
  const int waves_per_block = blockDim.x / WAVE;
  for (int t = blockIdx.x * waves_per_block + wave; t < T; t += gridDim.x * waves_per_block) {
    const float* row = logits + (size_t)t * E;
    const bool act = lane < k;
    int my_idx = act ? topk_idx[(size_t)t * k + lane] : -1;
    if (act) my_idx = my_idx < 0 ? 0 : (my_idx >= E ? E - 1 : my_idx);   // a corrupt index must not read out of bounds
    const float my_dg = act ? dgate[(size_t)t * k + lane] : 0.f;
    const float my_logit = act ? row[my_idx] : 0.f;
    float out[VPL];
#pragma unroll
    for (int i = 0; i < VPL; ++i) out[i] = 0.f;
    float d_sel = 0.f;
    if (mode == MOE_GATE_SOFTMAX_RENORM) {
      const float top = __shfl(my_logit, 0, WAVE);          // slot 0 holds the largest logit
      const float ex = act ? expf(my_logit - top) : 0.f;
      const float w = ex / wave_sum_f(ex);
      const float c = wave_sum_f(w * my_dg);
      d_sel = w * (my_dg - c);
    } else if (mode == MOE_GATE_SIGMOID_RENORM) {
      const float sg = act ? 1.0f / (1.0f + expf(-my_logit)) : 0.f;
      const float S = wave_sum_f(sg);
      const float c = wave_sum_f(sg / S * my_dg);
      d_sel = (my_dg - c) / S * sg * (1.0f - sg);
    } else {
      float v[VPL];
      float m = -INFINITY;
#pragma unroll
      for (int i = 0; i < VPL; ++i) {
        const int e = lane + i * WAVE;
        v[i] = e < E ? row[e] : -INFINITY;
        m = fmaxf(m, v[i]);
      }
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, WAVE));
      float den = 0.f;
#pragma unroll
      for (int i = 0; i < VPL; ++i) {
        v[i] = lane + i * WAVE < E ? expf(v[i] - m) : 0.f;
        den += v[i];
      }
      den = wave_sum_f(den);
      const float p_sel = act ? expf(my_logit - m) / den : 0.f;
      const float inner = wave_sum_f(p_sel * my_dg);
      d_sel = p_sel * (my_dg - inner);
#pragma unroll
      for (int i = 0; i < VPL; ++i) out[i] = -(v[i] / den) * inner;
    }
    for (int j = 0; j < k; ++j) {
      const int e = __shfl(my_idx, j, WAVE);
      const float dv = __shfl(d_sel, j, WAVE);
#pragma unroll
      for (int i = 0; i < VPL; ++i)
        if (lane + i * WAVE == e) out[i] = dv;
    }
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
      const int e = lane + i * WAVE;
      if (e < E) dlogits[(size_t)t * E + e] = out[i];
    }
  }
}

inline int tiles(int n, int t) { return (n + t - 1) / t; }

// split of the token contraction for the plain path: enough blocks to fill the chip, chunk sums
// bounded to 64 MB
int valu_splits(int T, int d, int E) {
  const long long blocks = (long long)tiles(d, TM) * tiles(E, TN);
  long long s = (4LL * device_cu_count() + blocks - 1) / blocks;
  const long long by_bytes = (64LL << 20) / ((long long)d * E * 4);
  if (s > by_bytes) s = by_bytes;
  if (s > tiles(T, 4 * TK)) s = tiles(T, 4 * TK);
  if (s > 64) s = 64;
  return s < 1 ? 1 : (int)s;
}

inline bool mfma_shape(int dtype, int T, int d, int E) {
  return dtype == MOE_BF16 && T > 0 && E % 64 == 0 && d % 64 == 0;
}

inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

}  // namespace

size_t router_ws_bytes(int dtype, int T, int d, int E) {
  size_t b = 256;                                           // ticket counters
  if (mfma_shape(dtype, T, d, E)) {
    // backward: dlogits rounded to bf16 + the chunk sums of dWr; forward: the logits of each range
    // of a cut contraction (the two calls use the same bytes one after the other)
    const size_t bwd = align256((size_t)T * E * 2) + align256((size_t)router_dw_splits(T, d, E) * d * E * 4);
    const int fs = router_fwd_splits(T, d, E);
    const size_t fwd = fs > 1 ? align256((size_t)fs * T * E * 4) : 0;
    b += bwd > fwd ? bwd : fwd;
  } else {
    b += align256((size_t)valu_splits(T, d, E) * d * E * 4);
  }
  return b;
}

int launch_router_fwd(const void* x, const void* wr, int dtype, int T, int d, int E, float* logits, void* ws,
                      hipStream_t s) {
  if (T == 0) return MOE_OK;
  if (dtype == MOE_BF16 && E % 8 == 0 && d % 64 == 0 && E < 64) return launch_router_fwd_narrow(x, wr, T, d, E, logits, s);
  if (dtype == MOE_BF16 && E % 8 == 0 && d % 64 == 0) {
    float* partial = (float*)((char*)ws + 256);
    const int room = mfma_shape(dtype, T, d, E) ? router_fwd_splits(T, d, E) : 1;      // what the workspace holds
    int splits = 1;
    // The streaming kernel reads the weights once per 64 tokens.  Up to a block of 64 tokens by 128 experts per CU it is the
    // faster one; beyond that it depends, mostly on d.  Calls one after the other (and with other memory written in between), streaming / big
    // tiles, us:
    //   within  T = 8192, d = 2048, E = 128 12.0 / 34.9 (22.8 / 43.7)    16384, 4096, 128 27.9 / 50.9 (56.4 / 73.4)    16384, 2048, 64 15.1 / 33.1 (33.8 / 49.3)
    //           8192, 4096, 256 27.6 / 55.6 (43.8 / 71.0)                16384, 7168, 128 44.5 / 68.9 (88.4 / 110.7)   8192, 7168, 256 43.0 / 65.1 (64.2 / 83.5)
    //   beyond  T = 20000, d = 4096, E = 128 47.1 / 55.0 (91.5 / 86.3)   32768, 4096, 128 67.6 / 83.4 (114.5 / 143.2)  32768, 2048, 64 30.7 / 44.0 (59.1 / 69.2)
    //           12000, 4096, 256 51.0 / 59.8 (70.7 / 79.1)               12000, 7168, 256 81.9 / 72.9 (110.7 / 107.3)  32768, 7168, 256 230 / 152 (262 / 182)
    // The two add a logit's products in different orders, so this line also decides bits; it has stayed where the two met before the
    // streaming kernel loaded x through LDS.
    const bool stream = !mfma_shape(dtype, T, d, E) || (long long)tiles(T, 64) * tiles(E, 128) <= device_cu_count();
    int rc;
    if (stream) {
      rc = launch_router_fwd_small(x, wr, T, d, E, logits, partial, room, &splits, s);
    } else {
      splits = room;
      rc = launch_router_fwd_bf16(x, wr, T, d, E, logits, partial, splits, (int32_t*)ws, s);
    }
    if (rc || splits == 1) return rc;
    ProfScope prof(MOE_K_ROUTER_FWD, s);
    hipLaunchKernelGGL((reduce_chunks<float>), dim3(device_cu_count() * 4), dim3(256), 0, s, partial, splits, (size_t)T * E,
                       logits, 0);
    HIP_CHECK_LAUNCH();
    return MOE_OK;
  }
  ProfScope prof(MOE_K_ROUTER_FWD, s);
  if (E <= 64) {
    if (dtype == MOE_BF16)
      hipLaunchKernelGGL((router_fwd_small_e<bf16_t>), dim3(T), dim3(256), 0, s, (const bf16_t*)x, (const bf16_t*)wr, logits, d, E);
    else
      hipLaunchKernelGGL((router_fwd_small_e<float>), dim3(T), dim3(256), 0, s, (const float*)x, (const float*)wr, logits, d, E);
  } else {
    dim3 grid(tiles(E, TN), tiles(T, TM)), blk(256);
    if (dtype == MOE_BF16)
      hipLaunchKernelGGL((gemm_rows_valu<bf16_t, bf16_t, float>), grid, blk, 0, s, (const bf16_t*)x, d, (const bf16_t*)wr,
                         (long)E, 1L, logits, E, T, E, d, 0);
    else
      hipLaunchKernelGGL((gemm_rows_valu<float, float, float>), grid, blk, 0, s, (const float*)x, d, (const float*)wr,
                         (long)E, 1L, logits, E, T, E, d, 0);
  }
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}

int launch_combine_bwd(const void* dy, const void* o, int dtype, int T, int d, int k, const int32_t* inv,
                       const float* topk_w, void* d_o, float* dgate, hipStream_t s) {
  if (T == 0) return MOE_OK;
  ProfScope prof(MOE_K_COMBINE_BWD, s);
  const int row_vecs = dtype == MOE_BF16 ? d / 8 : d / 4;
  int bs = (row_vecs + WAVE - 1) / WAVE * WAVE;
  if (bs > 1024) bs = 1024;
  if (bs < 64) bs = 64;
  if (dtype == MOE_BF16)
    hipLaunchKernelGGL((combine_bwd_rows<true>), dim3(T), dim3(bs), 0, s, (const u32x4*)dy, (const u32x4*)o, row_vecs, k,
                       inv, topk_w, (u32x4*)d_o, dgate);
  else
    hipLaunchKernelGGL((combine_bwd_rows<false>), dim3(T), dim3(bs), 0, s, (const u32x4*)dy, (const u32x4*)o, row_vecs, k,
                       inv, topk_w, (u32x4*)d_o, dgate);
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}

int launch_gate_bwd(const float* logits, const int32_t* topk_idx, const float* dgate, int T, int E, int k,
                    int gate_mode, float* dlogits, hipStream_t s) {
  if (T == 0) return MOE_OK;
  ProfScope prof(MOE_K_GATE_BWD, s);
  const int wpb = 4;
  int blocks = (T + wpb - 1) / wpb;
  const int maxb = device_cu_count() * 8;
  if (blocks > maxb) blocks = maxb;
  const int vpl = (E + WAVE - 1) / WAVE;
#define GATE_CASE(V)                                                                                          \
  hipLaunchKernelGGL(gate_bwd_kernel<V>, dim3(blocks), dim3(256), 0, s, logits, topk_idx, dgate, T, E, k, gate_mode, \
                     dlogits)
  if (vpl <= 1) GATE_CASE(1);
  else if (vpl <= 2) GATE_CASE(2);
  else if (vpl <= 4) GATE_CASE(4);
  else if (vpl <= 8) GATE_CASE(8);
  else GATE_CASE(16);
#undef GATE_CASE
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}

int launch_router_bwd(const void* x, const void* wr, const float* dlogits, int dtype, int T, int d, int E, void* dwr,
                      int dwr_acc, void* dx, int dx_acc, void* ws, hipStream_t s) {
  int32_t* sched = (int32_t*)ws;
  char* base = (char*)ws + 256;
  const size_t n_w = (size_t)d * E;
  const int red_blocks = device_cu_count() * 4;
  int rc;
  // Weight gradient: router_dw.hip where router_dw_ranges says so; else, up to 128 experts, the streaming kernel of few rows if the
  // workspace's partial sums leave room for its operand beside at least one sum per plane.  Its sums need no more bytes than the cut
  // product's.  More than 64 rows of planes take two passes over x, which the big tiles overtake where x is large: E = 128, few rows /
  // tiles, us: T = 32768, d = 2048 62 / 71; 16384, 4096 60 / 63; 16384, 7168 91 / 84; 32768, 4096 109 / 101; 65536, 4096 198 / 164.
  const bool mfma = mfma_shape(dtype, T, d, E);
  const int planes = mfma ? 1 : 3;
  const size_t sum_bytes = n_w * 4;
  const int splits = T == 0 ? 0 : mfma ? router_dw_splits(T, d, E) : valu_splits(T, d, E);
  const size_t room = align256((size_t)splits * sum_bytes);
  const size_t piece_bytes = align256((size_t)((T + 31) / 32) * 32 * planes * E * 2);
  const int max_sums = room > piece_bytes ? (int)((room - piece_bytes) / sum_bytes) : 0;
  const int ranges = dwr && dtype == MOE_BF16 ? router_dw_ranges(T, d, E, max_sums, splits) : 0;
  const bool dw_small = ranges > 0 || (dwr && dtype == MOE_BF16 && T >= 32 && d % 64 == 0 && planes * E <= 128 &&
                        !(mfma && E > 64 && (long long)T * d > (1ll << 26)) && max_sums >= planes);
  const auto dw_operands = [&](bf16_t* dlb, bf16_t* pieces) -> int {
    ProfScope prof(dwr ? MOE_K_ROUTER_DW : MOE_K_ROUTER_DX, s);
    if (!pieces)
      hipLaunchKernelGGL(round_to_bf16, dim3(red_blocks), dim3(256), 0, s, dlogits, dlb, (size_t)T * E, sched, 16);
    else if (planes == 1)
      hipLaunchKernelGGL(router_dl_operands<1>, dim3((T + 31) / 32), dim3(256), 0, s, dlogits, T, E, dlb, pieces, 1.f, sched, 16);
    else
      hipLaunchKernelGGL(router_dl_operands<3>, dim3((T + 31) / 32), dim3(256), 0, s, dlogits, T, E, dlb, pieces, ranges > 0 ? DL_SCALE : 1.f,
                         sched, 0);
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_EHIP;
  };
  const auto dw_stream = [&](bf16_t* pieces) -> int {
    float* sums = (float*)((char*)pieces + piece_bytes);
    int n = ranges;
    const int rc2 = ranges > 0 ? launch_router_dw_stream(x, pieces, dlogits, T, d, E, sums, ranges, s)
                               : launch_router_dw_small(x, pieces, planes, T, d, E, sums, max_sums, &n, s);
    if (rc2) return rc2;
    ProfScope prof(MOE_K_ROUTER_DW, s);
    hipLaunchKernelGGL((reduce_chunks<bf16_t>), dim3(red_blocks), dim3(256), 0, s, sums, n, n_w, (bf16_t*)dwr, dwr_acc);
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_EHIP;
  };
  if (mfma) {
    bf16_t* dlb = (bf16_t*)base;
    float* partial = (float*)(base + align256((size_t)T * E * 2));
    if ((rc = dw_operands(dlb, dw_small ? (bf16_t*)partial : nullptr))) return rc;
    if (dw_small) {
      if ((rc = dw_stream((bf16_t*)partial))) return rc;
    } else if (dwr) {
      if ((rc = launch_router_dw_bf16(x, dlb, T, d, E, partial, splits, sched, s))) return rc;
      ProfScope prof(MOE_K_ROUTER_DW, s);
      hipLaunchKernelGGL((reduce_chunks<bf16_t>), dim3(red_blocks), dim3(256), 0, s, partial, splits, n_w, (bf16_t*)dwr,
                         dwr_acc);
      HIP_CHECK_LAUNCH();
    }
    if (dx && router_dx_streams(E, d)) return launch_router_dx_stream(dlb, wr, T, d, E, dx, dx_acc, s);
    if (dx) return launch_router_dx_bf16(dlb, wr, T, d, E, dx, dx_acc, sched + 8, s);
    return MOE_OK;
  }
  float* partial = (float*)base;
  if (dw_small) {
    if ((rc = dw_operands(nullptr, (bf16_t*)base))) return rc;
    if ((rc = dw_stream((bf16_t*)base))) return rc;
  } else if (dwr) {
    if (splits > 0) {
      ProfScope prof(MOE_K_ROUTER_DW, s);
      const int chunk = (T + splits - 1) / splits;
      dim3 grid(tiles(E, TN), tiles(d, TM), splits), blk(256);
      if (dtype == MOE_BF16)
        hipLaunchKernelGGL((gemm_tn_valu<bf16_t>), grid, blk, 0, s, (const bf16_t*)x, d, dlogits, E, partial, d, E, T, chunk);
      else
        hipLaunchKernelGGL((gemm_tn_valu<float>), grid, blk, 0, s, (const float*)x, d, dlogits, E, partial, d, E, T, chunk);
      HIP_CHECK_LAUNCH();
    }
    if (dtype == MOE_BF16)
      hipLaunchKernelGGL((reduce_chunks<bf16_t>), dim3(red_blocks), dim3(256), 0, s, partial, splits, n_w, (bf16_t*)dwr, dwr_acc);
    else
      hipLaunchKernelGGL((reduce_chunks<float>), dim3(red_blocks), dim3(256), 0, s, partial, splits, n_w, (float*)dwr, dwr_acc);
    HIP_CHECK_LAUNCH();
  }
  if (dx && T > 0 && dtype == MOE_BF16 && router_dx_streams(E, d)) return launch_router_dx_stream(dlogits, wr, T, d, E, dx, dx_acc, s);
  if (dx && T > 0) {
    ProfScope prof(MOE_K_ROUTER_DX, s);
    if (dtype == MOE_BF16 && (E == 8 || E == 16) && (long long)T * d * E >= (1ll << 23)) {
      // Below that a block per token is faster; walking tokens, the longer the fewer blocks there are, is what a small
      // batch waits for.  A block per token / 8 / 16 / 32 tokens per block, us:
      //   E = 8:  T = 64, d = 4096 3.8 / 4.7 / 6.6 / 10.7    512, 2048 4.9 / 4.9 / 6.8 / 11.0    2000, 4096 19 / 8.5 / 8.2 / 11.7
      //           4096, 4096 35 / 15.5 / 13.9 / 15.1         9001, 7168 151 / 60 / 54 / 57       16384, 4096 128 / - / 53 / 52
      //   E = 16: T = 64, d = 4096 4.7 / 6.6 / 9.8 / 16.5    512, 2048 7.5 / 6.8 / 10.0 / 16.7   2000, 4096 41 / 12.0 / 12.0 / 17.7
      //           4096, 4096 81 / 20.5 / 18.4 / 20.4         9001, 7168 483 / 70 / 68 / 66       16384, 4096 318 / - / 65 / 58
      const int tokens = (long long)T * d < (1ll << 23) ? 8 : ((long long)T * d < (1ll << 26) ? 16 : 32);
      const int col_groups = tiles(d, 2048);
      dim3 grid((unsigned)col_groups * tiles(T, tokens)), blk(256);
      if (E == 8)
        hipLaunchKernelGGL(router_dx_columns<8>, grid, blk, 0, s, dlogits, (const bf16_t*)wr, (bf16_t*)dx, T, d, dx_acc, tokens, col_groups);
      else
        hipLaunchKernelGGL(router_dx_columns<16>, grid, blk, 0, s, dlogits, (const bf16_t*)wr, (bf16_t*)dx, T, d, dx_acc, tokens, col_groups);
    } else if (E <= 64) {
      // a handful of experts: per-token dot products against contiguous weight rows
      const int col_groups = tiles(d, 1024);
      if ((long long)col_groups * T >= (1ll << 31)) return MOE_EUNSUPPORTED;
      dim3 grid((unsigned)(col_groups * T)), blk(256);
      if (dtype == MOE_BF16)
        hipLaunchKernelGGL((router_dx_small_e<bf16_t>), grid, blk, 0, s, dlogits, (const bf16_t*)wr, (bf16_t*)dx, d, E, dx_acc, col_groups);
      else
        hipLaunchKernelGGL((router_dx_small_e<float>), grid, blk, 0, s, dlogits, (const float*)wr, (float*)dx, d, E, dx_acc, col_groups);
    } else {
      // dx[t,n] (+)= sum_e dl[t,e] * Wr[n,e] : B(k = e, n) = Wr[n*E + e]
      dim3 grid(tiles(d, TN), tiles(T, TM)), blk(256);
      if (dtype == MOE_BF16)
        hipLaunchKernelGGL((gemm_rows_valu<float, bf16_t, bf16_t>), grid, blk, 0, s, dlogits, E, (const bf16_t*)wr, 1L, (long)E,
                           (bf16_t*)dx, d, T, d, E, dx_acc);
      else
        hipLaunchKernelGGL((gemm_rows_valu<float, float, float>), grid, blk, 0, s, dlogits, E, (const float*)wr, 1L, (long)E,
                           (float*)dx, d, T, d, E, dx_acc);
    }
    HIP_CHECK_LAUNCH();
  }
  return MOE_OK;
}
