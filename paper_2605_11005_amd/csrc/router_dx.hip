// Input gradient of the trainable router, dx (+)= dlogits Wr^T, in bf16 for 32 to 256 experts: a stream over dx.
//
// Bound by memory: dx is read and written once (2 T d 2 bytes), and everything else is kept off that path.  A wavefront owns 64
// columns and holds their weights, all of the contraction, in registers while it walks tokens; the dlogits of 32 or 64 tokens
// travel through LDS, two buffers, and serve the 256 columns of a block.  The weights are the matrix instruction's first operand, in an
// order of columns that leaves a lane with eight consecutive columns of a token twice: old values and results move as 16 bytes per
// lane and 64 per token without passing through LDS.  Two blocks per CU, so that one's loads travel while the other multiplies.
// Input gradient alone (where E % 64 == 0 with the pass that rounds the dlogits), us; before, on 256x256 tiles or, E = 32 and 96, in
// plain fp32 products, / now / dx read and written at 6.5 TB/s:
//   T = 4096, d = 2048, E = 64      18.6 / 13.9 / 5      T = 16384, d = 4096, E = 128   67 / 51 / 41     T = 30000, d = 7168, E = 128  215 / 203 / 132
//   T = 9001, d = 2880, E = 128     35 / 30 / 16         T = 16384, d = 7168, E = 256  125 / 97 / 72     T = 4096, d = 7168, E = 192   39 / 32 / 18
//   T = 64, d = 4096, E = 96        19 / 10              T = 8192, d = 4096, E = 96    151 / 30 / 21     T = 30000, d = 7168, E = 32  3191 / 187 / 132
// Small batches of 32 experts, a block per token / now: T = 1, d = 512 4.2 / 3.6; 32, 512 4.4 / 4.0; 64, 512 4.5 / 4.5; 128, 512 4.5 / 4.7; 400, 512 4.7 / 4.7;
// 64, 2048 5.3 / 4.7; 200, 2048 6.6 / 5.0: no line in T is drawn for the 0.2 us between 100 and 400 tokens of d <= 512.
// Long rows leave few walks: T = 600, d = 16384, E = 64 19.5 / 15.8, 128 20.1 / 21.5, 192 21.0 / 19.8 (with tiles of 64 tokens, whose registers
// did not suffice, 24.0), 256 22.4 / 22.2.
// Old values fetched a tile ahead changed nothing.
#include "common.h"
#include "kernels.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NT = 256, COLS = 256, WAVE_COLS = 64;

// NK: experts / 32.  SPLIT: the dlogits stay fp32, as three bf16 terms that keep all 24 bits; else they come rounded to bf16.
template <int NK, bool SPLIT> struct Shape {
  static constexpr int E = 32 * NK, PLANES = SPLIT ? 3 : 1;
  static constexpr int ROW = (PLANES * E * 2 + 127) / 128 * 128;       // bytes of a token in LDS
  static constexpr int TG = NK >= 6 || (SPLIT && NK > 1) ? 2 : 4;      // groups of 16 tokens in a tile: what registers and LDS hold
  static constexpr int TOKENS = 16 * TG, BUFFER = TOKENS * ROW;
  // place of 16-byte chunk c of a token: sixteen lanes that read one chunk of consecutive tokens must cover 256 distinct bytes
  static __device__ __forceinline__ int swizzle(int token, int c) { return ROW % 256 ? c ^ ((token >> 1) & 7) : c ^ (token & 15); }
};

template <int NK, bool SPLIT>
__global__ __launch_bounds__(NT, 2) void router_dx_stream(const void* __restrict__ dl, const bf16_t* __restrict__ wr, bf16_t* __restrict__ dx,
                                                         int T, int d, int accumulate, int n_cols, int n_walks) {
  using S = Shape<NK, SPLIT>;
  constexpr int TOKENS = S::TOKENS, TG = S::TG;
  extern __shared__ __align__(16) char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, g = lane >> 4;
  // a walk takes every n_walks-th tile; its column blocks run on one XCD, whose L2 then holds their dlogits
  const int at = blockIdx.x / 8, walk = at / n_cols * 8 + blockIdx.x % 8;
  if (walk >= n_walks) return;
  const int c0 = (at % n_cols) * COLS + wave * WAVE_COLS;
  const bool active = c0 < d;                                          // d % 64 == 0: all of a wavefront's columns or none
  const int n_tiles = (T + TOKENS - 1) / TOKENS;

  // element r of lane group g of column block b is column 8 (4 (b / 2) + g) + 4 (b % 2) + r: blocks 2j and 2j + 1 make eight
  // consecutive ones
  bf16x8 w[4][NK];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int col = (active ? c0 : 0) + 8 * (4 * (b >> 1) + (i >> 2)) + 4 * (b & 1) + (i & 3);
#pragma unroll
    for (int q = 0; q < NK; ++q) w[b][q] = *reinterpret_cast<const bf16x8*>(wr + (size_t)col * S::E + 32 * q + 8 * g);
  }

  // bf16 dlogits: straight to LDS, 1 KB per load in the order of the buffer; fp32: through registers
  constexpr int LOADS = S::BUFFER / 1024 / 4, VECS = TOKENS * S::E / 4 / NT;
  float4 v[SPLIT ? VECS : 1];
  auto fetch = [&](int tile, int buf) {
    const int t0 = tile * TOKENS;
    if constexpr (SPLIT) {
#pragma unroll
      for (int n = 0; n < VECS; ++n) {
        const int at4 = tid + NT * n, token = min(at4 / (S::E / 4), T - 1 - t0);
        v[n] = *reinterpret_cast<const float4*>((const float*)dl + (size_t)(t0 + token) * S::E + 4 * (at4 % (S::E / 4)));
      }
    } else {
#pragma unroll
      for (int n = 0; n < LOADS; ++n) {
        const int place = (wave * LOADS + n) * 1024 + lane * 16, token = place / S::ROW, c = S::swizzle(token, place % S::ROW / 16);
        lds_load16((const bf16_t*)dl + (size_t)t0 * S::E, (uint32_t)(min(token, T - 1 - t0) * S::E * 2 + c * 16),
                   lds_addr(lds) + buf * S::BUFFER + (wave * LOADS + n) * 1024);
      }
    }
  };
  auto publish = [&](int buf) {          // the fetched tile is in LDS once a barrier follows
    if constexpr (SPLIT) {
#pragma unroll
      for (int n = 0; n < VECS; ++n) {
        const int at4 = tid + NT * n, token = at4 / (S::E / 4), e = 4 * (at4 % (S::E / 4));
        float x[4] = {v[n].x * DL_SCALE, v[n].y * DL_SCALE, v[n].z * DL_SCALE, v[n].w * DL_SCALE};
#pragma unroll
        for (int p = 0; p < 3; ++p) {      // the leading 8 bits each time
          uint32_t h[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            h[r] = __float_as_uint(x[r]) & 0xFFFF0000u;
            x[r] -= __uint_as_float(h[r]);
          }
          const int k = p * S::E + e;
          *reinterpret_cast<uint2*>(lds + buf * S::BUFFER + token * S::ROW + S::swizzle(token, k >> 3) * 16 + (k & 4) * 2) =
              make_uint2(h[1] | h[0] >> 16, h[3] | h[2] >> 16);
        }
      }
    } else {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
  };

  if (walk < n_tiles) {
    fetch(walk, 0);
    publish(0);
  }
  __syncthreads();
  for (int tile = walk, buf = 0; tile < n_tiles; tile += n_walks, buf ^= 1) {
    const int t0 = tile * TOKENS;
    const bool more = tile + n_walks < n_tiles;
    if (more) fetch(tile + n_walks, buf ^ 1);
    bf16_t* const rows = dx + (size_t)t0 * d + (active ? c0 : 0) + 8 * g;      // token i of group t: (16 t + i) d further on
    uint4 old[TG][2];
    if (accumulate) {
#pragma unroll
      for (int t = 0; t < TG; ++t)
#pragma unroll
        for (int j = 0; j < 2; ++j) old[t][j] = *reinterpret_cast<const uint4*>(rows + (size_t)min(16 * t + i, T - 1 - t0) * d + 32 * j);
    }
    f32x4 acc[4][TG];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int t = 0; t < TG; ++t) acc[b][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < S::PLANES * NK; ++k)
#pragma unroll
      for (int t = 0; t < TG; ++t) {
        const int token = 16 * t + i;
        const bf16x8 f = *reinterpret_cast<const bf16x8*>(lds + buf * S::BUFFER + token * S::ROW + S::swizzle(token, 4 * k + g) * 16);
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[b][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[b][k % NK], f, acc[b][t], 0, 0, 0);
      }
    if (more) publish(buf ^ 1);
    // The terms of an infinite dlogit are no sum of it, and an empty term makes NaN of an infinite weight: outputs whose sums are no
    // numbers are formed in plain fp32, by the lanes that hold some.
    float probe = 0.f;
    if constexpr (SPLIT) {
#pragma unroll
      for (int n = 0; n < 16 * TG; ++n) probe += acc[n >> 2 & 3][n >> 4][n & 3] * 0.f;
    }
    if (SPLIT && probe != 0.f) {
#pragma unroll 1
      for (int n = 0; n < 16 * TG; ++n) {
        const int t = n >> 4, b = n >> 2 & 3, token = t0 + 16 * t + i;
        if (!active || token >= T) continue;
        float sum = 0.f;
#pragma unroll
        for (int o = 0; o < 16 * TG; ++o) sum = o == n ? acc[o >> 2 & 3][o >> 4][o & 3] : sum;
        const int col = c0 + 8 * (4 * (b >> 1) + g) + 4 * (b & 1) + (n & 3);
        if (fabsf(sum) < INFINITY) {
          sum *= DL_UNSCALE;
        } else {
          sum = 0.f;
          for (int e = 0; e < S::E; ++e) sum += ((const float*)dl)[(size_t)token * S::E + e] * bf16_to_f32(wr[(size_t)col * S::E + e]);
        }
        bf16_t* const out = dx + (size_t)token * d + col;
        *out = (bf16_t)pack_bf16x2(accumulate ? bf16_to_f32(*out) + sum : sum, 0.f);
      }
    } else {
#pragma unroll
      for (int t = 0; t < TG; ++t)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          float x[8];
#pragma unroll
          for (int r = 0; r < 8; ++r) x[r] = acc[2 * j + (r >> 2)][t][r & 3] * (SPLIT ? DL_UNSCALE : 1.f);
          if (accumulate) {
            const uint32_t u[4] = {old[t][j].x, old[t][j].y, old[t][j].z, old[t][j].w};
#pragma unroll
            for (int r = 0; r < 4; ++r) { x[2 * r] += bf16lo(u[r]); x[2 * r + 1] += bf16hi(u[r]); }
          }
          if (active && t0 + 16 * t + i < T)
            *reinterpret_cast<uint4*>(rows + (size_t)(16 * t + i) * d + 32 * j) =
                make_uint4(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]), pack_bf16x2(x[6], x[7]));
        }
    }
    __syncthreads();
  }
}

template <int NK, bool SPLIT>
int launch(const void* dl, const bf16_t* wr, bf16_t* dx, int T, int d, int accumulate, hipStream_t s) {
  constexpr int LDS = 2 * Shape<NK, SPLIT>::BUFFER;
  static_assert(LDS <= 64 * 1024, "more needs an opt-in");
  // two blocks per CU, and as many walks on every XCD: with the 18 that d = 7168 would allow two XCDs have three (T = 30000, E = 128:
  // 261 us)
  const int n_cols = (d + COLS - 1) / COLS, n_tiles = (T + Shape<NK, SPLIT>::TOKENS - 1) / Shape<NK, SPLIT>::TOKENS;
  const int most = 2 * device_cu_count() / n_cols, n_walks = most < 8 ? (most > 0 ? most : 1) : most / 8 * 8;
  const long long blocks = (long long)((n_walks + 7) / 8) * 8 * n_cols;
  if (blocks >= (1ll << 31)) return MOE_EUNSUPPORTED;
  hipLaunchKernelGGL((router_dx_stream<NK, SPLIT>), dim3((unsigned)blocks), dim3(NT), LDS, s, dl, wr, dx, T, d, accumulate, n_cols, n_walks);
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}

}  // namespace

// dl: bf16 where E % 64 == 0, else fp32 (E = 32, 96 or 160: their three terms fit LDS twice)
bool router_dx_streams(int E, int d) { return d % 64 == 0 && (E == 32 || E == 96 || E == 160 || (E % 64 == 0 && E <= 256)); }
int launch_router_dx_stream(const void* dl, const void* wr, int T, int d, int E, void* dx, int accumulate, hipStream_t s) {
  if (T == 0) return MOE_OK;
  ProfScope prof(MOE_K_ROUTER_DX, s);
  const bf16_t* w = (const bf16_t*)wr;
  bf16_t* x = (bf16_t*)dx;
  switch (E / 32) {
    case 1: return launch<1, true>(dl, w, x, T, d, accumulate, s);
    case 2: return launch<2, false>(dl, w, x, T, d, accumulate, s);
    case 3: return launch<3, true>(dl, w, x, T, d, accumulate, s);
    case 4: return launch<4, false>(dl, w, x, T, d, accumulate, s);
    case 5: return launch<5, true>(dl, w, x, T, d, accumulate, s);
    case 6: return launch<6, false>(dl, w, x, T, d, accumulate, s);
    default: return launch<8, false>(dl, w, x, T, d, accumulate, s);
  }
}
