// Shared device helpers for the gfx950 MoE kernels (wave64, CDNA4).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define WAVE 64

typedef uint16_t bf16_t;   // raw bfloat16 bits in memory

__device__ __forceinline__ float bf16_to_f32(bf16_t v) { return __uint_as_float(((uint32_t)v) << 16); }

// round-to-nearest-even; inputs are finite
__device__ __forceinline__ bf16_t f32_to_bf16(float x) {
  uint32_t u = __float_as_uint(x);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

// two floats -> packed bf16 pair, round-to-nearest-even, in one v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
__device__ __forceinline__ float bf16lo(uint32_t v) { return __uint_as_float(v << 16); }
__device__ __forceinline__ float bf16hi(uint32_t v) { return __uint_as_float(v & 0xFFFF0000u); }

__device__ __forceinline__ int lane_id() { return threadIdx.x & (WAVE - 1); }

// f(Int<0>{}), .., f(Int<N - 1>{})
template <int V> struct Int { static constexpr int value = V; };
template <int N, typename F>
__device__ __forceinline__ void static_for(F f) {
  if constexpr (N > 1) static_for<N - 1>(f);
  f(Int<N - 1>{});
}

// The tile of workgroup b in a launch whose list of tiles is known on the device only: experts in ascending order, each
// cut into row tiles of TM rows, each of them into n_cols column tiles (fastest).  Workgroup b runs on XCD b % 8, and every
// XCD takes a contiguous eighth of the list, so that an expert's weights pass through one or two of the eight L2s instead
// of all of them.  The grid is the host's bound on the list rounded up to a multiple of eight: false for a surplus
// workgroup.  Called by whole wavefronts; 64 experts per step.
template <int TM>
__device__ __forceinline__ int row_tiles_scan(const int32_t* __restrict__ off, int e_cnt, int e, int lane, int& n) {
  n = e < e_cnt ? (off[e + 1] - off[e] + TM - 1) / TM : 0;
  int incl = n;
#pragma unroll
  for (int o = 1; o < WAVE; o <<= 1) {
    const int v = __shfl_up(incl, o, WAVE);
    if (lane >= o) incl += v;
  }
  return incl;
}
template <int TM>
__device__ __forceinline__ bool ragged_tile(const int32_t* __restrict__ off, int e_cnt, int n_cols, int b, int lane, int& e,
                                            int& row_tile, int& col_tile) {
  int n, incl = row_tiles_scan<TM>(off, e_cnt, lane, lane, n);
  int total = __builtin_amdgcn_readfirstlane(__shfl(incl, WAVE - 1, WAVE));
  for (int base = WAVE; base < e_cnt; base += WAVE) {
    int m;
    total += __builtin_amdgcn_readfirstlane(__shfl(row_tiles_scan<TM>(off, e_cnt, base + lane, lane, m), WAVE - 1, WAVE));
  }
  const int share = (total * n_cols + 7) / 8;
  const int tile = (b % 8) * share + b / 8;
  if (b / 8 >= share || tile >= total * n_cols) return false;
  int t = tile / n_cols;
  col_tile = tile - t * n_cols;
  for (int base = 0;; base += WAVE) {          // ends: t < total
    if (base > 0) incl = row_tiles_scan<TM>(off, e_cnt, base + lane, lane, n);
    const unsigned long long past = __ballot(incl > t);
    if (past) {
      const int who = __builtin_ctzll(past);
      row_tile = __builtin_amdgcn_readfirstlane(t - __shfl(incl - n, who, WAVE));
      e = base + who;
      return true;
    }
    t = __builtin_amdgcn_readfirstlane(t - __shfl(incl, WAVE - 1, WAVE));
  }
}

// logistic function with the hardware exp2 and reciprocal (about 1 ulp each; used by the bf16
// epilogues, whose results are rounded to 8 bits of mantissa)
__device__ __forceinline__ float sigmoid_fast(float z) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896f * z));
}
__device__ __forceinline__ float silu_f(float z) { return z * sigmoid_fast(z); }
// returns silu(z) and writes silu'(z) = s (1 + z (1 - s))
__device__ __forceinline__ float silu_grad_f(float z, float* ds) {
  float s = sigmoid_fast(z);
  *ds = s * (1.0f + z * (1.0f - s));
  return z * s;
}

#define HIP_CHECK_LAUNCH()                                  \
  do {                                                      \
    if (hipGetLastError() != hipSuccess) return MOE_EHIP;   \
  } while (0)
