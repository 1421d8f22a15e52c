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

// inclusive sums over a wavefront, on the DPP network: within rows of 16, then across them
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_add(int v) { return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, false); }
__device__ __forceinline__ int wave_scan(int v) {
  v = dpp_add<0x111, 0xF>(v);      // row_shr:1, 2, 4, 8
  v = dpp_add<0x112, 0xF>(v);
  v = dpp_add<0x114, 0xF>(v);
  v = dpp_add<0x118, 0xF>(v);
  v = dpp_add<0x142, 0xA>(v);      // row_bcast:15 into rows 1 and 3
  return dpp_add<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
}
__device__ __forceinline__ int wave_sum(int v) { return __builtin_amdgcn_readlane(wave_scan(v), WAVE - 1); }

// The tiles of a launch whose list is known on the device only: experts in ascending order, each cut into row tiles of TM rows,
// each of them into n_cols column tiles (fastest).  Workgroup b runs on XCD b % 8, and every XCD takes a contiguous eighth of the
// list, so that an expert's weights pass through one or two of the eight L2s instead of all of them.  The grid is the host's bound
// on the list rounded up to a multiple of eight.  Called by whole wavefronts; 64 experts per step.
template <int TM>
struct RaggedTiles {
  const int32_t* off;
  int e_cnt, lane;
  int n, incl;         // row tiles of expert `lane`, and of all up to it
  int total;           // row tiles of all experts
  int active;          // experts that have rows
  __device__ __forceinline__ int scan(int e, int& rows) const {
    rows = e < e_cnt ? (off[e + 1] - off[e] + TM - 1) / TM : 0;
    return wave_scan(rows);
  }
  __device__ __forceinline__ RaggedTiles(const int32_t* __restrict__ off_, int e_cnt_, int lane_) : off(off_), e_cnt(e_cnt_), lane(lane_) {
    incl = scan(lane, n);
    total = __builtin_amdgcn_readlane(incl, WAVE - 1);
    active = __popcll(__ballot(n > 0));
    for (int base = WAVE; base < e_cnt; base += WAVE) {
      int m;
      total += __builtin_amdgcn_readlane(scan(base + lane, m), WAVE - 1);
      active += __popcll(__ballot(m > 0));
    }
  }
  // the tile of workgroup b; false for a surplus one
  __device__ __forceinline__ bool tile(int n_cols, int b, int& e, int& row_tile, int& col_tile) const {
    const int share = (total * n_cols + 7) / 8;
    const int at = (b % 8) * share + b / 8;
    if (b / 8 >= share || at >= total * n_cols) return false;
    int t = at / n_cols, rows = n, up_to = incl;
    col_tile = at - t * n_cols;
    for (int base = 0;; base += WAVE) {          // ends: t < total
      if (base > 0) up_to = scan(base + lane, rows);
      const unsigned long long past = __ballot(up_to > t);
      if (past) {
        const int who = __builtin_ctzll(past);
        row_tile = t - __builtin_amdgcn_readlane(up_to - rows, who);
        e = base + who;
        return true;
      }
      t -= __builtin_amdgcn_readlane(up_to, WAVE - 1);
    }
  }
};

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

// 16 bytes per lane from global memory straight into LDS: lane l lands at lds_wave_base + 16*l
// (lds_wave_base is wave-uniform and travels in M0).  The global address is a wave-uniform
// 64-bit base in SGPRs plus a 32-bit per-lane byte offset: with 64-bit per-lane addresses the
// address path, not the data path, limits a CU to ~27 B/clk; this form sustains ~42 B/clk.
// Written as inline assembly so that the compiler's wait-count pass does not serialise later
// LDS reads against these loads; the kernel waits for them itself (s_waitcnt vmcnt) before
// the barrier that publishes a tile.
// STREAM: the line is used once ("nt").
template <bool STREAM = false>
__device__ __forceinline__ void lds_load16(const bf16_t* sbase, uint32_t voff_bytes, uint32_t lds_wave_base) {
  // make the uniformity of the base explicit so that it is allocated to an SGPR pair
  const uint64_t u = (uint64_t)sbase;
  const uint64_t ub = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(u >> 32)) << 32) |
                      (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
  sbase = (const bf16_t*)ub;
  if (STREAM)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                 :
                 : "s"(lds_wave_base), "v"(voff_bytes), "s"(sbase)
                 : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds_wave_base), "v"(voff_bytes), "s"(sbase)
                 : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

#define HIP_CHECK_LAUNCH()                                  \
  do {                                                      \
    if (hipGetLastError() != hipSuccess) return MOE_EHIP;   \
  } while (0)
