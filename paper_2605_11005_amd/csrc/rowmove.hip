// Row movers: dispatch (token order -> expert order) and combine (expert order -> token
// order, gate-weighted).  Both are token-major (a token's row is split over a few blocks), so every row
// of x / o is read exactly once and every row of xp / y is written exactly once:
//   dispatch : read x[t] once (skipped when the token has no local slot, but for a few slots, whose
//              plan is made meanwhile), write it to each of the token's local rows
//                                                   -> (U + R) * d * b bytes
//   combine  : read the token's local rows, write y[t] once (zeros when none)
//                                                   -> (R + T) * d * b bytes
// Accesses are 16 bytes per lane and one vector per thread: on this chip a plain copy is fastest
// with the largest possible number of small threads.  Dispatch numbers its blocks row-segment
// fastest, token next, so that blocks resident together work on consecutive 2 KB pieces of the
// same rows (source and destinations): DRAM pages are used while they are open.
#include "common.h"
#include "kernels.h"

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <bool BF16>
__device__ __forceinline__ u32x4 scale_vec(u32x4 v, float sc) {
  if (BF16) {
    u32x4 r;
    r.x = pack_bf16x2(bf16lo(v.x) * sc, bf16hi(v.x) * sc);
    r.y = pack_bf16x2(bf16lo(v.y) * sc, bf16hi(v.y) * sc);
    r.z = pack_bf16x2(bf16lo(v.z) * sc, bf16hi(v.z) * sc);
    r.w = pack_bf16x2(bf16lo(v.w) * sc, bf16hi(v.w) * sc);
    return r;
  } else {
    u32x4 r;
    r.x = __float_as_uint(__uint_as_float(v.x) * sc);
    r.y = __float_as_uint(__uint_as_float(v.y) * sc);
    r.z = __float_as_uint(__uint_as_float(v.z) * sc);
    r.w = __float_as_uint(__uint_as_float(v.w) * sc);
    return r;
  }
}

// row_vecs = number of 16-byte vectors per row; one vector per thread.
// dispatch: 1-D grid of T * n_seg blocks of 128 threads, block = (token t, segment of 128 vectors),
//   segment fastest.  Measured at T = 32768, d = 7168 (896 vectors = 7 segments): 6.3 TB/s against
//   5.4 TB/s with the token index fastest and 256-thread blocks (whose fourth block is half empty).
// combine: the same numbering and block size (6.5 TB/s against 6.1-6.3 TB/s with one block per token row).
constexpr int DISPATCH_BLOCK = 128;
constexpr int COMBINE_BLOCK = 128;

template <bool BF16, bool SCALED>
__global__ __launch_bounds__(DISPATCH_BLOCK) void dispatch_rows(const u32x4* __restrict__ x, int T, int row_vecs, int n_seg,
                                                    int k, const int32_t* __restrict__ inv,
                                                    const float* __restrict__ row_scale,
                                                    u32x4* __restrict__ xp) {
  const int t = blockIdx.x / n_seg;
  const int c = (blockIdx.x - t * n_seg) * DISPATCH_BLOCK + threadIdx.x;
  const int32_t* irow = inv + (size_t)t * k;         // uniform address: scalar loads
  int first = -1;
  for (int j = 0; j < k; ++j)
    if (irow[j] >= 0) { first = j; break; }
  if (first < 0 || c >= row_vecs) return;             // token without a local slot: nothing is read
  const u32x4 v = __builtin_nontemporal_load(x + (size_t)t * row_vecs + c);
  for (int j = first; j < k; ++j) {
    const int row = irow[j];
    if (row < 0) continue;
    const float sc = SCALED ? row_scale[(size_t)t * k + j] : 1.0f;
    const u32x4 o = SCALED ? scale_vec<BF16>(v, sc) : v;
    __builtin_nontemporal_store(o, xp + (size_t)row * row_vecs + c);
  }
}

// The plan of a few slots and the move in one launch: a token's block finds the rows of its own slots by counting, over all slots,
// those that come before them in the order (local expert, slot).  The block behind the movers adds the row counts up to offsets.
// Bound by its launch and by the latency of one read of the slots: a lane per own slot, and counts by ballots.
constexpr int FEW_SLOTS = 2048;

template <bool BF16, bool SCALED>
__global__ __launch_bounds__(DISPATCH_BLOCK) void plan_and_dispatch(const u32x4* __restrict__ x, int T, int row_vecs, int n_seg, int k,
                                                                    const int32_t* __restrict__ topk_idx, const float* __restrict__ row_scale,
                                                                    int e_lo, int e_cnt, int cap, int32_t* __restrict__ offsets,
                                                                    int32_t* __restrict__ perm, int32_t* __restrict__ inv,
                                                                    int32_t* __restrict__ status, u32x4* __restrict__ xp) {
  constexpr int WAVES = DISPATCH_BLOCK / WAVE, KEYS = FEW_SLOTS / DISPATCH_BLOCK, BATCH = 4, ELSEWHERE = 0x7FFFFFFF;
  __shared__ int32_t hist[MOE_MAX_LOCAL];
  __shared__ int32_t before[WAVES][MOE_MAX_TOPK];
  const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
  const int n_slots = T * k, t = blockIdx.x / n_seg;
  const auto key_of = [&](int s) {        // place of a slot in the order; beyond all others if its expert is not local
    const int le = topk_idx[s] - e_lo;
    return le >= 0 && le < e_cnt ? le * FEW_SLOTS + s : ELSEWHERE;
  };
  const int seg = blockIdx.x - t * n_seg, c = seg * DISPATCH_BLOCK + tid;
  u32x4 v = {0, 0, 0, 0};
  if (t < T && c < row_vecs) v = __builtin_nontemporal_load(x + (size_t)t * row_vecs + c);
  int key[KEYS];
#pragma unroll
  for (int b = 0; b < KEYS; b += BATCH)
    if (b * DISPATCH_BLOCK < n_slots)     // (uniform)
#pragma unroll
      for (int i = b; i < b + BATCH; ++i) {
        const int s = i * DISPATCH_BLOCK + tid;
        key[i] = s < n_slots ? key_of(s) : ELSEWHERE;
      }
  if (t == T) {
    for (int i = tid; i < e_cnt; i += DISPATCH_BLOCK) hist[i] = 0;
    __syncthreads();
#pragma unroll
    for (int b = 0; b < KEYS; b += BATCH)
      if (b * DISPATCH_BLOCK < n_slots)
#pragma unroll
        for (int i = b; i < b + BATCH; ++i)
          if (key[i] != ELSEWHERE) atomicAdd(&hist[key[i] / FEW_SLOTS], 1);
    __syncthreads();
    if (wave == 0) {
      int sum = 0;
      for (int e0 = 0; e0 < e_cnt; e0 += WAVE) {
        const int n = e0 + lane < e_cnt ? hist[e0 + lane] : 0, incl = wave_scan(n);
        if (e0 + lane < e_cnt) offsets[e0 + lane] = min(sum + incl - n, cap);
        sum += __builtin_amdgcn_readlane(incl, WAVE - 1);
      }
      if (lane == 0) {
        offsets[e_cnt] = min(sum, cap);
        *status = sum > cap ? 1 : 0;
      }
    }
    return;
  }
  const int slot = t * k + lane, own = lane < k ? key_of(slot) : ELSEWHERE;
  const float scale = SCALED && lane < k ? row_scale[slot] : 1.f;
  const unsigned long long locals = __ballot(own != ELSEWHERE);
  int row = 0;                            // of slot `lane`
  for (unsigned long long m = locals; m; m &= m - 1) {
    const int j = __builtin_ctzll(m), mine = __builtin_amdgcn_readlane(own, j);
    int n = 0;
#pragma unroll
    for (int b = 0; b < KEYS; b += BATCH)
      if (b * DISPATCH_BLOCK < n_slots)
#pragma unroll
        for (int i = b; i < b + BATCH; ++i) n += __popcll(__ballot(key[i] < mine));
    row = lane == j ? n : row;
  }
  if (lane < k) before[wave][lane] = row;
  __syncthreads();
  if (own != ELSEWHERE) {
    row = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) row += before[w][lane];
  }
  if (own == ELSEWHERE || row >= cap) row = -1;
  if (seg == 0 && tid < k) {
    inv[slot] = row;
    if (row >= 0) perm[row] = slot;
  }
  for (unsigned long long m = __ballot(row >= 0); m; m &= m - 1) {
    const int j = __builtin_ctzll(m);
    const u32x4 o = SCALED ? scale_vec<BF16>(v, __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(scale), j))) : v;
    if (c < row_vecs) __builtin_nontemporal_store(o, xp + (size_t)__builtin_amdgcn_readlane(row, j) * row_vecs + c);
  }
}

template <bool BF16>
__device__ __forceinline__ void fma_vec(float* acc, u32x4 v, float w) {
  if (BF16) {
    acc[0] += w * bf16lo(v.x); acc[1] += w * bf16hi(v.x);
    acc[2] += w * bf16lo(v.y); acc[3] += w * bf16hi(v.y);
    acc[4] += w * bf16lo(v.z); acc[5] += w * bf16hi(v.z);
    acc[6] += w * bf16lo(v.w); acc[7] += w * bf16hi(v.w);
  } else {
    acc[0] += w * __uint_as_float(v.x); acc[1] += w * __uint_as_float(v.y);
    acc[2] += w * __uint_as_float(v.z); acc[3] += w * __uint_as_float(v.w);
  }
}

template <bool BF16>
__device__ __forceinline__ u32x4 pack_acc(const float* acc) {
  u32x4 r;
  if (BF16) {
    r.x = pack_bf16x2(acc[0], acc[1]); r.y = pack_bf16x2(acc[2], acc[3]);
    r.z = pack_bf16x2(acc[4], acc[5]); r.w = pack_bf16x2(acc[6], acc[7]);
  } else {
    r.x = __float_as_uint(acc[0]); r.y = __float_as_uint(acc[1]);
    r.z = __float_as_uint(acc[2]); r.w = __float_as_uint(acc[3]);
  }
  return r;
}

template <bool BF16>
__global__ __launch_bounds__(COMBINE_BLOCK) void combine_rows(const u32x4* __restrict__ o, int T, int row_vecs, int n_seg,
                                                   int k, const int32_t* __restrict__ inv,
                                                   const float* __restrict__ topk_w,
                                                   u32x4* __restrict__ y) {
  const int t = blockIdx.x / n_seg;
  const int c = (blockIdx.x - t * n_seg) * COMBINE_BLOCK + threadIdx.x;
  if (c >= row_vecs) return;
  const int32_t* irow = inv + (size_t)t * k;         // uniform address: scalar loads
  float acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.f;
  for (int j = 0; j < k; ++j) {                       // ascending slot j
    const int row = irow[j];
    if (row < 0) continue;
    const float w = topk_w ? topk_w[(size_t)t * k + j] : 1.0f;
    const u32x4 v = __builtin_nontemporal_load(o + (size_t)row * row_vecs + c);
    fma_vec<BF16>(acc, v, w);
  }
  __builtin_nontemporal_store(pack_acc<BF16>(acc), y + (size_t)t * row_vecs + c);
}

}  // namespace

int launch_dispatch_rows(const void* x, int dtype, int T, int d, int k, const int32_t* inv,
                         const float* row_scale, void* xp, hipStream_t s) {
  if (T == 0) return MOE_OK;
  ProfScope prof(MOE_K_DISPATCH, s);
  const int row_vecs = dtype == MOE_BF16 ? d / 8 : d / 4;
  const int n_seg = (row_vecs + DISPATCH_BLOCK - 1) / DISPATCH_BLOCK;
  if ((long long)T * n_seg >= (1ll << 31)) return MOE_EUNSUPPORTED;      // 1-D grid limit (checked by the entry point too)
  dim3 grid((unsigned)(T * n_seg)), block(DISPATCH_BLOCK);
  const u32x4* xs = (const u32x4*)x;
  u32x4* xd = (u32x4*)xp;
  if (dtype == MOE_BF16) {
    if (row_scale) hipLaunchKernelGGL((dispatch_rows<true, true>), grid, block, 0, s, xs, T, row_vecs, n_seg, k, inv, row_scale, xd);
    else hipLaunchKernelGGL((dispatch_rows<true, false>), grid, block, 0, s, xs, T, row_vecs, n_seg, k, inv, row_scale, xd);
  } else {
    if (row_scale) hipLaunchKernelGGL((dispatch_rows<false, true>), grid, block, 0, s, xs, T, row_vecs, n_seg, k, inv, row_scale, xd);
    else hipLaunchKernelGGL((dispatch_rows<false, false>), grid, block, 0, s, xs, T, row_vecs, n_seg, k, inv, row_scale, xd);
  }
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}

// Every block reads all slots: up to 2^20 reads in all.  Plan and move in a captured graph, us, two launches / one (one launch less is 4
// to 5 us of the host's time as well): 4 tokens, k = 8, d = 4096, 16 of 128 experts local 5.5 / 2.7, all local 5.7 / 3.6; 64, 8, 4096, all on
// eight experts 6.2 / 4.4; 724, 2, 1024, 8 of 8 6.4 / 4.8; 128, 8, 7168 (2^20), 64 of 64 8.1 / 7.0; 200, 8, 2048, 256 of 256 8.7 / 7.2.  (Counting
// slot by slot with a reduction each made the local ones of k = 8 slower than two launches: 6.3, 7.1 and 9.2.)  Where the line lies was measured
// with that: forward of 250 tokens (2^21 reads) 166.4 / 166.4; 256, 8, 7168 (2^22) 321 / 325.
bool plan_and_dispatch_fits(int T, int k, int d, int dtype) {
  const long long slots = (long long)T * k, n_seg = ((dtype == MOE_BF16 ? d / 8 : d / 4) + DISPATCH_BLOCK - 1) / DISPATCH_BLOCK;
  return T > 0 && slots <= FEW_SLOTS && T * n_seg * slots <= (1 << 20);
}
int launch_plan_and_dispatch(const void* x, int dtype, int T, int d, int k, const int32_t* topk_idx, const float* row_scale, int e_lo,
                             int e_cnt, int32_t* offsets, int32_t* perm, int32_t* inv, int cap, int32_t* status, void* xp, hipStream_t s) {
  ProfScope prof(MOE_K_DISPATCH, s);
  const int row_vecs = dtype == MOE_BF16 ? d / 8 : d / 4;
  const int n_seg = (row_vecs + DISPATCH_BLOCK - 1) / DISPATCH_BLOCK;
  if ((long long)T * n_seg + 1 >= (1ll << 31)) return MOE_EUNSUPPORTED;
  const dim3 grid((unsigned)(T * n_seg + 1)), block(DISPATCH_BLOCK);
#define PLAN_AND_DISPATCH(BF16, SCALED)                                                                                              \
  hipLaunchKernelGGL((plan_and_dispatch<BF16, SCALED>), grid, block, 0, s, (const u32x4*)x, T, row_vecs, n_seg, k, topk_idx, row_scale, \
                     e_lo, e_cnt, cap, offsets, perm, inv, status, (u32x4*)xp)
  if (dtype == MOE_BF16) {
    if (row_scale) PLAN_AND_DISPATCH(true, true);
    else PLAN_AND_DISPATCH(true, false);
  } else {
    if (row_scale) PLAN_AND_DISPATCH(false, true);
    else PLAN_AND_DISPATCH(false, false);
  }
#undef PLAN_AND_DISPATCH
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}

int launch_combine_rows(const void* o, int dtype, int T, int d, int k, const int32_t* inv,
                        const float* topk_w, void* y, hipStream_t s) {
  if (T == 0) return MOE_OK;
  ProfScope prof(MOE_K_COMBINE, s);
  const int row_vecs = dtype == MOE_BF16 ? d / 8 : d / 4;
  const int n_seg = (row_vecs + COMBINE_BLOCK - 1) / COMBINE_BLOCK;
  if ((long long)T * n_seg >= (1ll << 31)) return MOE_EUNSUPPORTED;      // 1-D grid limit (checked by the entry point too)
  dim3 grid((unsigned)(T * n_seg)), block(COMBINE_BLOCK);
  if (dtype == MOE_BF16)
    hipLaunchKernelGGL((combine_rows<true>), grid, block, 0, s, (const u32x4*)o, T, row_vecs, n_seg, k, inv, topk_w, (u32x4*)y);
  else
    hipLaunchKernelGGL((combine_rows<false>), grid, block, 0, s, (const u32x4*)o, T, row_vecs, n_seg, k, inv, topk_w, (u32x4*)y);
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}
