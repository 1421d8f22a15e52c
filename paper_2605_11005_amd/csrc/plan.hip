// The dispatch plan: a stable counting sort of the flat slots s = t*k + j by local expert.
//
// Three small kernels, no order-dependent atomics, so perm/inv are unique and reproducible:
//   1. plan_hist    -- every wavefront owns CHUNK consecutive slots and writes the histogram
//                      of their local experts to ws_hist[e][chunk] (chunks contiguous per expert,
//                      so that the scan reads coalesced).
//   2. plan_scan    -- one block, one wavefront per expert: an exclusive running sum over the chunks
//                      (-> first row of that expert inside each chunk), then the exclusive
//                      prefix over experts (-> offsets), clamped to cap with a status word.
//   3. plan_scatter -- every wavefront revisits its chunk in slot order; within each group
//                      of 64 slots the rank among equal keys comes from ballots (one per bit of
//                      the key) and a popcount of the lower lanes, and a per-wave LDS counter
//                      carries it forward.
// Up to some ten thousand slots plan_direct does the three steps in one launch.  The smallest batches are planned by the dispatch
// itself (plan_and_dispatch in rowmove.hip).
#include "common.h"
#include "kernels.h"

#include <mutex>

namespace {

constexpr int CHUNK = 512;   // slots per wavefront

__global__ __launch_bounds__(64) void plan_hist(const int32_t* __restrict__ topk_idx, int n_slots, int e_lo,
                                               int e_cnt, int32_t* __restrict__ ws_hist) {
  extern __shared__ int32_t h[];
  const int lane = threadIdx.x;
  for (int i = lane; i < e_cnt; i += WAVE) h[i] = 0;
  __syncthreads();
  const int base = blockIdx.x * CHUNK;
  for (int i = lane; i < CHUNK; i += WAVE) {
    int s = base + i;
    if (s < n_slots) {
      int le = topk_idx[s] - e_lo;
      if (le >= 0 && le < e_cnt) atomicAdd(&h[le], 1);
    }
  }
  __syncthreads();
  for (int i = lane; i < e_cnt; i += WAVE) ws_hist[(size_t)i * gridDim.x + blockIdx.x] = h[i];   // [expert][chunk]
}

// ws_hist[e][c] becomes the first row (before the expert's offset is added) of expert e in chunk c.
// One wavefront per expert: 64 chunks at a time, exclusive scan by lane shuffles, carry across
// groups of 64.
__global__ __launch_bounds__(1024) void plan_scan(int32_t* __restrict__ ws_hist, int n_chunks, int e_cnt, int cap,
                                                 int32_t* __restrict__ offsets, int32_t* __restrict__ status) {
  __shared__ int32_t total[MOE_MAX_LOCAL + 1];
  const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE, n_waves = blockDim.x / WAVE;
  for (int e = wave; e < e_cnt; e += n_waves) {
    int carry = 0;
    // eight groups of 64 chunks per batch: all loads of a batch are issued before the first scan,
    // so a batch costs one memory round trip instead of eight
    for (int b0 = 0; b0 < n_chunks; b0 += 8 * WAVE) {
      int v[8];
#pragma unroll
      for (int g = 0; g < 8; ++g) {
        const int c = b0 + g * WAVE + lane;
        v[g] = c < n_chunks ? ws_hist[(size_t)e * n_chunks + c] : 0;
      }
#pragma unroll
      for (int g = 0; g < 8; ++g) {
        const int c = b0 + g * WAVE + lane;
        int incl = v[g];
#pragma unroll
        for (int off = 1; off < WAVE; off <<= 1) {
          int t = __shfl_up(incl, off, WAVE);
          if (lane >= off) incl += t;
        }
        if (c < n_chunks) ws_hist[(size_t)e * n_chunks + c] = carry + incl - v[g];
        carry += __shfl(incl, WAVE - 1, WAVE);
      }
    }
    if (lane == 0) total[e] = carry;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int run = 0;
    for (int i = 0; i < e_cnt; ++i) {
      int v = total[i];
      total[i] = run;
      run += v;
    }
    total[e_cnt] = run;
    *status = run > cap ? 1 : 0;
  }
  __syncthreads();
  // unclamped expert bases stay in ws (after the chunk table) for the scatter pass
  int32_t* ebase = ws_hist + (size_t)n_chunks * e_cnt;
  for (int i = threadIdx.x; i <= e_cnt; i += blockDim.x) {
    int v = total[i];
    ebase[i] = v;
    offsets[i] = v < cap ? v : cap;
  }
}

// Lanes of the wavefront that hold the same key (key < 2^bits; lanes with key < 0 are in nobody's set): one ballot per bit.
// The group's rank and size come from it without a loop over the distinct keys, of which a group of 64 slots can hold 64
// (3000 slots over 16 experts: scatter 17.2 -> 5 us).
__device__ __forceinline__ unsigned long long same_key(int key, int bits) {
  unsigned long long m = __ballot(key >= 0);
  for (int b = 0; b < bits; ++b) {
    const unsigned long long on = __ballot((key >> b) & 1);
    m &= (key >> b) & 1 ? on : ~on;
  }
  return m;
}

// Rows of the 64 slots s0 .. s0 + 63 (run[e]: next row of expert e for this wavefront, in LDS; carried forward).
// Called by whole wavefronts; LDS serves a wavefront's accesses in order.
__device__ __forceinline__ void scatter_group(int s, int le, int bits, int lane, int n_slots, int cap, volatile int32_t* run,
                                              int32_t* __restrict__ perm, int32_t* __restrict__ inv) {
  const unsigned long long same = same_key(le, bits);
  const int rank = __popcll(same & ((1ull << lane) - 1ull));
  const int first = le >= 0 ? run[le] : 0;
  __builtin_amdgcn_wave_barrier();
  if (le >= 0 && rank == 0) run[le] = first + __popcll(same);
  __builtin_amdgcn_wave_barrier();
  if (s < n_slots) {
    int row = le >= 0 ? first + rank : -1;
    if (row >= cap) row = -1;                        // dropped: caller's cap was too small
    inv[s] = row;
    if (row >= 0) perm[row] = s;
  }
}

__device__ __forceinline__ int local_expert(const int32_t* __restrict__ topk_idx, int s, int n_slots, int e_lo, int e_cnt) {
  if (s >= n_slots) return -1;
  const int le = topk_idx[s] - e_lo;
  return le >= 0 && le < e_cnt ? le : -1;
}

__global__ __launch_bounds__(64) void plan_scatter(const int32_t* __restrict__ topk_idx, int n_slots, int e_lo,
                                                  int e_cnt, int bits, int cap, const int32_t* __restrict__ ws_hist,
                                                  int n_chunks, int32_t* __restrict__ perm,
                                                  int32_t* __restrict__ inv) {
  extern __shared__ int32_t run[];
  const int lane = threadIdx.x;
  const int32_t* ebase = ws_hist + (size_t)n_chunks * e_cnt;
  for (int i = lane; i < e_cnt; i += WAVE) run[i] = ebase[i] + ws_hist[(size_t)i * n_chunks + blockIdx.x];
  const int base = blockIdx.x * CHUNK;
  int le[CHUNK / WAVE];
#pragma unroll
  for (int g = 0; g < CHUNK / WAVE; ++g) le[g] = local_expert(topk_idx, base + g * WAVE + lane, n_slots, e_lo, e_cnt);
  __syncthreads();
#pragma unroll
  for (int g = 0; g < CHUNK / WAVE; ++g) scatter_group(base + g * WAVE + lane, le[g], bits, lane, n_slots, cap, run, perm, inv);
}

// All three steps in one launch, for a few ten thousand slots (direct_slots()): block b owns the DIRECT_CHUNK slots from b * DIRECT_CHUNK on, one group
// of 64 per wavefront, and counts the experts of all slots by itself.  Additions to one word wait for each other, and one expert may
// hold most of the slots, so lanes add to `copies` tables in turn (direct_copies()).
// LDS: hist[DIRECT_WAVES][e_cnt] (of the own groups; becomes each wavefront's next row per expert), before[copies][pitch] (slots of the
// blocks before this one), total[copies][pitch] (the other slots; the first copy becomes the first row per expert).
constexpr int DIRECT_WAVES = 16, DIRECT_CHUNK = DIRECT_WAVES * WAVE;
constexpr int DIRECT_MAX_LOCAL = 900;      // the tables fit the 64 KB of LDS that need no opt-in

__global__ __launch_bounds__(DIRECT_CHUNK) void plan_direct(const int32_t* __restrict__ topk_idx, int n_slots, int e_lo, int e_cnt, int bits,
                                                           int copies, int cap, int32_t* __restrict__ offsets,
                                                           int32_t* __restrict__ perm, int32_t* __restrict__ inv,
                                                           int32_t* __restrict__ status) {
  extern __shared__ int32_t hist[];
  const int pitch = e_cnt | 1;                       // odd: an expert's copies are on different banks
  int32_t* const before = hist + DIRECT_WAVES * e_cnt;
  int32_t* const total = before + copies * pitch;
  const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
  const int n_groups = (n_slots + WAVE - 1) / WAVE, first = blockIdx.x * DIRECT_WAVES, own = (first + wave) * WAVE + lane;
  int32_t* const mine = hist + wave * e_cnt;
  const int le_own = local_expert(topk_idx, own, n_slots, e_lo, e_cnt);
  for (int i = tid; i < DIRECT_WAVES * e_cnt + 2 * copies * pitch; i += DIRECT_CHUNK) hist[i] = 0;
  const unsigned long long same = same_key(le_own, bits);
  const int rank = __popcll(same & ((1ull << lane) - 1ull));
  __syncthreads();
  if (le_own >= 0 && rank == 0) mine[le_own] = __popcll(same);
  const int copy = (lane & (copies - 1)) * pitch;
  // eight groups at a time: one memory round trip for all of them
  for (int g0 = wave; g0 < n_groups; g0 += 8 * DIRECT_WAVES) {
    int le[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) le[i] = local_expert(topk_idx, (g0 + i * DIRECT_WAVES) * WAVE + lane, n_slots, e_lo, e_cnt);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (le[i] >= 0) atomicAdd((g0 + i * DIRECT_WAVES < first ? before : total) + copy + le[i], 1);
  }
  __syncthreads();
  if (tid < e_cnt) {                                 // e_cnt <= 900 < threads of the block
    int run = 0, rest = 0;
#pragma unroll 8
    for (int c = 0; c < copies; ++c) {
      run += before[c * pitch + tid];
      rest += total[c * pitch + tid];
    }
    total[tid] = run + rest;
#pragma unroll
    for (int w = 0; w < DIRECT_WAVES; ++w) {
      const int v = hist[w * e_cnt + tid];
      hist[w * e_cnt + tid] = run;
      run += v;
    }
  }
  __syncthreads();
  if (wave == 0) {                                   // exclusive scan over the experts, 64 at a time
    int carry = 0;
    for (int e0 = 0; e0 < e_cnt; e0 += WAVE) {
      const int v = e0 + lane < e_cnt ? total[e0 + lane] : 0, start = carry + wave_scan(v) - v;
      if (e0 + lane < e_cnt) total[e0 + lane] = start;
      if (blockIdx.x == 0 && e0 + lane < e_cnt) offsets[e0 + lane] = min(start, cap);
      carry = __builtin_amdgcn_readlane(start + v, WAVE - 1);
    }
    if (blockIdx.x == 0 && lane == 0) {
      offsets[e_cnt] = min(carry, cap);
      *status = carry > cap ? 1 : 0;
    }
  }
  __syncthreads();
  if (own >= n_slots) return;
  int row = le_own >= 0 ? mine[le_own] + total[le_own] + rank : -1;
  if (row >= cap) row = -1;                          // dropped: caller's cap was too small
  inv[own] = row;
  if (row >= 0) perm[row] = own;
}

}  // namespace

// ---- plan scratch that lives in the code object, for callers that cannot allocate ---------
// One array per GPU (each device that loads the library holds its own copy at its own address
// until the process ends).  Host code never passes the array's name to a kernel: the name is a
// host-side stand-in, the device address comes from hipGetSymbolAddress, once per device.
static __device__ __align__(256) unsigned char scratch[MOE_STATIC_PLAN_BYTES];

namespace {
std::mutex g_scratch_lock;
void* g_scratch_ptr[64] = {};
}  // namespace

int plan_static_scratch(void** ptr) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MOE_EHIP;
  std::lock_guard<std::mutex> hold(g_scratch_lock);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return MOE_EHIP;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return MOE_OK;
}

// Every block counts all slots, in one round of LDS additions per 1024 of them; the three launches' scan takes a round per 16 experts.
// Plan and move of 16 bytes per row in a captured graph, us, three launches (one block up to 8192 slots) / one launch whose lanes all add
// to one table / now:
//   slots, local experts of E, experts alike         8192, 8 of 8      13.1 / 11.6 / 9.4     16384, 8 of 8  18.6 / 16.8 / 13.0    32768, 16 of 16  20.0 / 20.1 / 16.3
//                                                    16384, 16 of 128  17.0 / 10.4 / 9.9     65536, 64 of 64  28.8 / 23.5 / 21.9  65536, 256 of 256  62.1 / 24.3 / 23.0
//   one expert holding all slots                     2049, 8 of 8      8.9 / 9.8 / 6.7       8192, 8 of 8   18.5 / 22.0 / 9.2     16384, 8 of 8    18.4 / 37.6 / 12.7
//   half of them; a quarter                          32768, 16 of 16   20.0 / 38.4 / 16.4    32768, 32 of 32  21.6 / 23.6 / 14.9
// (Where the lines lie was measured before there were copies: 60000 slots of 8 experts 22.2 in three launches, 37.9 in one.)
static int direct_slots(int e_cnt) {
  return e_cnt > DIRECT_MAX_LOCAL ? -1 : (e_cnt >= 64 ? 65536 : (e_cnt >= 16 ? 32768 : 16384));
}
// 8 / 16 / 32 copies: 16384 slots of 8 experts alike 13.0 / 13.1 / 13.3, on one of them 12.7 / 12.6 / 12.8; the many tables of many experts
// take LDS, and their additions rarely meet.
static int direct_copies(int e_cnt) { return e_cnt <= 128 ? 8 : e_cnt <= 256 ? 4 : 1; }

size_t plan_ws_bytes(int T, int k, int e_cnt) {
  size_t n_slots = (size_t)T * (size_t)k;
  size_t n_chunks = (n_slots + CHUNK - 1) / CHUNK;
  // status word (own 256-byte line) + chunk table + expert bases
  return 256 + (n_chunks * (size_t)e_cnt + (size_t)e_cnt + 1) * sizeof(int32_t);
}

int launch_plan(const int32_t* topk_idx, int T, int k, int e_lo, int e_cnt, int32_t* offsets,
                int32_t* perm, int32_t* inv, int cap, void* ws, int32_t* status_out, hipStream_t s) {
  ProfScope prof(MOE_K_PLAN, s);
  int32_t* status = status_out ? status_out : (int32_t*)ws;
  int32_t* ws_hist = (int32_t*)((char*)ws + 256);
  const long long n_slots = (long long)T * k;
  int bits = 0;                                      // of a local expert's index
  while ((1 << bits) < e_cnt) ++bits;
  if (n_slots <= direct_slots(e_cnt)) {
    const int copies = direct_copies(e_cnt);
    const size_t shm = ((size_t)DIRECT_WAVES * e_cnt + 2 * (size_t)copies * (e_cnt | 1)) * sizeof(int32_t);
    const int blocks = (int)((n_slots + DIRECT_CHUNK - 1) / DIRECT_CHUNK);
    hipLaunchKernelGGL(plan_direct, dim3(blocks > 0 ? blocks : 1), dim3(DIRECT_CHUNK), shm, s, topk_idx, (int)n_slots, e_lo, e_cnt, bits, copies,
                       cap, offsets, perm, inv, status);
    HIP_CHECK_LAUNCH();
    return MOE_OK;
  }
  const int n_chunks = (int)((n_slots + CHUNK - 1) / CHUNK);
  size_t shm = (size_t)(e_cnt > 0 ? e_cnt : 1) * sizeof(int32_t);
  if (n_chunks > 0) {
    hipLaunchKernelGGL(plan_hist, dim3(n_chunks), dim3(64), shm, s, topk_idx, (int)n_slots, e_lo, e_cnt, ws_hist);
    HIP_CHECK_LAUNCH();
  }
  hipLaunchKernelGGL(plan_scan, dim3(1), dim3(1024), 0, s, ws_hist, n_chunks, e_cnt, cap, offsets, status);
  HIP_CHECK_LAUNCH();
  if (n_chunks > 0) {
    hipLaunchKernelGGL(plan_scatter, dim3(n_chunks), dim3(64), shm, s, topk_idx, (int)n_slots, e_lo, e_cnt, bits, cap,
                       ws_hist, n_chunks, perm, inv);
    HIP_CHECK_LAUNCH();
  }
  return MOE_OK;
}
