// bf16 grouped GEMMs for the expert FFNs on gfx950 (CDNA4): MFMA 32x32x16 bf16, fp32 accumulate.
//
// One persistent kernel template covers the six GEMM shapes of the expert layer:
//   UP     h1|h3 = xp [W1|W3]        ragged M, B read transposed, fused SwiGLU epilogue -> a
//   DOWN   o     = a W2              ragged M, B read transposed
//   DA     dA    = d_o W2^T          ragged M, B K-contiguous, fused SwiGLU-backward epilogue
//   DX     dxp   = dH1 W1^T + dH3 W3^T   ragged M, K = 2f in two segments
//   WG     dW2   = a^T d_o           ragged K (the expert's rows), both operands read transposed
//   WGD    dW1|dW3 = xp^T [dH1|dH3]  ragged K, two outputs sharing the A operand
//
// Tiling: 256x256 block tile, 32-deep k-tiles, 256 threads = 4 wavefronts in a 2x2 grid,
// 128x128 per wavefront = 4x4 MFMA blocks (256 accumulator registers), one wavefront per SIMD.
//
// Data path: global memory -> LDS directly (global_load_lds_dwordx4, 16 bytes per lane, no
// staging registers), through a 128 KB ring (four k-tiles of both operands), so up to three
// k-tiles (96 KB per CU) are in flight while one is being multiplied.  Every load fetches whole
// 128-byte cache lines where the layout allows it: the K-contiguous operand A of the ragged-M
// shapes is fetched two k-tiles at a time (128 bytes per row) into two double stages, because a
// panel walked in 64-byte pieces crosses the L2-to-CU path twice.  Because a wavefront's 64
// lanes always land on 1 KB of consecutive LDS, bank conflicts are avoided by choosing WHICH
// global chunk each lane fetches (an XOR swizzle of the chunk index), not by padding:
//   K-contiguous A, two k-tiles [256 rows][8 chunks of 8 k]  chunk' = chunk ^ ((row>>1)&7)
//   K-contiguous B, one k-tile  [256 rows][4 chunks of 8 k]  chunk' = chunk ^ ((row>>2)&3)
//   transposed operand tile    2 x [32 k][16 chunks of 8 n]  chunk' = chunk ^ (4*(k&3))
// (LDS has 64 four-byte banks: the 16 lanes served together by a 16-byte read, or the 32 lanes
// of an 8-byte transposing read, must cover 256 distinct bytes modulo 256.)
// Operands whose contraction index is not the contiguous one in memory (the weights in the
// forward pass, both operands of the weight gradients) are kept in their memory layout in
// LDS and transposed on the way to registers by ds_read_b64_tr_b16.
// Per k-tile each wavefront runs two k-steps of 16 MFMAs; the fragments of the next k-step
// are fetched while the current one multiplies, and there is one workgroup barrier per k-tile.
// Workgroups are persistent and walk a device-built tile list (row counts never visit the
// host); the list is ordered so that the tiles resident on one XCD share operand panels.  In the
// ragged-M shapes a second list of 128x128 tiles (quarter tiles) follows where that ends sooner.
#include "few_rows.h"
#include "kernels.h"

namespace {

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
// 16-byte store of a finished output vector.  The epilogues' bf16 outputs stream out once (2-8 GB per step) and
// are next read by another kernel: a nontemporal store keeps them from displacing operand panels in the caches
// (measured: -0.3 % at the DeepSeek-V3-like share, -0.5 % at the Mixtral-like layer over the six GEMMs).
__device__ __forceinline__ void store16(void* ptr, uint4 v) {
  __builtin_nontemporal_store(__builtin_bit_cast(u32x4_t, v), reinterpret_cast<u32x4_t*>(ptr));
}

// 16 bytes that nothing else in the launch reads (h1 and h3 in dA's epilogue, old gradients): likewise.  Qwen-like share 855 -> 848 us
// per training step, GPT-OSS share of 9001 tokens that adds to its gradients 2034 -> 2016, larger shares unchanged.
__device__ __forceinline__ uint4 load16_once(const void* ptr) {
  return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(ptr)));
}

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int BM = 256, BN = 256, BK = 32;
constexpr int QT = 128, QK = 64;        // quarter tiles
constexpr int NT = 256;                 // threads
constexpr int NSTAGE = 4;
constexpr int OPER_BYTES = 256 * BK * 2;           // 16384: one operand tile
constexpr int STAGE_BYTES = 2 * OPER_BYTES;        // 32768
constexpr int TILE_LDS = NSTAGE * STAGE_BYTES;     // 131072
// Epilogue staging, outside the tile ring: one private slab per wavefront, fp32.
//   single-output tiles: 16 rows x 64 columns, pitch 68 floats; dual tiles: 8 rows x 128 columns, pitch 132
constexpr int SPITCH = 68, DPITCH = 132;
constexpr int STAGING_WAVE_BYTES = 16 * SPITCH * 4;   // 4352 >= 8 * DPITCH * 4 = 4224
static_assert(8 * DPITCH * 4 <= STAGING_WAVE_BYTES, "dual slab must fit");
// scheduler tables after the ring: tile_start[L+1], offs[L+1], split[L+1] (int32), order[L] (uint16), ticket
constexpr int SCHED_BYTES = 3 * (MOE_MAX_LOCAL + 1) * 4 + MOE_MAX_LOCAL * 2 + 16;
constexpr int STAGING_OFF = (TILE_LDS + SCHED_BYTES + 15) & ~15;
constexpr int SMEM_BYTES = STAGING_OFF + 4 * STAGING_WAVE_BYTES;
static_assert(SMEM_BYTES <= 160 * 1024, "one workgroup per CU: 160 KB of LDS");

enum { UP = 0, DOWN = 1, DA = 2, DX = 3, WG = 4, WGD = 5,
       // the trainable router reuses the same machinery on one full-height "expert":
       RL = 6,    // logits = x Wr            ragged-M shape, B read transposed, fp32 output
       RW = 7,    // dWr partials = x^T dl    ragged-K shape over fixed chunks of the tokens, fp32 output
       RX = 8 };  // dx (+)= dl Wr^T          ragged-M shape, B K-contiguous, optional bf16 accumulate

struct GArgs {
  const bf16_t* A0; const bf16_t* A1;     // A sources (A1: second K segment of DX)
  const bf16_t* B0; const bf16_t* B1;     // B sources (B1: second half of a dual tile / second K segment)
  long lda, ldb;                          // leading dimensions (elements)
  long b_es;                              // expert stride of B (elements); 0 for row-indexed B
  bf16_t* C0; bf16_t* C1; bf16_t* C2;     // outputs
  long ldc, c_es;
  const bf16_t* H1; const bf16_t* H3;     // DA epilogue inputs
  float* F0;                              // fp32 output (RL, RW)
  const int32_t* off;                     // row offsets; NULL: segment e = [min(e*chunk, rows), min((e+1)*chunk, rows))
  int rows, chunk;
  // Weight gradients of experts with far more rows than the average are cut along the rows into
  // up to split_budget pieces in total, whose fp32 partial tiles go to P0 (piece s at
  // P0 + s * p_stride; the second output of a dual tile at + M*N) and are added up, in piece
  // order, by wgrad_reduce.  plan[e] = (first piece << 8) | pieces  (pieces == 1: not cut).
  float* P0;
  long p_stride;
  int split_budget;
  int32_t* plan;
  int32_t* sched;                         // 8 zeroed ticket counters (one per XCD); ragged-M shapes of the experts: 8 more for the quarter tiles
  int e_cnt;
  int M;                                  // WG/WGD: rows of the output (d or f)
  int N;                                  // output columns (per half for dual tiles)
  int K;                                  // contraction length per segment (ragged-M modes)
  // RL only: the contraction is cut into ksplit ranges of K columns each (the last one may be
  // shorter; k_total columns in all); range j writes its fp32 tile to F0 + j * c_es and a
  // separate pass adds the ranges up.  0 or 1: not cut.
  int ksplit, k_total;
  int accumulate;
  int save_h;
  int pair_first;                         // another GEMM follows in this launch and fills the last round
  int cached;                             // UP, DOWN: cached_experts
};

template <int MODE> struct Traits {
  static constexpr bool A_TRANS = MODE == WG || MODE == WGD || MODE == RW;
  static constexpr bool B_TRANS = MODE == UP || MODE == DOWN || MODE == WG || MODE == WGD || MODE == RL || MODE == RW;
  static constexpr bool DUAL = MODE == UP || MODE == WGD;
  static constexpr bool RAGGED_K = MODE == WG || MODE == WGD || MODE == RW;
  static constexpr int BN_EFF = DUAL ? BN / 2 : BN;   // output columns covered per tile
};

// ---- K-contiguous operand B (source rows are tile rows; a k-tile is 64 contiguous bytes) -
// Wavefront w issues 4 loads per k-tile; load j covers LDS chunks [(4w+j)*64, +64):
// row = 16*(4w+j) + lane/4, LDS slot = lane%4, logical chunk = slot ^ ((row>>2)&3).
// Rows past the valid range re-read the last valid row (their products land in output rows
// or columns that the epilogue never stores).
struct KcIssue {
  const bf16_t* base;      // wave-uniform: first row of the tile
  uint32_t voff[4];        // byte offset of this lane's chunk in load j
  __device__ __forceinline__ void setup(const bf16_t* base_, long ld, int rows_valid, int wave, int lane) {
    base = base_;
    const int c = (lane & 3) ^ ((lane >> 4) & 3);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int r = 16 * (4 * wave + j) + (lane >> 2);
      if (r > rows_valid - 1) r = rows_valid - 1;
      voff[j] = (uint32_t)(r * ld * 2 + c * 16);
    }
  }
  template <bool STREAM>
  __device__ __forceinline__ void issue1(int j, uint32_t oper_lds, int wave, long kofs) const {
    lds_load16<STREAM>(base + kofs, voff[j], oper_lds + (4 * wave + j) * 1024);
  }
};

// ---- K-contiguous operand A of the ragged-M shapes, fetched two k-tiles at a time ----------
// A 64-byte piece is half a cache line, and walking a panel in such pieces moves every line
// from L2 to the CU twice (a load stream of 64-byte pieces sustains half the rate of one of
// 128-byte pieces).  So operand A lives in two double stages of [256 rows][128 bytes] = k-tiles
// 2p and 2p+1 of pair p, filled by 8 loads per wavefront that each fetch whole lines:
// load q covers LDS chunks [(8w+q)*64, +64): row = 8*(8w+q) + lane/8, LDS slot = lane%8,
// logical chunk = slot ^ ((row>>1)&7)  (chunks 0..3: k-tile 2p, 4..7: k-tile 2p+1).
struct KcPairIssue {
  const bf16_t* base;      // wave-uniform: first row of the tile
  uint32_t voff[8];        // byte offset of this lane's chunk in load q
  __device__ __forceinline__ void setup(const bf16_t* base_, long ld, int rows_valid, int wave, int lane) {
    base = base_;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int rl = 8 * (8 * wave + q) + (lane >> 3);
      const int c = (lane & 7) ^ ((rl >> 1) & 7);
      const int r = rl > rows_valid - 1 ? rows_valid - 1 : rl;
      voff[q] = (uint32_t)(r * ld * 2 + c * 16);
    }
  }
  __device__ __forceinline__ void issue1(int q, uint32_t dstage_lds, int wave, long kofs) const {
    lds_load16(base + kofs, voff[q], dstage_lds + (8 * wave + q) * 1024);
  }
};

// ---- transposed operand (source is [k][n], n contiguous) --------------------------------
// Kept in LDS as two sub-tiles [32 k][128 n] of 8 KB (for a dual tile they come from two
// source matrices).  A tile is 16 loads; load id = 4*wave + j covers sub-tile id/8 and the
// four k rows 4*(id%8) + lane/16; LDS slot = lane%16, logical n chunk = slot ^ (4*(k&3)).
// Columns past n_lim are clamped (garbage output columns, never stored); with CLAMP, source
// rows past the last valid one are clamped (the caller zeroes the matching A fragments).
struct TrIssue {
  const bf16_t* src;       // wave-uniform: column n0 of this wavefront's sub-tile source, row 0
  long ld;
  uint32_t coff;           // byte offset of this lane's column chunk
  // a wavefront's four loads all belong to sub-tile wave/2
  __device__ __forceinline__ void setup(const bf16_t* b0, const bf16_t* b1, bool dual, long ld_, int n0, int n_lim,
                                        int wave, int lane) {
    ld = ld_;
    const int sub = wave >> 1;
    const int nc = (lane & 15) ^ (4 * (lane >> 4));
    src = (dual && sub) ? b1 : b0;
    int n = n0 + (dual ? 0 : sub * 128) + nc * 8;
    if (n > n_lim - 8) n = n_lim - 8;
    coff = (uint32_t)(n * 2);
  }
  // load j of the k-tile whose first source row is k0 (rows above k_last_rel clamped if CLAMP)
  template <bool CLAMP, bool STREAM = false>
  __device__ __forceinline__ void issue1(int j, uint32_t oper_lds, int wave, int lane, long k0, int k_last_rel) const {
    const int id = 4 * wave + j;
    int kr = 4 * (id & 7) + (lane >> 4);
    if (CLAMP && kr > k_last_rel) kr = k_last_rel;
    lds_load16<STREAM>(src + k0 * ld, (uint32_t)(kr * ld * 2) + coff, oper_lds + id * 1024);
  }
};

template <int V> struct IntC { static constexpr int value = V; };

// Fragment addressing.  MFMA 32x32x16 operand: lane l holds row (l&31), k = 8*(l>>5) + 0..7.
// K-contiguous tile: one 16-byte read.  byte offset of (row, k-step s) = row*64 + ((2s + (l>>5)) ^ ((row>>2)&3))*16
// (k-step 1 is k-step 0 with bit 5 flipped: the swizzle is an XOR, not an addition)
__device__ __forceinline__ int kc_frag_off(int row, int lane, int s) {
  return row * 64 + (((2 * s + (lane >> 5)) ^ ((row >> 2) & 3)) << 4);
}
// Double stage of operand A: byte offset of (row, k-tile parity h, k-step s) =
// row*128 + ((4h + 2s + (l>>5)) ^ ((row>>1)&7))*16; h and s enter as XORs of 64 and 32.
__device__ __forceinline__ int kcp_frag_off(int row, int lane) {
  return row * 128 + (((lane >> 5) ^ ((row >> 1) & 7)) << 4);
}
// Transposed tile: two 8-byte transposing reads (k 0..3 and 4..7 of the lane's group).  Within
// each group of 16 lanes, lane i supplies the address of T[kb + i/4][nb16 + 4*(i%4) ..+3] and
// receives T[kb + 0..3][nb16 + i].  Offset for k-step 0, first read; add s*4096 + t*1024.
__device__ __forceinline__ int tr_frag_off(int nb, int lane) {
  const int i = lane & 15, g = lane >> 4;
  const int k = 8 * (g >> 1) + (i >> 2);
  const int n = nb + 16 * (g & 1) + 4 * (i & 3);
  const int sub = n >> 7, nl = n & 127;
  return sub * 8192 + k * 256 + (((nl >> 3) ^ (4 * (k & 3))) << 4) + ((n & 4) << 1);
}

__device__ __forceinline__ bf16x8 lds_frag_kc(const char* p) { return *reinterpret_cast<const bf16x8*>(p); }
__device__ __forceinline__ bf16x8 lds_frag_tr(const char* p) {
  s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p));
  s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p + 1024));
  s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, v);
}

extern __shared__ __align__(16) char smem[];

// Dynamic, XCD-aware tile scheduler.  A list of `total` tiles is cut into chunks of 32 consecutive ones, chunk c belongs to XCD
// c mod 8 (workgroup b runs on XCD b mod 8), whose workgroups draw tiles from it in order through one atomic counter per XCD.
// take_ticket takes the ticket waiting in next_q[0], drawn from `queue`, and returns its tile, or -1 when the list is finished.
// A workgroup whose queue has run dry draws from the next XCD's queue that still has tiles.
// first: the tickets of every queue below it are not drawn: the workgroups of a launch's first GEMM begin with one each (256
// atomics at a time take 1.7 us on average, the last of them 3).
// spread: what is left after whole rounds of eight chunks is cut into eight equal ones.  A list shorter than the chip would
// otherwise sit on a few XCDs, each of which reads memory at an eighth of the chip's rate (d = f = 4096, 4 experts of 250 rows: the
// down projection's 64 tiles on two XCDs take 97 us, on eight 74).  Not where the tiles differ in length (ragged K): there a
// last round of short tiles in every queue keeps workgroups from the long ones that another queue still holds, and for the same
// reason not in the dA that shares a launch with dW2 (116 us for 126 at 5538 rows, d = 2048, f = 1408, 8 experts).  The dX that shares
// one with dW1|dW3 gains 1 % on average over 150 cases (5 shapes, 1 to 3 rounds; -6 to +3 %), but rows by 1/r that leave 8 or 16
// tiles beyond a round take 232 us for 215 (8000 rows, d = 2048, f = 1408, 8 experts) or 480 for 457 (16400 rows, d = 1024, f =
// 3584); spreading more than 16 or 64 tiles only, or lists of less than one or four rounds only, was no better on the whole.
template <bool SPREAD>
__device__ __forceinline__ int take_ticket(int32_t* counters, int n_queues, int& queue, int total, int32_t* next_q, int wave, int lane,
                                           int first, bool spread = SPREAD) {
  const int rounds = total / (32 * n_queues), rest = total - rounds * 32 * n_queues;
  const int share = SPREAD && spread ? (rest + n_queues - 1) / n_queues : 32;
  while (true) {
    // (the slot is next written after a whole k loop of barriers)
    const int q = __builtin_amdgcn_readfirstlane(next_q[0]), i = q - 32 * rounds;
    const int L = !SPREAD || i < 0 ? 32 * (n_queues * (q >> 5) + queue) + (q & 31)
                                   : (i < share && queue * share + i < rest ? rounds * 32 * n_queues + queue * share + i : total);
    if (L < total) return L;
    // Tickets only grow, so this queue is finished, and so is every queue whose counter has passed
    // its last ticket.  All counters are looked at in one round trip (an atomic add of zero, one lane
    // per queue): when none is open the workgroup is done; otherwise it draws from the first open
    // queue after its own (work stealing at the tail of the schedule) and, should others have emptied
    // that queue in between, looks again.  Every failed draw means that others took tiles meanwhile,
    // so the loop ends when the list does.
    __syncthreads();                         // everyone has read the ticket before it is replaced
    if (wave == 0) {
      int open = 0;
      if (lane < n_queues) open = first + atomicAdd(counters + lane, 0) < 32 * rounds + max(0, min(share, rest - lane * share));
      const unsigned all = (1u << n_queues) - 1u;
      const unsigned m = (unsigned)__ballot(open) & all;
      if (lane == 0) {
        if (m == 0) {
          next_q[0] = -1;
        } else {
          const unsigned rot = ((m >> (queue + 1)) | (m << (n_queues - queue - 1))) & all;
          const int pick = (queue + 1 + __builtin_ctz(rot)) % n_queues;
          next_q[1] = pick;
          next_q[0] = first + atomicAdd(counters + pick, 1);
        }
      }
    }
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(next_q[0]) < 0) return -1;
    queue = __builtin_amdgcn_readfirstlane(next_q[1]);
  }
}

// Time in us until n_big 256x256 tiles and then n_quarter quarter tiles are done.  active_big, active_quarter: experts whose
// weights either kind reads (one with both is read twice); rows: of all experts, most: of the heaviest.  A quarter tile moves half
// of a 256x256 tile's bytes to the CU for a quarter of its work, and both are bound by that path (about 70 GB/s per CU where the
// panels are shared): 19 us for 47 at a contraction of 2048.  The constants are fitted to the four GEMMs alone over 76 cases
// (eight shapes, 500 to 40000 rows: even, 1/r, half of them on one expert), each of the four plans forced.  Over 297 others (nine
// shapes, 40 to 2500 rows per expert, the same three ways) the plan taken is the best one or within 2 % of it in 86 to 88 % of the
// cases of each GEMM, 0.7 to 0.9 % above it on average and at worst 13 (UP), 14 (DOWN), 17 (DA) and 11 % (DX).  Against 256x256
// tiles only it saves 3, 10, 13 and 16 % on average; 21 of the 1188 cases lose more than 3 %, at worst 8, 7, 17 and 11 % (DA, d = 4096,
// f = 14336, 4 experts of 290 rows: 202 us, as plan 1 237).  Other constants or margins that do better on one half of the cases do
// worse on the other.  The set-up takes 1.4 us longer for it (4100 cycles for 900: most of it fetching the instructions).
template <int MODE>
__device__ __forceinline__ float plan_price(const GArgs& p, int n_big, int n_quarter, int active_big, int active_quarter, int n_quarters_n,
                                            int rows, int most, bool tails) {
  const float k = (float)(MODE == DX ? 2 * p.K : p.K);
  const float alone = (float)(active_quarter * n_quarters_n) / fmaxf((float)n_quarter, 1.f);      // 1 / row tiles that share a weight panel
  const float big = MODE == DA ? 0.024f * k + 12.f : 0.0215f * k + 3.f;
  const float quarter = MODE == DA ? (0.008f + 0.0025f * alone) * k + 6.f : (0.0073f + 0.0025f * alone) * k + 4.5f;
  // the weights at the rate that either kind streams them, MB per us (UP's quarters read 128 bytes of a row, DA's and DX's
  // 256x256 tiles 64)
  constexpr float RATE_BIG = MODE == UP || MODE == DOWN ? 5.6f : 5.1f, RATE_QUARTER = MODE == UP ? 4.8f : 5.8f;
  const float weights = k * (float)p.N * (MODE == UP ? 4e-6f : 2e-6f) * ((float)active_big / RATE_BIG + (float)active_quarter / RATE_QUARTER);
  const int grid = gridDim.x, full = n_big / grid, rest = n_big - full * grid;
  const float per_cu = 1.f / (float)grid;
  // row tiles of which half is empty share no weight panel when they are quarters: their price is the least certain (without this
  // the plan taken for UP is 1.3 % above the best on average instead of 0.9, and 22 cases of 297 lose more than 3 % instead of 10)
  const float doubt = tails && n_big > 0 ? 1.05f : 1.f;
  // The weight gradient that follows in this launch fills the last round: all tiles of one kind.  tile and start are the weight
  // gradients' time per row and tile, in us.  Over 90 pairs of each kind (5 shapes, 240 to 3000 rows per expert, even and 1/r) dA|dW2
  // takes 0.93 to 1.07 times, 1.013 on average, and dX|dW1|dW3 0.86 to 1.08 times, 0.99 on average, what 256x256 tiles alone took.
  if (p.pair_first) {
    const float tile = 0.027f, start = 6.f;
    const float n_second = (float)(((p.N + BM - 1) / BM) * ((p.K + (MODE == DX ? 127 : 255)) / (MODE == DX ? 128 : 256)));
    const float second = n_second * (tile * (float)rows + start * (float)p.e_cnt) * per_cu, longest = tile * (float)most + start;
    if (n_big == 0) return fmaxf(quarter * ceilf((float)n_quarter * per_cu), weights) + fmaxf(second, longest);
    if (n_quarter > 0) return 1e30f;
    return fmaxf(fmaxf((float)(full + (rest ? 1 : 0)) * big, longest), fmaxf((float)n_big * big * per_cu, weights) + second);
  }
  float t = (float)(full + (rest ? 1 : 0)) * big;
  if (n_quarter) t = fmaxf(t, (float)full * big + (n_big ? 3.f : 0.f) + quarter * ceilf(((float)n_quarter + (float)rest * (big / quarter)) * per_cu));
  return doubt * fmaxf(t, weights);
}

// Position of tile L in an ascending table of first tiles [0, n]: usually the last one's or the one after it (tickets of a
// queue ascend), otherwise a binary search.
__device__ __forceinline__ int find_position(const int32_t* start, int n, int L, int hint) {
  int a = hint;
  const int t0 = start[a], t1 = start[a + 1], t2 = start[min(a + 2, n)];
  if (L >= t1 && L < t2) a = a + 1;
  else if (L < t0 || L >= t1) {
    a = 0;
    int c = n;
    while (c - a > 1) {
      int mid = (a + c) >> 1;
      if (start[mid] <= L) a = mid; else c = mid;
    }
  }
  return __builtin_amdgcn_readfirstlane(a);
}

// Position of lane `lane` when the lanes are listed by descending v, ties by lane (whole wavefronts; lanes n .. 63 all hold the same
// v, which is lower than the others').
__device__ __forceinline__ int descending_rank(int v, int n, int lane) {
  int rank = 0;
  for (int first = 0; first < n; first += 8)
#pragma unroll
    for (int o = 0; o < 8; ++o) {
      const int v2 = __builtin_amdgcn_readlane(v, first + o);
      rank += (v2 > v || (v2 == v && first + o < lane)) ? 1 : 0;
    }
  return rank;
}

// ---- what an epilogue does with eight finished columns of a row
__device__ __forceinline__ uint4 pack8(const float* x) {
  return make_uint4(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]), pack_bf16x2(x[6], x[7]));
}
__device__ __forceinline__ void add8(float* x, uint4 old) {
  const uint32_t u[4] = {old.x, old.y, old.z, old.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) { x[2 * i] += bf16lo(u[i]); x[2 * i + 1] += bf16hi(u[i]); }
}
// UP: h1, h3 and a = silu(h1) h3
__device__ __forceinline__ void finish_up(const GArgs& p, size_t idx, const float* x1, const float* x3) {
  float a[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = silu_f(x1[i]) * x3[i];
  if (p.save_h) {
    store16(p.C0 + idx, pack8(x1));
    store16(p.C1 + idx, pack8(x3));
  }
  store16(p.C2 + idx, pack8(a));
}
// DA: a, dH1, dH3 from x = dA and the stored h1, h3
__device__ __forceinline__ void finish_da(const GArgs& p, size_t idx, const float* x, uint4 q1, uint4 q3) {
  const uint32_t u1[4] = {q1.x, q1.y, q1.z, q1.w}, u3[4] = {q3.x, q3.y, q3.z, q3.w};
  float av[8], d1[8], d3[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float z = (i & 1) ? bf16hi(u1[i >> 1]) : bf16lo(u1[i >> 1]);
    const float gv = (i & 1) ? bf16hi(u3[i >> 1]) : bf16lo(u3[i >> 1]);
    float ds;
    const float sl = silu_grad_f(z, &ds);
    av[i] = sl * gv;
    d1[i] = x[i] * gv * ds;
    d3[i] = x[i] * sl;
  }
  if (p.C0) store16(p.C0 + idx, pack8(av));      // not stored when the forward's copy is at hand
  store16(p.C1 + idx, pack8(d1));
  store16(p.C2 + idx, pack8(d3));
}


// ---- quarter tiles: 128x128 (a dual tile: 64 columns of either output) --------------------------------------------------
// What is left of a GEMM when the 256x256 tiles no longer fill a round of the chip, and the row tiles of which half is empty, is
// multiplied in quarters.  The four wavefronts hold 64x64 each; a k-tile is 64 deep, so that every load fetches whole cache
// lines of either operand, and four of them (128 KB) make the ring.  Every output is the same chain of sums as in a 256x256
// tile, bit for bit.
//   K-contiguous operand   [128 rows][8 chunks of 8 k]       chunk' = chunk ^ ((row>>1)&7)
//   transposed operand     2 x [64 k][8 chunks of 8 n]       chunk' = chunk ^ (4*((k>>1)&1))
constexpr int QOPER_BYTES = QT * QK * 2;
static_assert(NSTAGE * 2 * QOPER_BYTES == TILE_LDS, "the ring holds four k-tiles of quarter tiles");

struct QuarterKc {         // load j of a wavefront: rows 8*(4w+j) + lane/8, whole 128-byte lines
  const bf16_t* base;
  uint32_t voff[4];
  __device__ __forceinline__ void setup(const bf16_t* base_, long ld, int rows_valid, int wave, int lane) {
    base = base_;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int rl = 8 * (4 * wave + j) + (lane >> 3);
      const int c = (lane & 7) ^ ((rl >> 1) & 7);
      voff[j] = (uint32_t)(min(rl, rows_valid - 1) * ld * 2 + c * 16);
    }
  }
  __device__ __forceinline__ void issue1(int j, uint32_t oper_lds, int wave, long kofs) const {
    lds_load16(base + kofs, voff[j], oper_lds + (4 * wave + j) * 1024);
  }
};
struct QuarterTr {         // sub-tile wave/2, load j: k rows 8*(4*(w%2)+j) + lane/8, 64 columns each
  const bf16_t* src;
  long ld;
  uint32_t coff;
  __device__ __forceinline__ void setup(const bf16_t* b0, const bf16_t* b1, bool dual, long ld_, int n0, int n_lim, int wave, int lane) {
    ld = ld_;
    const int sub = wave >> 1, c = (lane & 7) ^ (4 * ((lane >> 4) & 1));
    src = (dual && sub) ? b1 : b0;
    coff = (uint32_t)(2 * min(n0 + (dual ? 0 : sub * 64) + c * 8, n_lim - 8));
  }
  template <bool CLAMP>    // source rows above k_last_rel are clamped (the caller zeroes the matching A fragments)
  __device__ __forceinline__ void issue1(int j, uint32_t oper_lds, int wave, int lane, long k0, int k_last_rel) const {
    int kr = 8 * (4 * (wave & 1) + j) + (lane >> 3);
    if (CLAMP && kr > k_last_rel) kr = k_last_rel;
    lds_load16(src + k0 * ld, (uint32_t)(kr * ld * 2) + coff, oper_lds + (4 * wave + j) * 1024);
  }
};
// transposed sub-tile: byte offset of the first transposing read of 32 columns at nl (0 or 32), k-step 0; add s*2048 + t*512
__device__ __forceinline__ int quarter_tr_off(int sub, int nl, int lane) {
  const int i = lane & 15, g = lane >> 4;
  const int k = 8 * (g >> 1) + (i >> 2);
  const int n = nl + 16 * (g & 1) + 4 * (i & 3);
  return sub * 8192 + k * 128 + (((n >> 3) ^ (4 * ((k >> 1) & 1))) << 4) + ((n & 4) << 1);
}
__device__ __forceinline__ bf16x8 quarter_frag_tr(const char* p) {
  s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p));
  s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p + 512));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// The list of quarter tiles: positions in order[], each with the rows that its 256-row tiles leave.
struct Quarters {
  const int32_t* offs;
  const uint16_t* order;
  const int32_t* tile_start;               // 256x256 tiles before a position
  const int32_t* start;                    // quarter tiles before a position
  int n_tiles_n;                           // column tiles of 256x256
  int total;
  int32_t* next_q;
};

template <int MODE>
__device__ __forceinline__ void quarter_tiles(const GArgs& p, const Quarters& list) {
  using TR = Traits<MODE>;
  static_assert(!TR::RAGGED_K, "");
  constexpr int QN = TR::DUAL ? QT / 2 : QT;             // output columns
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int n_cols = (p.N + QN - 1) / QN;
  const uint32_t smem_base = lds_addr(smem);
  int32_t* const counters = p.sched + 8;
  const int n_queues = (gridDim.x % 8) == 0 ? 8 : 1;
  int queue = blockIdx.x % n_queues;
  int hint = 0;

  int a_off[2], b_off[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = wm * 64 + i * 32 + (lane & 31), col = wn * 64 + i * 32 + (lane & 31);
    a_off[i] = row * 128 + (((lane >> 5) ^ ((row >> 1) & 7)) << 4);
    b_off[i] = QOPER_BYTES + (!TR::B_TRANS ? col * 128 + (((lane >> 5) ^ ((col >> 1) & 7)) << 4)
                                           : TR::DUAL ? quarter_tr_off(i, wn * 32, lane) : quarter_tr_off(wn, i * 32, lane));
  }

  int row0 = 0, row_end = 0, n0 = 0, nk0 = 0, nk = 0;
  QuarterKc ia, ib_kc;
  QuarterTr ib_tr;
  // q = 0..3: operand A of k-tile kt, 4..7: operand B.  kt is clamped to the last one as in the 256x256 tiles.
  auto issue_one = [&](int kt, int q) {
    if (kt > nk - 1) kt = nk - 1;
    const uint32_t st = smem_base + (kt & (NSTAGE - 1)) * (2 * QOPER_BYTES);
    const bool seg1 = MODE == DX && kt >= nk0;
    const long k0 = (long)(seg1 ? kt - nk0 : kt) * QK;
    if (q < 4) ia.issue1(q, st, wave, k0 + (seg1 ? p.A1 - p.A0 : 0));
    else if (TR::B_TRANS) ib_tr.template issue1<false>(q - 4, st + QOPER_BYTES, wave, lane, k0, 0);
    else ib_kc.issue1(q - 4, st + QOPER_BYTES, wave, k0 + (seg1 ? p.B1 - p.B0 : 0));
  };
  auto next_tile = [&]() -> bool {
    const int L = take_ticket<true>(counters, n_queues, queue, list.total, list.next_q, wave, lane, 0);
    if (L < 0) return false;
    const int pos = find_position(list.start, p.e_cnt, L, hint);
    hint = pos;
    const int li = __builtin_amdgcn_readfirstlane(L - list.start[pos]);
    const int e = __builtin_amdgcn_readfirstlane((int)list.order[pos]);
    const int lo = __builtin_amdgcn_readfirstlane(list.offs[e]) +
                   BM * (__builtin_amdgcn_readfirstlane(list.tile_start[pos + 1] - list.tile_start[pos]) / list.n_tiles_n);
    const int hi = __builtin_amdgcn_readfirstlane(list.offs[e + 1]);
    const int m_tiles = (hi - lo + QT - 1) / QT;
    const int band = li / (8 * n_cols), in_band = li - band * 8 * n_cols, band_rows = min(8, m_tiles - band * 8);
    const int nt = in_band / band_rows;
    row0 = lo + (band * 8 + in_band - nt * band_rows) * QT;
    row_end = hi;
    n0 = nt * QN;
    nk0 = p.K / QK;
    nk = MODE == DX ? 2 * nk0 : nk0;
    ia.setup(p.A0 + (size_t)row0 * p.lda, p.lda, hi - row0, wave, lane);
    if (TR::B_TRANS) ib_tr.setup(p.B0 + (size_t)e * p.b_es, p.B1 + (size_t)e * p.b_es, TR::DUAL, p.ldb, n0, p.N, wave, lane);
    else ib_kc.setup(p.B0 + (size_t)e * p.b_es + (size_t)n0 * p.ldb, p.ldb, p.N - n0, wave, lane);
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int q = 0; q < 8; ++q) issue_one(t, q);
#pragma unroll
    for (int q = 0; q < 4; ++q) issue_one(3, q);
    return true;
  };

  if (tid == 0) list.next_q[0] = atomicAdd(counters + queue, 1);
  __syncthreads();
  bool have = next_tile();
  while (have) {
    int my_ticket = 0;
    const int kt_draw = nk > 4 ? nk - 4 : 0;
    // DA: this tile's h1 and h3 (clamped addresses) are here before its k loop ends; 4 slabs of 16 rows, 2 passes of 8
    uint4 pre1[4][2], pre3[4][2];
    const int c8 = lane & 7;
    if (MODE == DA) {
#pragma unroll
      for (int sl = 0; sl < 4; ++sl)
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
          const int grow = min(row0 + wm * 64 + 16 * sl + pass * 8 + (lane >> 3), row_end - 1);
          const int gcol = min(n0 + wn * 64 + c8 * 8, p.N - 8);
          const size_t idx = (size_t)grow * p.ldc + gcol;
          pre1[sl][pass] = load16_once(p.H1 + idx);
          pre3[sl][pass] = load16_once(p.H3 + idx);
        }
    }
    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // Set h holds the fragments of half h of a k-tile (two k-steps of 16).  While a half multiplies, the other half's fragments
    // are read; at the barrier between the halves of k-tile kt all of its fragments are in registers, so its stage is free, and
    // k-tile kt+1 has landed.  The first half issues operand B of k-tile kt+3, the second operand A of kt+4, as in the 256x256
    // tiles: 16 loads may remain at the barrier.
    bf16x8 fa[2][2][2], fb[2][2][2];
    auto frag_op = [&](int h, int kt, int o) {           // o: k-step o/4; A0, B0, B1, A1
      const char* st = smem + (kt & (NSTAGE - 1)) * (2 * QOPER_BYTES);
      const int s = 2 * h + (o >> 2), i = (o & 3) == 1 ? 0 : (o & 3) == 2 ? 1 : (o & 3) / 3;
      if ((o & 3) == 0 || (o & 3) == 3) fa[h][o >> 2][i] = lds_frag_kc(st + (a_off[i] ^ (s * 32)));
      else fb[h][o >> 2][i] = TR::B_TRANS ? quarter_frag_tr(st + b_off[i] + s * 2048) : lds_frag_kc(st + (b_off[i] ^ (s * 32)));
    };
    auto mfma_one = [&](int h, int m) {                  // blocks (0,0), (0,1), (1,1), (1,0) of k-step m/4
      const int i = (m >> 1) & 1, j = i ^ (m & 1);
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[h][m >> 2][i], fb[h][m >> 2][j], acc[i][j], 0, 0, 0);
    };
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    // MV: 32-row blocks of this wavefront that hold valid rows
    auto k_loop = [&](auto mv_tag) {
      constexpr int MV = decltype(mv_tag)::value;
      auto live = [](int o) { return MV == 2 || (MV == 1 && (o & 3) != 3); };
      auto half = [&](int kt, auto h_tag) {
        constexpr int H = decltype(h_tag)::value;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < 8; m += 2) {
          if ((m & 3) < 2 * MV) mfma_one(H, m);
          if (m < 4) {
#pragma unroll
            for (int o = 2 * m; o < 2 * m + 2; ++o)
              if (live(o)) frag_op(1 - H, H ? kt + 1 : kt, o);
          }
          if ((m & 3) < 2 * MV) mfma_one(H, m + 1);
          if (m < 4) {
#pragma unroll
            for (int o = 2 * m + 2; o < 2 * m + 4; ++o)
              if (live(o)) frag_op(1 - H, H ? kt + 1 : kt, o);
          }
          issue_one(H ? kt + 4 : kt + 3, H ? m >> 1 : 4 + (m >> 1));
          __builtin_amdgcn_sched_barrier(0);
        }
      };
#pragma unroll
      for (int o = 0; o < 8; ++o)
        if (live(o)) frag_op(0, 0, o);
      for (int kt = 0; kt < nk; ++kt) {
        if (kt == kt_draw && tid == 0) my_ticket = atomicAdd(counters + queue, 1);
        half(kt, IntC<0>{});
        asm volatile("s_waitcnt vmcnt(16) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        half(kt, IntC<1>{});
      }
    };
    const int rows_left = row_end - (row0 + wm * 64);
    if (rows_left > 32) k_loop(IntC<2>{});
    else if (rows_left > 0) k_loop(IntC<1>{});
    else k_loop(IntC<0>{});
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    if (MODE == DA) {      // these have arrived: the compiler is to wait for them here, not behind the next tile's first loads
#pragma unroll
      for (int sl = 0; sl < 4; ++sl)
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
          u32x4_t u1 = __builtin_bit_cast(u32x4_t, pre1[sl][pass]), u3 = __builtin_bit_cast(u32x4_t, pre3[sl][pass]);
          asm volatile("" : "+v"(u1), "+v"(u3));
          pre1[sl][pass] = __builtin_bit_cast(uint4, u1);
          pre3[sl][pass] = __builtin_bit_cast(uint4, u3);
        }
    }
    if (tid == 0) list.next_q[0] = my_ticket;
    __syncthreads();
    const int ep_row0 = row0 + wm * 64, ep_row_end = row_end, ep_n0 = n0;
    have = next_tile();

    // epilogue: slabs of 16 rows x 64 columns (a dual tile: 32 of either output) through the wavefront's own staging area
    float* stage = reinterpret_cast<float*>(smem + STAGING_OFF) + wave * (STAGING_WAVE_BYTES / 4);
    const int acc_col = lane & 31, acc_rg = lane >> 5;
#pragma unroll
    for (int sl = 0; sl < 4; ++sl) {
      const int mi = sl >> 1, h = sl & 1;
#pragma unroll
      for (int gg = 0; gg < 2; ++gg)
#pragma unroll
        for (int nn = 0; nn < 2; ++nn)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            stage[(8 * gg + 4 * acc_rg + i) * SPITCH + nn * 32 + acc_col] = acc[mi][nn][4 * (2 * h + gg) + i];
      __builtin_amdgcn_wave_barrier();
      float xs[2][8];
#pragma unroll
      for (int pass = 0; pass < 2; ++pass) {             // a dual tile's passes are its two outputs
        const float* sp = TR::DUAL ? stage + (lane >> 2) * SPITCH + pass * 32 + (lane & 3) * 8
                                   : stage + (pass * 8 + (lane >> 3)) * SPITCH + c8 * 8;
#pragma unroll
        for (int i = 0; i < 8; ++i) xs[pass][i] = sp[i];
      }
      __builtin_amdgcn_wave_barrier();
      if (TR::DUAL) {
        const int grow = ep_row0 + 16 * sl + (lane >> 2), gcol = ep_n0 + wn * 32 + (lane & 3) * 8;
        if (grow < ep_row_end && gcol < p.N) finish_up(p, (size_t)grow * p.ldc + gcol, xs[0], xs[1]);
      } else {
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
          const int grow = ep_row0 + 16 * sl + pass * 8 + (lane >> 3), gcol = ep_n0 + wn * 64 + c8 * 8;
          if (grow < ep_row_end && gcol < p.N) {
            const size_t idx = (size_t)grow * p.ldc + gcol;
            if (MODE == DA) finish_da(p, idx, xs[pass], pre1[sl][pass], pre3[sl][pass]);
            else store16(p.C0 + idx, pack8(xs[pass]));
          }
        }
      }
    }
  }
}

// One grouped GEMM from its set-up to its last tile, run by a persistent workgroup.  FIRST: the launch's first one, which all
// workgroups begin together.
template <int MODE, bool FIRST>
__device__ __forceinline__ void gg_body(const GArgs& p) {
  using TR = Traits<MODE>;
  int32_t* tile_start = reinterpret_cast<int32_t*>(smem + TILE_LDS);
  int32_t* offs = tile_start + (MOE_MAX_LOCAL + 1);      // LDS copy of the row offsets
  int32_t* split = offs + (MOE_MAX_LOCAL + 1);           // ragged-K modes: (first piece << 8) | pieces, by expert
  int32_t* q_start = split;                              // ragged-M modes: quarter tiles before a position
  constexpr bool SPLIT = MODE <= DX;                     // the rest of a GEMM may be multiplied in quarter tiles
  uint16_t* order = reinterpret_cast<uint16_t*>(split + MOE_MAX_LOCAL + 1);   // experts by descending row count
  int32_t* next_q = reinterpret_cast<int32_t*>(order + MOE_MAX_LOCAL);    // hand-over slot of the tile scheduler

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int e_cnt = p.e_cnt;

  // ---- tile list.  Experts are taken heaviest first (ties by id), so that the cheap tiles
  // come last and even out the end of the schedule.  position -> expert in order[];
  // tile_start[pos] = number of tiles before that position (ragged-M modes).
  // (RL: the ranges of a cut contraction are listed like further column tiles)
  const int n_tiles_cols = (p.N + TR::BN_EFF - 1) / TR::BN_EFF;
  const int n_tiles_n = MODE == RL && p.ksplit > 1 ? n_tiles_cols * p.ksplit : n_tiles_cols;
  int big;                                 // 256x256 tiles
  int wg_tiles_per_e = 0, wg_mt = 0;
  for (int e = tid; e <= e_cnt; e += NT) {
    const long long cut = (long long)e * p.chunk;
    offs[e] = p.off ? p.off[e] : (int)(cut < p.rows ? cut : p.rows);
  }
  __syncthreads();
  // (up to 64 experts: every wavefront by itself, one expert per lane)
  const bool in_lanes = e_cnt <= WAVE;
  int sorted = 0;                          // rows at position `lane`
  if (in_lanes) {
    const int rows = lane < e_cnt ? offs[lane + 1] - offs[lane] : -1;
    const int rank = descending_rank(rows, e_cnt, lane);
    sorted = __builtin_amdgcn_ds_permute(4 * rank, rows);
    if (wave == 0 && lane < e_cnt) order[rank] = (uint16_t)lane;
  } else {
    for (int e = tid; e < e_cnt; e += NT) {
      const int rows = offs[e + 1] - offs[e];
      int rank = 0;
      for (int o = 0; o < e_cnt; ++o) {
        const int r2 = offs[o + 1] - offs[o];
        rank += (r2 > rows || (r2 == rows && o < e)) ? 1 : 0;
      }
      order[rank] = (uint16_t)e;
    }
  }
  __syncthreads();
  const auto rows_at = [&](int pos) {      // pos: the lane's of the 64 positions at hand
    return pos >= e_cnt ? 0 : (in_lanes ? sorted : offs[order[pos] + 1] - offs[order[pos]]);
  };
  if (TR::RAGGED_K) {
    // Every expert has the same number of output tiles, but a tile's cost is the expert's row
    // count.  An expert whose k loop is longer than a workgroup's fair share of the whole launch
    // (in k-tiles) bounds the kernel from below; it may be cut into pieces of a target length
    // (at least 16 k-tiles) when the time saved exceeds the time to write and re-read the fp32
    // partial tiles (p_stride floats per piece, priced at ~4 TB/s against ~0.85 us per k-tile),
    // heaviest experts first while the budget of partial tiles lasts.
    // No target length is right everywhere: longer pieces end later, shorter ones mean more partial
    // tiles.  So each wavefront prices one plan -- targets of 0.7, 1 and 1.4 fair shares, and no cut --
    // and the cheapest is taken.  A plan's end is the larger of the total work per workgroup and, over
    // the lengths of tiles, of the rounds that the tiles of at least this length need, times the length;
    // in quarter microseconds, 3 per k-tile, 10 per tile and 60 per partial tile (fp32 stores); the
    // reduction adds 12 and its bytes at 1.5 TB/s.  (Fitted to the backward's time under each plan.)  Over 220
    // shares (10 shapes of d, f, experts; 3000 to 48000 rows; even, Zipf, one hot expert, half of them
    // heavier, all rows on one) the whole backward takes 0.96 of its time with pieces of half a share, at
    // most 1.07 of it; always 1.4 shares took 0.98 and up to 1.18.
    wg_mt = (p.M + BM - 1) / BM;
    wg_tiles_per_e = wg_mt * n_tiles_n;
    constexpr int HEAVY = WAVE;                       // experts that may be cut: one per lane
    int32_t* trial = reinterpret_cast<int32_t*>(smem);      // [plan][position]: pieces (the tile ring is still free)
    float* price = reinterpret_cast<float*>(trial + 4 * HEAVY);
    const int grid = gridDim.x;
    const auto k_tiles = [&](int pos) { return (offs[order[pos] + 1] - offs[order[pos]] + BK - 1) / BK; };
    const float inv_grid = 1.f / (float)grid;
    float all = 0.f;                                  // k-tiles of one output tile of every expert
    for (int pos = lane; pos < e_cnt; pos += WAVE) all += (float)((rows_at(pos) + BK - 1) / BK);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) all += __shfl_xor(all, o, WAVE);
    const float share = all * (float)wg_tiles_per_e * inv_grid;
    const auto target = [&](int plan) { return max(16, (int)((plan == 0 ? 0.7f : (plan == 1 ? 1.f : 1.4f)) * share)); };
    const bool may_cut = e_cnt > 0 && p.split_budget >= 2 && __builtin_amdgcn_readfirstlane(k_tiles(0)) > target(0);
    if (may_cut) {
      const int heavy = min(e_cnt, HEAVY);
      volatile int32_t* mine = trial + wave * HEAVY;
      const int goal = target(wave), piece_cost = (int)(p.p_stride / 400000) + 1;
      // every expert by itself while the budget holds them all, else one after the other
      const int own = lane < heavy ? (rows_at(lane) + BK - 1) / BK : 0, want = min(255, (own + goal - 1) / goal);
      const bool worth = wave < 3 && own > goal && own - (own + want - 1) / want > want * piece_cost;
      mine[lane] = worth ? want : 1;
      const bool over = wave_sum(wave < 3 && own > goal ? want : 0) > p.split_budget;
      if (over) mine[lane] = 1;
      __builtin_amdgcn_wave_barrier();
      if (lane == 0 && over) {
        int used = 0;
        for (int pos = 0; pos < heavy; ++pos) {
          const int nke = k_tiles(pos);
          if (nke <= goal) break;                     // heaviest first: nor will the others be cut
          int pieces = (nke + goal - 1) / goal;
          if (pieces > 255) pieces = 255;
          if (pieces > p.split_budget - used) pieces = p.split_budget - used;
          if (pieces < 2 || nke - (nke + pieces - 1) / pieces <= pieces * piece_cost) continue;
          used += pieces;
          mine[pos] = pieces;
        }
      }
      __builtin_amdgcn_wave_barrier();
      const int pieces = mine[lane];
      const float tiles = lane < heavy ? (float)(pieces * wg_tiles_per_e) : 0.f;
      const float len = lane < heavy ? (float)(3 * ((k_tiles(lane) + pieces - 1) / pieces) + (pieces > 1 ? 60 : 10)) : 0.f;
      float work = tiles * len, parts = pieces > 1 ? (float)pieces : 0.f;
      for (int pos = HEAVY + lane; pos < e_cnt; pos += WAVE) work += (float)wg_tiles_per_e * (float)(3 * k_tiles(pos) + 10);
      float as_long = 0.f;                            // tiles of at least this lane's length
      for (int j = 0; j < heavy; ++j) {
        const float other = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(len), j));
        as_long += other >= len ? __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(tiles), j)) : 0.f;
      }
      float end = ceilf(as_long * inv_grid) * len;
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) {
        work += __shfl_xor(work, o, WAVE);
        parts += __shfl_xor(parts, o, WAVE);
        end = fmaxf(end, __shfl_xor(end, o, WAVE));
      }
      if (lane == 0) price[wave] = fmaxf(end, work * inv_grid) + (parts > 0.f ? parts * (float)p.p_stride * (4.f / 375000.f) + 12.f : 0.f);
    }
    __syncthreads();
    int best = 0;
    if (may_cut) {
#pragma unroll
      for (int c = 1; c < 4; ++c)
        if (price[c] < price[best]) best = c;
    }
    for (int pos = tid; pos < e_cnt; pos += NT) split[order[pos]] = may_cut && pos < HEAVY ? trial[best * HEAVY + pos] : 1;
    __syncthreads();
    // list the experts again, now by the length of one tile's k loop (a cut expert's pieces are
    // shorter than the tiles of the next heaviest ones), longest first
    const auto length = [&](int e) { return ((offs[e + 1] - offs[e] + BK - 1) / BK + split[e] - 1) / split[e]; };
    if (in_lanes) {
      if (wave == 0) {
        const int rank = descending_rank(lane < e_cnt ? length(lane) : -1, e_cnt, lane);
        if (lane < e_cnt) order[rank] = (uint16_t)lane;
      }
    } else {
      for (int e = tid; e < e_cnt; e += NT) {
        const int len = length(e);
        int rank = 0;
        for (int o = 0; o < e_cnt; ++o) {
          const int l2 = length(o);
          rank += (l2 > len || (l2 == len && o < e)) ? 1 : 0;
        }
        order[rank] = (uint16_t)e;
      }
      __syncthreads();
    }
    if (wave == 0) {
      int tiles = 0, used = 0;
      for (int base = 0; base < e_cnt; base += WAVE) {
        const int pos = base + lane, e = pos < e_cnt ? order[pos] : 0, pieces = pos < e_cnt ? split[e] : 0;
        const int t = wave_scan(pieces), cut = pieces > 1 ? pieces : 0, c = wave_scan(cut);
        if (pos < e_cnt) {
          tile_start[pos] = (tiles + t - pieces) * wg_tiles_per_e;
          if (cut) split[e] = ((used + c - cut) << 8) | pieces;
        }
        tiles += __builtin_amdgcn_readlane(t, WAVE - 1);
        used += __builtin_amdgcn_readlane(c, WAVE - 1);
      }
      if (lane == 0) tile_start[e_cnt] = tiles * wg_tiles_per_e;
    }
    __syncthreads();
    big = tile_start[e_cnt];
    if (p.plan && blockIdx.x == 0)
      for (int e = tid; e < e_cnt; e += NT) p.plan[e] = split[e];
  } else {
    // Which rows go to 256x256 tiles and which to quarters.  Wavefront c prices plan c: row tiles of which at most half is
    // filled as quarters or not (c & 1), and, with c & 2, 256x256 tiles only as many as fill whole rounds of the chip.
    // Against 256x256 tiles only: d = 4096, f = 1536, 16 experts, 4000 rows by 1/r 174 -> 150 us (UP) and 84 -> 78 (DOWN); d =
    // 2048, f = 1408, 8 experts of 100 rows 48 -> 28 and 39 -> 24; d = f = 2880, 16 experts of 562 rows 179 -> 162 (DOWN).
    float* price = reinterpret_cast<float*>(smem);            // (the tile ring is still free)
    int32_t* limits = reinterpret_cast<int32_t*>(price + 4);
    const int n_quarters_n = (p.N + TR::BN_EFF / 2 - 1) / (TR::BN_EFF / 2);
    const auto tiles_m = [&](int rows, int plan) { return (rows + (plan & 1 ? BM / 2 - 1 : BM - 1)) / BM; };
    // the part of a plan's 256x256 tiles that lies below its limit, and the quarters of the rest, of the 64 positions at base
    const auto place = [&](int base, int plan, int limit, int& before, int& quarters) {
      const int pos = base + lane;
      const int rows = rows_at(pos);
      int m = tiles_m(rows, plan);
      const int first = before + wave_scan(m * n_tiles_n) - m * n_tiles_n;
      m = min(m, max(0, limit - first) / n_tiles_n);
      quarters = SPLIT ? (max(0, rows - BM * m) + QT - 1) / QT * n_quarters_n : 0;
      return m * n_tiles_n;
    };
    int limit = 0x7FFFFFFF;
    if (SPLIT) {
      int all = 0;
      for (int pos = lane; pos < e_cnt; pos += WAVE) all += tiles_m(rows_at(pos), wave) * n_tiles_n;
      all = wave_sum(all);
      if (wave & 2) limit = all / (int)gridDim.x * (int)gridDim.x;
      int n_big = 0, n_quarter = 0, active_big = 0, active_quarter = 0;
      for (int base = 0; base < e_cnt; base += WAVE) {
        int q;
        const int t = place(base, wave, limit, n_big, q);
        n_big += wave_sum(t);
        n_quarter += wave_sum(q);
        active_big += __popcll(__ballot(t > 0));
        active_quarter += __popcll(__ballot(q > 0));
      }
      if (lane == 0) {
        price[wave] = plan_price<MODE>(p, n_big, n_quarter, active_big, active_quarter, n_quarters_n, offs[e_cnt] - offs[0],
                                       e_cnt > 0 ? offs[order[0] + 1] - offs[order[0]] : 0, wave & 1);
        limits[wave] = limit;
      }
    }
    __syncthreads();
    int plan = 0;
    if (SPLIT) {
      // (0.97: without it 16 of 297 UPs lose more than 3 % against 256x256 tiles instead of 10, at worst 12 % instead of 8)
#pragma unroll
      for (int c = 1; c < 4; ++c)
        if (price[c] < (plan == 0 ? 0.97f : 1.f) * price[plan]) plan = c;
      limit = limits[plan];
    }
    if (wave == 0) {
      int n_big = 0, n_quarter = 0;
      for (int base = 0; base < e_cnt; base += WAVE) {
        int q;
        const int t = place(base, plan, limit, n_big, q), t_end = wave_scan(t), q_end = SPLIT ? wave_scan(q) : 0;
        if (base + lane < e_cnt) {
          tile_start[base + lane] = n_big + t_end - t;
          if (SPLIT) q_start[base + lane] = n_quarter + q_end - q;
        }
        n_big += __builtin_amdgcn_readlane(t_end, WAVE - 1);
        if (SPLIT) n_quarter += __builtin_amdgcn_readlane(q_end, WAVE - 1);
      }
      if (lane == 0) {
        tile_start[e_cnt] = n_big;
        if (SPLIT) q_start[e_cnt] = n_quarter;
      }
    }
    __syncthreads();
    big = tile_start[e_cnt];
  }

  // LDS ring.  Ragged-K shapes: four stages of [A tile | B tile].  Ragged-M shapes (PAIR): operand A
  // in two double stages of 32 KB (k-tiles 2p, 2p+1) at 0, operand B in four 16 KB stages at 64 KB.
  constexpr bool PAIR = !TR::RAGGED_K;
  static_assert(PAIR == !TR::A_TRANS, "operand A is K-contiguous exactly in the ragged-M shapes");
  constexpr int B_REGION = PAIR ? NSTAGE * OPER_BYTES : OPER_BYTES;
  // per-lane fragment offsets inside an operand tile (k-step 0; k-tile 2p of a double stage)
  int a_off[4], b_off[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int arow = wm * 128 + i * 32;
    const int brow = TR::DUAL ? (i < 2 ? 0 : 128) + wn * 64 + (i & 1) * 32 : wn * 128 + i * 32;
    a_off[i] = TR::A_TRANS ? tr_frag_off(arow, lane) : kcp_frag_off(arow + (lane & 31), lane);
    b_off[i] = B_REGION + (TR::B_TRANS ? tr_frag_off(brow, lane) : kc_frag_off(brow + (lane & 31), lane, 0));
  }

  const int G = gridDim.x;
  const int n_queues = (G % 8) == 0 ? 8 : 1;
  int queue = blockIdx.x % n_queues;       // the queue this workgroup currently draws from
  const int first_ticket = FIRST ? G / n_queues : 0;
  int pos_hint = 0;                        // list position of the last decoded tile
  const uint32_t smem_base = lds_addr(smem);

  // ---- state of the tile whose k loop runs next (written by next_tile)
  int e = 0, lo = 0, hi = 0, n0 = 0;
  int piece = -1;         // ragged-K modes: index of the fp32 partial tile to write, or -1
  int krange = 0;         // RL: which range of a cut contraction
  // Weights that one tile reads, of a layer whose active experts' weights do not fit the Infinity Cache, are loaded nontemporally (stream_rule.h):
  // decode of 128 tokens at the DSv3-like share 301 -> 280 us, prefill of 2047 at the GPT-OSS-like share 242 -> 237, training step of
  // 1936 tokens at the former 1616 -> 1586.  (Of layers that fit, the backward finds them: Qwen-like share 821 against 829.  In every
  // tile, which drops panels that tiles share, steps take 1 to 3 % longer; in dA and dX, whose weights are read 64 bytes of a row at a
  // time, up to 7 % even in tiles that share nothing.)  A loop of its own: a branch at every load costs 2 %.
  constexpr bool ONCE = MODE == UP || MODE == DOWN;
  bool once = false;      // no other tile reads this one's weights
  int active = 0;         // experts that have rows, of a layer that does not fit as a whole
  if (ONCE && e_cnt > p.cached)
    for (int base = 0; base < e_cnt; base += WAVE) active += __popcll(__ballot(rows_at(base + lane) > 0));
  int nk0 = 0, nk = 0;    // k-tiles in segment 0 / in total
  int row0 = 0;           // first output row (global row for ragged-M, i for the weight gradients)
  int row_end = 0;        // one past the last valid output row
  KcPairIssue ia_kp;
  KcIssue ib_kc;
  TrIssue ia_tr, ib_tr;

  // One of the 8 loads (q = 0..3: operand A, 4..7: operand B) of k-tile kt.  kt is clamped to
  // the last tile, so every iteration issues the same number of loads and the vmcnt
  // arithmetic below is uniform; the surplus loads re-fetch the last tile into a free stage.
  auto issue_one = [&](int kt, int q) {       // ragged-K shapes
    if (kt > nk - 1) kt = nk - 1;
    const uint32_t st = smem_base + (kt & (NSTAGE - 1)) * STAGE_BYTES;
    const int j = q & 3;
    const long k0 = (long)lo + kt * BK;
    const int k_last_rel = hi - 1 - lo - kt * BK;
    if (q < 4) ia_tr.template issue1<true>(j, st, wave, lane, k0, k_last_rel);
    else ib_tr.template issue1<true>(j, st + OPER_BYTES, wave, lane, k0, k_last_rel);
  };
  // Ragged-M shapes: one of the 8 loads of operand A's pair pj (k-tiles 2pj, 2pj+1; K is a
  // multiple of 64 per segment, so a pair never straddles DX's two segments) and one of the 4
  // loads of operand B's k-tile kt.  Both indices are clamped like kt above.
  auto issue_a_pair = [&](int pj, int q) {
    if (pj > (nk >> 1) - 1) pj = (nk >> 1) - 1;
    const int kt0 = 2 * pj;
    const bool seg1 = MODE == DX && kt0 >= nk0;
    const long kofs = (long)(seg1 ? kt0 - nk0 : kt0) * BK + (seg1 ? p.A1 - p.A0 : 0);
    ia_kp.issue1(q, smem_base + (pj & 1) * (2 * OPER_BYTES), wave, kofs);
  };
  auto issue_b = [&](int kt, int j, auto once_tag) {
    constexpr bool STREAM = decltype(once_tag)::value != 0;
    if (kt > nk - 1) kt = nk - 1;
    const uint32_t st = smem_base + B_REGION + (kt & (NSTAGE - 1)) * OPER_BYTES;
    const bool seg1 = MODE == DX && kt >= nk0;
    const int k0 = (seg1 ? kt - nk0 : kt) * BK;
    if (TR::B_TRANS) ib_tr.template issue1<false, STREAM>(j, st, wave, lane, k0, 0);
    else ib_kc.template issue1<STREAM>(j, st, wave, k0 + (seg1 ? p.B1 - p.B0 : 0));
  };
  auto issue_tile = [&](int kt) {
#pragma unroll
    for (int q = 0; q < 8; ++q) issue_one(kt, q);
  };

  // A chunk of 32 tiles (take_ticket) is an 8 x 4 block of one expert: 8 A panels and 4 B panels.
  // The ticket for the next tile is drawn near the end of the current k loop.
  //
  // next_tile: takes the ticket waiting in *next_q, decodes it into the tile state above and
  // starts the loads of that tile's first k-tiles.  The tile ring must be free when it is
  // called (it is called after the barrier that ends a k loop, before that tile's epilogue,
  // so the first operands of the next tile travel while the finished one is being stored).
  auto next_tile = [&]() -> bool {
    const int L = take_ticket<!TR::RAGGED_K>(p.sched, n_queues, queue, big, next_q, wave, lane, first_ticket, MODE != DA || !p.pair_first);
    if (L < 0) return false;
    // Within an expert, tiles are ordered in bands of 8 m-tiles, n-tile next, m-tile inside the
    // band fastest: 32 consecutive tiles (one chunk) then form an 8 x 4 block that shares 8 A
    // panels and 4 B panels through one XCD's L2.
    int mt, nt;
    {
      int li, mte;
      const int a = find_position(tile_start, e_cnt, L, pos_hint);
      pos_hint = a;
      li = __builtin_amdgcn_readfirstlane(L - tile_start[a]);
      e = __builtin_amdgcn_readfirstlane((int)order[a]);
      lo = __builtin_amdgcn_readfirstlane(offs[e]);
      hi = __builtin_amdgcn_readfirstlane(offs[e + 1]);
      if (TR::RAGGED_K) {
        mte = wg_mt;
        const int sp = __builtin_amdgcn_readfirstlane(split[e]);
        const int pieces = sp & 255;
        piece = -1;
        if (pieces > 1) {                        // this tile covers one piece of the expert's rows
          const int c_idx = li / wg_tiles_per_e;
          li -= c_idx * wg_tiles_per_e;
          const int nke = (hi - lo + BK - 1) / BK;
          const int piece_rows = ((nke + pieces - 1) / pieces) * BK;
          lo = __builtin_amdgcn_readfirstlane(min(hi, lo + c_idx * piece_rows));
          hi = __builtin_amdgcn_readfirstlane(min(hi, lo + piece_rows));
          piece = (sp >> 8) + c_idx;
        }
      } else {
        mte = __builtin_amdgcn_readfirstlane(tile_start[pos_hint + 1] - tile_start[pos_hint]) / n_tiles_n;      // (quarters take the rest)
      }
      const int band = li / (8 * n_tiles_n);
      const int in_band = li - band * 8 * n_tiles_n;
      const int band_rows = min(8, mte - band * 8);
      nt = in_band / band_rows;
      mt = band * 8 + (in_band - nt * band_rows);
    }
    if (MODE == RL) {
      krange = nt / n_tiles_cols;
      nt -= krange * n_tiles_cols;
    }
    if (ONCE) once = stream_weights(active, p.cached, hi - lo, BM);
    n0 = nt * TR::BN_EFF;
    if (TR::RAGGED_K) {
      row0 = mt * BM;
      row_end = p.M;
      nk0 = nk = (hi - lo + BK - 1) / BK;
      ia_tr.setup(p.A0, p.A0, false, p.lda, row0, p.M, wave, lane);
      ib_tr.setup(p.B0, p.B1, TR::DUAL, p.ldb, n0, p.N, wave, lane);
    } else {
      row0 = lo + mt * BM;
      row_end = hi;
      const size_t kfirst = MODE == RL ? (size_t)krange * p.K : 0;      // first column of this tile's range
      nk0 = (MODE == RL && p.ksplit > 1 ? min(p.K, p.k_total - krange * p.K) : p.K) / BK;
      nk = MODE == DX ? 2 * nk0 : nk0;
      ia_kp.setup(p.A0 + (size_t)row0 * p.lda + kfirst, p.lda, hi - row0, wave, lane);
      if (TR::B_TRANS) ib_tr.setup(p.B0 + (size_t)e * p.b_es + kfirst * p.ldb, p.B1 + (size_t)e * p.b_es, TR::DUAL, p.ldb, n0, p.N, wave, lane);
      else ib_kc.setup(p.B0 + (size_t)e * p.b_es + (size_t)n0 * p.ldb, p.ldb, p.N - n0, wave, lane);
    }
    if (nk > 0) {
      if (PAIR) {       // what the k loop's iterations -2 and -1 would have issued, in its order
#pragma unroll
        for (int q = 0; q < 8; ++q) issue_a_pair(0, q);
        auto first_b = [&](auto tag) {
#pragma unroll
          for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) issue_b(t, j, tag);
        };
        if (ONCE && once) first_b(IntC<1>{});
        else first_b(IntC<0>{});
#pragma unroll
        for (int q = 0; q < 4; ++q) issue_a_pair(1, q);
      } else {
        issue_tile(0); issue_tile(1); issue_tile(2);
#pragma unroll
        for (int q = 0; q < 4; ++q) issue_one(3, q);
      }
    } else {
      __syncthreads();   // a tile without a k loop has no barrier between this read of the ticket and its replacement
    }
    return true;
  };

  bool have = big > 0;
  if (have) {
    if (tid == 0) *next_q = FIRST ? (int)blockIdx.x / n_queues : atomicAdd(p.sched + queue, 1);
    __syncthreads();
    have = next_tile();
  }

  while (have) {
    // The ticket of the tile after this one is drawn eight k-tiles before the end of the k loop
    // (at its start if it is shorter): late, so that a workgroup commits to its next tile only
    // when it is about to be free -- tiles are listed heaviest first and long ones must go to
    // whoever finishes first -- yet early enough that the atomic's latency is never waited for.
    // It is handed over through LDS after the k loop.
    int my_ticket = 0;
    const int kt_draw = nk > 8 ? nk - 8 : 0;
    if (nk == 0 && tid == 0) my_ticket = first_ticket + atomicAdd(p.sched + queue, 1);

    f32x16 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // Fragment sets: set h holds the A and B fragments of one k-step.  frag_op(h, kt, s, o)
    // performs the o-th of the 8 fragment reads of k-step s of tile kt, in the order the
    // MFMAs consume them: A0, B0, B1, B2, B3, A1, A2, A3.
    bf16x8 fa[2][4], fb[2][4];
    auto frag_op = [&](int h, int kt, int s, int o) {
      const char* st = smem + (kt & (NSTAGE - 1)) * (PAIR ? OPER_BYTES : STAGE_BYTES);
      const bool is_a = o == 0 || o >= 5;
      const int idx = o == 0 ? 0 : (o >= 5 ? o - 4 : o - 1);
      if (is_a) {
        const char* q = TR::A_TRANS ? st + a_off[idx] + s * 4096
                                    : smem + ((kt >> 1) & 1) * (2 * OPER_BYTES) + (a_off[idx] ^ ((kt & 1) * 64 + s * 32));
        fa[h][idx] = TR::A_TRANS ? lds_frag_tr(q) : lds_frag_kc(q);
      } else {
        const char* q = st + (TR::B_TRANS ? b_off[idx] + s * 4096 : b_off[idx] ^ (s * 32));
        fb[h][idx] = TR::B_TRANS ? lds_frag_tr(q) : lds_frag_kc(q);
      }
    };
    auto mfma_one = [&](int h, int m) {
      // The 4 x 4 grid of blocks is walked in a snake (columns 0..3, 3..0, 0..3, 3..0), so that exactly one of the
      // two operand fragments changes from one MFMA to the next.  Under the package power limit the rate follows the
      // switching activity: an MFMA-only loop runs 0.8 % faster this way than row-major and 2.4 % faster than a walk
      // that changes both operands every time.
      const int i = m >> 2, j = (i & 1) ? 3 - (m & 3) : (m & 3);
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[h][i], fb[h][j], acc[i][j], 0, 0, 0);
    };
    // ragged contraction: zero the A fragment elements whose source row is past the expert's
    // last row (only the last k-tile can contain such rows)
    auto mask_tail = [&](int h, int kt, int s) {
      const int kbase = lo + kt * BK + 16 * s + 8 * (lane >> 5);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s16x8 v = __builtin_bit_cast(s16x8, fa[h][i]);
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = (kbase + j < hi) ? v[j] : (short)0;
        fa[h][i] = __builtin_bit_cast(bf16x8, v);
      }
    };

    // ---- k loop.  At the barrier of iteration kt every wavefront has all fragments of tile kt
    // in registers, so the LDS that held it is free, and tile kt+1 has landed.  Loads are spread
    // evenly over the iteration -- one per four MFMAs -- so that the CU's address unit (one
    // 64-lane load per ~24 cycles, shared by the four wavefronts) never backs up into the issue
    // stream.  Ragged-K shapes (k_loop): four stages, the first half issues operand B of tile
    // kt+3, the second half operand A of tile kt+4; issue order is A(t),B(t),A(t+1),..; at the
    // barrier the loads after B(kt+1) are A,B(kt+2) and A,B(kt+3): 16 may remain.  Ragged-M shapes:
    // k_loop_pair below.
    // The instruction order inside an iteration is fixed by hand (scheduling fences after every
    // MFMA pair): 16 MFMAs of k-step 0 with the 8 fragment reads of k-step 1 between them,
    // barrier, 16 MFMAs of k-step 1 with the next tile's first fragment reads between them.
    // The first loads (28: k-tiles 0..2 and operand A of k-tile 3; ragged-M shapes 24: A's pair
    // 0 and half of pair 1, B's k-tiles 0..2) were issued by next_tile; the stores of the previous
    // tile's epilogue were issued after them and share the counter, so the first wait is for
    // everything.
    if (nk > 0) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
#pragma unroll
      for (int o = 0; o < 8; ++o) frag_op(0, 0, 0, o);
    }
    // MV = number of 32-row MFMA blocks of this wavefront that hold valid output rows (4, 2 or
    // 0).  A tail tile's wavefronts whose rows lie past the expert's last row skip their MFMAs
    // and fragment reads but keep issuing their share of the loads and meeting the barriers.
    auto k_loop = [&](auto mv_tag) {
      constexpr int MV = decltype(mv_tag)::value;
      // fragment read o is needed iff it feeds a live MFMA: A0, B0..B3, A1, A2, A3
      auto live = [](int o) { return MV == 4 || (MV == 2 && o <= 5); };
      for (int kt = 0; kt < nk; ++kt) {
        if (kt == kt_draw && tid == 0) my_ticket = first_ticket + atomicAdd(p.sched + queue, 1);
        if (TR::RAGGED_K && kt == nk - 1) mask_tail(0, kt, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < 16; m += 2) {
          if (m < 4 * MV) mfma_one(0, m);
          if (m < 8) {                                   // all reads done well before the barrier
            if (live(m)) frag_op(1, kt, 1, m);
            if (live(m + 1)) frag_op(1, kt, 1, m + 1);
          }
          if (m < 4 * MV) mfma_one(0, m + 1);
          if ((m & 3) == 2) issue_one(kt + 3, 4 + (m >> 2));     // operand B of tile kt+3
          __builtin_amdgcn_sched_barrier(0);
        }
        asm volatile("s_waitcnt vmcnt(16) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if (TR::RAGGED_K && kt == nk - 1) mask_tail(1, kt, 1);
#pragma unroll
        for (int m = 0; m < 16; m += 2) {
          if (m < 4 * MV) mfma_one(1, m);
          if (live(m >> 1)) frag_op(0, kt + 1, 0, m >> 1);
          if (m < 4 * MV) mfma_one(1, m + 1);
          if ((m & 3) == 2) issue_one(kt + 4, m >> 2);           // operand A of tile kt+4
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    // Ragged-M shapes: the same iteration, two k-tiles per trip (nk is even).  Operand A arrives
    // in pairs of k-tiles, operand B one k-tile at a time in its own four stages, and the loads
    // stay one per four MFMAs: an even iteration kt issues the second half of A's pair kt/2+1,
    // then (after its barrier) B of tile kt+3; the odd one B of tile kt+3, then the first half
    // of A's pair (kt-1)/2+2, whose double stage its barrier has just freed.  Issue order is
    // .. B(2j+1) | B(2j+2) A(j+1)a | A(j+1)b B(2j+3) | B(2j+4) A(j+2)a | ..: at the barrier of
    // an even iteration 2j (tile 2j+1 must have landed) the 12 loads after B(2j+1) may remain,
    // at the barrier of an odd one the 8 after A(j+1)b.
    auto k_loop_pair = [&](auto mv_tag, auto once_tag) {
      constexpr int MV = decltype(mv_tag)::value;
      auto live = [](int o) { return MV == 4 || (MV == 2 && o <= 5); };
      auto iteration = [&](int kt, auto odd_tag) {
        constexpr bool ODD = decltype(odd_tag)::value != 0;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < 16; m += 2) {
          if (m < 4 * MV) mfma_one(0, m);
          if (m < 8) {
            if (live(m)) frag_op(1, kt, 1, m);
            if (live(m + 1)) frag_op(1, kt, 1, m + 1);
          }
          if (m < 4 * MV) mfma_one(0, m + 1);
          if ((m & 3) == 2) {
            if (ODD) issue_b(kt + 3, m >> 2, once_tag);
            else issue_a_pair((kt >> 1) + 1, 4 + (m >> 2));
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        if (ODD) asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(12) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < 16; m += 2) {
          if (m < 4 * MV) mfma_one(1, m);
          if (live(m >> 1)) frag_op(0, kt + 1, 0, m >> 1);
          if (m < 4 * MV) mfma_one(1, m + 1);
          if ((m & 3) == 2) {
            if (ODD) issue_a_pair((kt >> 1) + 2, m >> 2);
            else issue_b(kt + 3, m >> 2, once_tag);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      for (int kt = 0; kt < nk; kt += 2) {
        if (kt == kt_draw && tid == 0) my_ticket = first_ticket + atomicAdd(p.sched + queue, 1);
        iteration(kt, IntC<0>{});
        iteration(kt + 1, IntC<1>{});
      }
    };
    if (TR::RAGGED_K) {
      k_loop(IntC<4>{});
    } else {
      const int rows_left = row_end - (row0 + wm * 128);
      const int mv = rows_left > 64 ? 4 : (rows_left > 0 ? 2 : 0);
      auto rows_loop = [&](auto once_tag) {
        if (mv == 4) k_loop_pair(IntC<4>{}, once_tag);
        else if (mv == 2) k_loop_pair(IntC<2>{}, once_tag);
        else k_loop_pair(IntC<0>{}, once_tag);
      };
      if (ONCE && once) rows_loop(IntC<1>{});
      else rows_loop(IntC<0>{});
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    if (tid == 0) *next_q = my_ticket;
    __syncthreads();

    // the ring is free: decode the next tile and start its first loads, then store this one
    const int ep_e = e, ep_row0 = row0, ep_row_end = row_end, ep_n0 = n0, ep_piece = piece, ep_krange = krange;
    have = next_tile();

    // ---------------------------------------------------------------- epilogue
    // Each wavefront moves its 128x128 accumulators through a private LDS slab (outside the
    // tile ring, which already receives the next tile), 16 slabs per tile, and walks each slab
    // row-major so that global accesses are 16 bytes per lane and 128 bytes per row segment.
    // A slab is private to its wavefront and LDS executes a wavefront's accesses in order, so
    // no workgroup barrier is needed between the writes and the reads.
    // (three instances: a piece of a cut expert stores fp32 partial tiles, every other tile the final
    // result, either overwriting or adding to what is there; adding is an instance of its own so that
    // the loads of the old values are unconditional and stay where they are issued)
    auto epilogue = [&](auto partial_tag, auto rmw_tag) {
    constexpr bool PARTIAL = decltype(partial_tag)::value != 0;
    constexpr bool RMW_TAG = decltype(rmw_tag)::value != 0;
    float* stage = reinterpret_cast<float*>(smem + STAGING_OFF) + wave * (STAGING_WAVE_BYTES / 4);
    const int acc_col = lane & 31, acc_rg = lane >> 5;
    if (TR::DUAL) {
      // slab = 8 rows x 128 columns: both halves of a dual tile, so that a lane holds h1 and h3
      // (or dW1 and dW3) of the same position.  lanes: 8 per row (8 columns each).
      const int c8 = lane & 7, rl = lane >> 3;
      // WGD adding to existing gradients: the old values of a slab are fetched C_AHEAD slabs
      // before they are needed (clamped addresses), so that the read-modify-write does not
      // wait for memory once per slab
      constexpr int C_AHEAD = 3;
      constexpr bool rmw = MODE == WGD && !PARTIAL && RMW_TAG;
      uint4 old0[C_AHEAD + 1], old1[C_AHEAD + 1];
      auto old_fetch = [&](int sl) {
        int grow = ep_row0 + wm * 128 + (sl >> 2) * 32 + 8 * (sl & 3) + rl;
        int gcol = ep_n0 + wn * 64 + c8 * 8;
        if (grow > ep_row_end - 1) grow = ep_row_end - 1;
        if (gcol > p.N - 8) gcol = p.N - 8;
        const size_t idx = (size_t)ep_e * p.c_es + (size_t)grow * p.ldc + gcol;
        old0[sl % (C_AHEAD + 1)] = load16_once(p.C0 + idx);
        old1[sl % (C_AHEAD + 1)] = load16_once(p.C1 + idx);
      };
      if (rmw) {
#pragma unroll
        for (int sl = 0; sl < C_AHEAD; ++sl) old_fetch(sl);
      }
#pragma unroll
      for (int sl = 0; sl < 16; ++sl) {
        const int mi = sl >> 2, g = sl & 3;
        if (rmw && sl + C_AHEAD < 16) old_fetch(sl + C_AHEAD);
#pragma unroll
        for (int nj = 0; nj < 4; ++nj)
#pragma unroll
          for (int i = 0; i < 4; ++i) stage[(4 * acc_rg + i) * DPITCH + nj * 32 + acc_col] = acc[mi][nj][4 * g + i];
        __builtin_amdgcn_wave_barrier();
        const int grow = ep_row0 + wm * 128 + mi * 32 + 8 * g + rl;
        const int gcol = ep_n0 + wn * 64 + c8 * 8;
        const float* s1 = stage + rl * DPITCH + c8 * 8;
        const float* s3 = s1 + 64;
        float x1[8], x3[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) { x1[i] = s1[i]; x3[i] = s3[i]; }
        __builtin_amdgcn_wave_barrier();
        if (grow < ep_row_end && gcol < p.N) {
          if (MODE == UP) {
            const size_t idx = (size_t)grow * p.ldc + gcol;
            finish_up(p, idx, x1, x3);
          } else if (PARTIAL) {   // WGD, one piece of a cut expert: fp32 partial tiles
            float* c0 = p.P0 + (size_t)ep_piece * p.p_stride + (size_t)grow * p.ldc + gcol;
            float* c1 = c0 + (size_t)p.M * p.N;
            *reinterpret_cast<float4*>(c0) = make_float4(x1[0], x1[1], x1[2], x1[3]);
            *reinterpret_cast<float4*>(c0 + 4) = make_float4(x1[4], x1[5], x1[6], x1[7]);
            *reinterpret_cast<float4*>(c1) = make_float4(x3[0], x3[1], x3[2], x3[3]);
            *reinterpret_cast<float4*>(c1 + 4) = make_float4(x3[4], x3[5], x3[6], x3[7]);
          } else {   // WGD: two weight-gradient outputs
            const size_t idx = (size_t)ep_e * p.c_es + (size_t)grow * p.ldc + gcol;
            bf16_t* c0 = p.C0 + idx;
            bf16_t* c1 = p.C1 + idx;
            if (rmw) {
              add8(x1, old0[sl % (C_AHEAD + 1)]);
              add8(x3, old1[sl % (C_AHEAD + 1)]);
            }
            store16(c0, pack8(x1));
            store16(c1, pack8(x3));
          }
        }
      }
    } else {
      // slab = 16 rows x 64 columns; lanes: 8 per row (8 columns each), 8 rows per pass.
      // slab sl: accumulator block row mi = sl/4, row half h = (sl/2)%2, column pair np = sl%2.
      const int c8 = lane & 7;
      // DA: h1/h3 of a slab are fetched DA_AHEAD slabs before they are needed (clamped
      // addresses), so that their latency is hidden behind the slabs in between
      constexpr int DA_AHEAD = 3;
      uint4 pre1[DA_AHEAD + 1][2], pre3[DA_AHEAD + 1][2];
      auto da_fetch = [&](int sl) {
        const int mi = sl >> 2, h = (sl >> 1) & 1, np = sl & 1;
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
          int grow = ep_row0 + wm * 128 + mi * 32 + 16 * h + pass * 8 + (lane >> 3);
          int gcol = ep_n0 + wn * 128 + np * 64 + c8 * 8;
          if (grow > ep_row_end - 1) grow = ep_row_end - 1;
          if (gcol > p.N - 8) gcol = p.N - 8;
          const size_t idx = (size_t)grow * p.ldc + gcol;
          pre1[sl % (DA_AHEAD + 1)][pass] = load16_once(p.H1 + idx);
          pre3[sl % (DA_AHEAD + 1)][pass] = load16_once(p.H3 + idx);
        }
      };
      // WG and the router's dx adding to existing gradients: the same, with the old values
      constexpr bool rmw = (MODE == WG || MODE == RX) && !PARTIAL && RMW_TAG;
      auto old_fetch = [&](int sl) {
        const int mi = sl >> 2, h = (sl >> 1) & 1, np = sl & 1;
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
          int grow = ep_row0 + wm * 128 + mi * 32 + 16 * h + pass * 8 + (lane >> 3);
          int gcol = ep_n0 + wn * 128 + np * 64 + c8 * 8;
          if (grow > ep_row_end - 1) grow = ep_row_end - 1;
          if (gcol > p.N - 8) gcol = p.N - 8;
          const size_t idx = (MODE == WG ? (size_t)ep_e * p.c_es : (size_t)0) + (size_t)grow * p.ldc + gcol;
          pre1[sl % (DA_AHEAD + 1)][pass] = load16_once(p.C0 + idx);
        }
      };
      if (MODE == DA) {
#pragma unroll
        for (int sl = 0; sl < DA_AHEAD; ++sl) da_fetch(sl);
      }
      if (rmw) {
#pragma unroll
        for (int sl = 0; sl < DA_AHEAD; ++sl) old_fetch(sl);
      }
#pragma unroll
      for (int sl = 0; sl < 16; ++sl) {
        const int mi = sl >> 2, h = (sl >> 1) & 1, np = sl & 1;
        if (MODE == DA && sl + DA_AHEAD < 16) da_fetch(sl + DA_AHEAD);
        if (rmw && sl + DA_AHEAD < 16) old_fetch(sl + DA_AHEAD);
#pragma unroll
        for (int gg = 0; gg < 2; ++gg)
#pragma unroll
          for (int nn = 0; nn < 2; ++nn)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              stage[(8 * gg + 4 * acc_rg + i) * SPITCH + nn * 32 + acc_col] = acc[mi][2 * np + nn][4 * (2 * h + gg) + i];
        __builtin_amdgcn_wave_barrier();
        float xs[2][8];
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
          const float* sp = stage + (pass * 8 + (lane >> 3)) * SPITCH + c8 * 8;
#pragma unroll
          for (int i = 0; i < 8; ++i) xs[pass][i] = sp[i];
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
          const int grow = ep_row0 + wm * 128 + mi * 32 + 16 * h + pass * 8 + (lane >> 3);
          const int gcol = ep_n0 + wn * 128 + np * 64 + c8 * 8;
          float* x = xs[pass];
          if (grow < ep_row_end && gcol < p.N) {
            if (MODE == DA) {
              const size_t idx = (size_t)grow * p.ldc + gcol;
              finish_da(p, idx, x, pre1[sl % (DA_AHEAD + 1)][pass], pre3[sl % (DA_AHEAD + 1)][pass]);
            } else if (MODE == WG && PARTIAL) {   // one piece of a cut expert: fp32 partial tile
              float* c0 = p.P0 + (size_t)ep_piece * p.p_stride + (size_t)grow * p.ldc + gcol;
              *reinterpret_cast<float4*>(c0) = make_float4(x[0], x[1], x[2], x[3]);
              *reinterpret_cast<float4*>(c0 + 4) = make_float4(x[4], x[5], x[6], x[7]);
            } else if (MODE == RL || MODE == RW) {
              float* c0 = p.F0 + (size_t)(MODE == RW ? ep_e : ep_krange) * p.c_es + (size_t)grow * p.ldc + gcol;
              *reinterpret_cast<float4*>(c0) = make_float4(x[0], x[1], x[2], x[3]);
              *reinterpret_cast<float4*>(c0 + 4) = make_float4(x[4], x[5], x[6], x[7]);
            } else {
              const size_t idx = (MODE == WG ? (size_t)ep_e * p.c_es : (size_t)0) + (size_t)grow * p.ldc + gcol;
              bf16_t* c0 = p.C0 + idx;
              if (rmw) add8(x, pre1[sl % (DA_AHEAD + 1)][pass]);
              store16(c0, pack8(x));
            }
          }
        }
      }
    }
    };
    if ((MODE == WG || MODE == WGD) && ep_piece >= 0) epilogue(IntC<1>{}, IntC<0>{});
    else if ((MODE == WG || MODE == WGD || MODE == RX) && p.accumulate) epilogue(IntC<0>{}, IntC<1>{});
    else epilogue(IntC<0>{}, IntC<0>{});
  }
  if constexpr (SPLIT) {
    const Quarters list = {offs, order, tile_start, q_start, n_tiles_n, __builtin_amdgcn_readfirstlane(q_start[e_cnt]), next_q};
    if (list.total > 0) {
      __syncthreads();       // everyone has read the ticket that ended the 256x256 tiles
      quarter_tiles<MODE>(p, list);
    }
  }
}

template <int MODE>
__global__ __launch_bounds__(NT, 1) void gg_kernel(GArgs p) {
  gg_body<MODE, true>(p);
}

// Whether the kernel for few rows is the faster one at these row counts (whole wavefronts; the same answer in all of them): its
// time and the tiles', each from the rounds, the work per CU and the bytes of both GEMMs, in us, fitted to 12 shapes with 1 to 128
// rows per expert.  The estimate is good to a quarter: over 315 cases (9 shapes, bounds of 17 to 128 rows, filled evenly, by 1/r,
// by one expert, to an eighth) the kernel for few rows took 0.44 to 0.86 of the tiles' time where the ratio is below 0.75, and
// 0.6 to 1.9 above.  The tiles' price is that of 256x256 ones.  With quarter tiles among them the choice is 6 % above the better
// kernel on average over 64 cases (4 shapes, bounds of 32 to 128, the four ways of filling below), at worst 21 % (16 experts of
// d = f = 2880 with three rows each: 146 us for few rows, 174 for the tiles it takes).
__device__ __forceinline__ bool few_rows_pay(const int32_t* __restrict__ off, int e_cnt, int d, int f) {
  constexpr float C1 = 0.563f, C2 = 0.752f, C4 = 1.173f;       // a round of 128 k with up to 16, 32 and 64 rows
  float v[5] = {0.f, 0.f, 0.f, 0.f, 0.f};            // rounds' cost of a column block, tiles of 64 rows, of 256, active experts; longest
  for (int e = lane_id(); e < e_cnt; e += WAVE) {
    const int rows = off[e + 1] - off[e], rest = rows & 63;
    const float last = rest > 32 ? C4 : (rest > 16 ? C2 : (rest > 0 ? C1 : 0.f));
    v[0] += (float)(rows >> 6) * C4 + last;
    v[1] += (float)((rows + 63) >> 6);
    v[2] += (float)((rows + 255) >> 8);
    v[3] += rows > 0 ? 1.f : 0.f;
    v[4] = fmaxf(v[4], rows > 63 ? C4 : last);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] += __shfl_xor(v[k], o, WAVE);
    v[4] = fmaxf(v[4], __shfl_xor(v[4], o, WAVE));
  }
  const float inv_grid = 1.f / (float)gridDim.x;
  float few = 0.f, tiles = 2.f * (13.f - 3.85f);     // launch, first loads and last stores
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const int K = g == 0 ? d : f;
    const float few_cols = (float)(g == 0 ? (f + 63) / 64 : (d + 127) / 128), cols = (float)(g == 0 ? (f + 127) / 128 : (d + 255) / 256);
    const float rounds = (float)K / 128.f, bytes = (g == 0 ? 4e-6f : 2e-6f) * (float)d * (float)f;      // of one expert, MB
    few += fmaxf(fmaxf(v[4] * rounds, v[0] * few_cols * rounds * inv_grid), 0.194f * v[1] * bytes);
    const float n = v[2] * cols;
    tiles += fmaxf(fmaxf(0.419f * 4.f * rounds * ceilf(n * inv_grid), 0.866f * 4.f * rounds * n * inv_grid), 0.19f * v[3] * bytes);
  }
  return __builtin_amdgcn_readfirstlane(few < 0.75f * tiles);
}

// Forward GEMM of a call whose capacity leaves open which kernel pays: the row counts decide, in every block alike.
template <int MODE>
__global__ __launch_bounds__(NT, 1) void gg_or_few(GArgs p, int d, int f) {
  if (few_rows_pay(p.off, p.e_cnt, d, f)) {
    SArgs q = {};
    q.A = p.A0; q.lda = p.lda; q.B0 = p.B0; q.B1 = p.B1; q.ldb = p.ldb; q.b_es = p.b_es;
    q.C0 = p.C0; q.C1 = p.C1; q.C2 = p.C2; q.ldc = p.ldc; q.off = p.off; q.e_cnt = p.e_cnt; q.N = p.N; q.K = p.K; q.cached = p.cached;
    const RaggedTiles<ROWS> list(q.off, q.e_cnt, threadIdx.x & 63);
    for (int b = blockIdx.x; few_rows_tile<MODE == UP, NW_TILES, true>(q, list, reinterpret_cast<u32x4*>(smem), b); b += gridDim.x) {}
    return;
  }
  gg_body<MODE, true>(p);
}

// Two grouped GEMMs that do not depend on each other in one launch: a workgroup that finds no tile
// of the first left goes on to the second at once, so the second fills the first one's tail (the
// last round of whole tiles, in which most CUs would idle) and one launch boundary goes away.
template <int M1, int M2>
__global__ __launch_bounds__(NT, 1) void gg_pair(GArgs p1, GArgs p2) {
  gg_body<M1, true>(p1);
  __syncthreads();          // the first GEMM's scheduler tables in LDS are rewritten by the second's set-up
  gg_body<M2, false>(p2);
}

__global__ void zero_words(int32_t* p, int n) {
  if ((int)threadIdx.x < n) p[threadIdx.x] = 0;
}

// Adds up the fp32 partial tiles of the experts that the weight-gradient kernel cut into pieces
// (plan[e] = (first piece << 8) | pieces), in piece order, and writes the bf16 gradient.
// Every block first lists the cut experts, then the grid walks the elements of all of them
// together (n_out outputs of mn elements each per expert), so that a single hot expert is
// reduced by the whole chip; with no cut expert every block exits after reading the plan.
__global__ __launch_bounds__(256) void wgrad_reduce(const int32_t* __restrict__ plan, int e_cnt,
                                                   const float* __restrict__ P0, long p_stride, long mn, int n_out,
                                                   bf16_t* __restrict__ C0, bf16_t* __restrict__ C1, long c_es,
                                                   int accumulate) {
  __shared__ int32_t list[MOE_MAX_LOCAL];   // the cut experts in ascending order: the same list in every block
  __shared__ uint8_t cut[MOE_MAX_LOCAL];
  __shared__ int n_cut;
  if (threadIdx.x == 0) n_cut = 0;
  for (int e = threadIdx.x; e < e_cnt; e += 256) cut[e] = (plan[e] & 255) > 1;
  __syncthreads();
  for (int e = threadIdx.x; e < e_cnt; e += 256)
    if (cut[e]) {
      int rank = 0;
      for (int j = 0; j < e; ++j) rank += cut[j];
      list[rank] = e;
      atomicAdd(&n_cut, 1);
    }
  __syncthreads();
  const long vecs = mn / 8;                       // mn is a multiple of 64 * 64
  const long per_e = vecs * n_out;
  const long total = per_e * n_cut;
  for (long g = (long)blockIdx.x * 256 + threadIdx.x; g < total; g += (long)gridDim.x * 256) {
    const int e = list[g / per_e];
    const long r = g % per_e;
    const int o = (int)(r / vecs);
    const long v = r - o * vecs;
    const int sp = plan[e];
    const int pieces = sp & 255;
    const float* base = P0 + (size_t)(sp >> 8) * p_stride + (size_t)o * mn + v * 8;
    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.f;
    for (int c = 0; c < pieces; ++c) {
      const float* q = base + (size_t)c * p_stride;
      const float4 a = *reinterpret_cast<const float4*>(q), b = *reinterpret_cast<const float4*>(q + 4);
      acc[0] += a.x; acc[1] += a.y; acc[2] += a.z; acc[3] += a.w;
      acc[4] += b.x; acc[5] += b.y; acc[6] += b.z; acc[7] += b.w;
    }
    uint4* dst = reinterpret_cast<uint4*>((o ? C1 : C0) + (size_t)e * c_es + v * 8);
    if (accumulate) {
      const uint4 q0 = *dst;
      const uint32_t* u0 = reinterpret_cast<const uint32_t*>(&q0);
#pragma unroll
      for (int i = 0; i < 4; ++i) { acc[2 * i] += bf16lo(u0[i]); acc[2 * i + 1] += bf16hi(u0[i]); }
    }
    uint4 out;
    uint32_t* w = reinterpret_cast<uint32_t*>(&out);
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = pack_bf16x2(acc[2 * i], acc[2 * i + 1]);
    *dst = out;
  }
}

// ticket counters live in the 256 bytes of slack that moe_workspace_bytes adds after the
// activation scratch; each kernel of an entry point gets its own 8 (one per XCD)
inline int32_t* sched_area(void* ws, size_t scratch_bytes) {
  return reinterpret_cast<int32_t*>(static_cast<char*>(ws) + ((scratch_bytes + 255) & ~(size_t)255));
}

constexpr size_t WGRAD_PLAN_BYTES = 2 * MOE_MAX_LOCAL * 4;

template <int M1, int M2>
int launch_pair(const GArgs& a, const GArgs& b, int prof_id, hipStream_t s) {
  static bool attr_set[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MOE_EHIP;
  if (!attr_set[dev]) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&gg_pair<M1, M2>), hipFuncAttributeMaxDynamicSharedMemorySize,
                            SMEM_BYTES) != hipSuccess)
      return MOE_EHIP;
    attr_set[dev] = true;
  }
  ProfScope prof(prof_id, s);
  GArgs first = a;
  first.pair_first = 1;
  hipLaunchKernelGGL((gg_pair<M1, M2>), dim3(device_cu_count()), dim3(NT), SMEM_BYTES, s, first, b);
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}

template <int MODE>
int launch_gg_or_few(const GArgs& a, int d, int f, hipStream_t s) {
  static_assert(FEW_ROWS_PLACES<NW_TILES> * 16 <= SMEM_BYTES && NW_TILES * WAVE == NT, "one block serves both");
  static bool attr_set[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MOE_EHIP;
  if (!attr_set[dev]) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&gg_or_few<MODE>), hipFuncAttributeMaxDynamicSharedMemorySize,
                            SMEM_BYTES) != hipSuccess)
      return MOE_EHIP;
    attr_set[dev] = true;
  }
  ProfScope prof(MOE_K_UP + MODE, s);
  hipLaunchKernelGGL(gg_or_few<MODE>, dim3(device_cu_count()), dim3(NT), SMEM_BYTES, s, a, d, f);
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}

template <int MODE>
int launch_gg(const GArgs& a, hipStream_t s) {
  // the LDS opt-in is a per-device attribute of the kernel
  static bool attr_set[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MOE_EHIP;
  if (!attr_set[dev]) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&gg_kernel<MODE>), hipFuncAttributeMaxDynamicSharedMemorySize,
                            SMEM_BYTES) != hipSuccess)
      return MOE_EHIP;
    attr_set[dev] = true;
  }
  int grid = device_cu_count();
  ProfScope prof(MODE == RL ? MOE_K_ROUTER_FWD : MODE == RW ? MOE_K_ROUTER_DW : MODE == RX ? MOE_K_ROUTER_DX : MOE_K_UP + MODE, s);
  hipLaunchKernelGGL(gg_kernel<MODE>, dim3(grid), dim3(NT), SMEM_BYTES, s, a);
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}

}  // namespace

// Which kernel the forward takes: the one for few rows (few_rows.h; results are the same bit for bit) or the 256x256 tiles.  The
// former reads an expert's weights once per 64 rows, the tiles once per 256 with 256 rows' worth of work each.  The true row
// counts are on the device, the host knows a bound.  Forward of both GEMMs, few rows / tiles, in us, with the bound filled
// evenly, by 1/r (Zipf), by one expert alone, and to a tenth:
//   weights  d, f, experts       bound   even         Zipf         one          a tenth
//   138 MB   2048, 1408, 8       64      40 / 47      43 / 51      41 / 45      28 / 42
//                                96      54 / 49      61 / 54      60 / 46      28 / 43
//                                128     61 / 51      75 / 55      61 / 48      28 / 43
//   151 MB   2048, 768, 16       64      38 / 51      66 / 59      36 / 42      30 / 49
//                                128     66 / 50      77 / 75      65 / 46      31 / 50
//   604 MB   4096, 1536, 16      16      128 / 144    158 / 145    62 / 60      122 / 145
//                                128     247 / 153    296 / 176    208 / 109    129 / 143
//   796 MB   2880, 2880, 16      16      152 / 177    187 / 177    59 / 59      145 / 172
//                                64      197 / 185    269 / 189    148 / 84     148 / 174
//   2.8 GB   7168, 2048, 32      8       501 / 531    536 / 531    93 / 81      399 / 423
//                                16      514 / 532    652 / 537    123 / 83     492 / 527
//   2.8 GB   4096, 14336, 8      8       509 / 515    531 / 514    174 / 191    379 / 387
// While all weights fit the Infinity Cache (256 MB) few rows win up to a bound of 64, bar one case.  Between 64 and 128 they win where
// the bound is far above the counts and lose by up to 45 % where it is full: the line at 128 was drawn against tiles of 256x256 only,
// which took 87 us in the first row of 128.  Up to a bound of 16, with more than 1 GB of 8, they win or lose little.  Up to 1 GB
// and 128 rows it depends on the counts: gg_or_few looks at them.
enum { MANY_ROWS, FEW_ROWS, COUNTS_DECIDE };
inline int rows_route(int cap, int d, int f, int e_cnt) {
  const long long mb = 6ll * d * f * e_cnt >> 20;
  const long long bound = mb <= 256 ? 128 : (mb <= 1024 ? 16 : 8);
  return cap <= bound * e_cnt ? FEW_ROWS : (mb <= 1024 && cap <= 128ll * e_cnt ? COUNTS_DECIDE : MANY_ROWS);
}

int launch_expert_fwd_bf16(const void* xp, int cap, int d, int f, int e_cnt, const int32_t* offsets,
                           const void* w1, const void* w3, const void* w2, void* h1, void* h3, void* a_out, void* o,
                           void* a_ws, hipStream_t s) {
  if (cap == 0 || e_cnt == 0) return MOE_OK;
  bf16_t* act = a_out ? (bf16_t*)a_out : (bf16_t*)a_ws;
  const int route = rows_route(cap, d, f, e_cnt);
  if (route == FEW_ROWS) return launch_expert_fwd_small(xp, cap, d, f, e_cnt, offsets, w1, w3, w2, h1, h3, act, o, s);
  int32_t* sched = sched_area(a_ws, (size_t)cap * f * 2);
  hipLaunchKernelGGL(zero_words, dim3(1), dim3(64), 0, s, sched, 32);
  HIP_CHECK_LAUNCH();
  GArgs u = {}, w = {};
  u.A0 = u.A1 = (const bf16_t*)xp; u.lda = d;
  u.B0 = (const bf16_t*)w1; u.B1 = (const bf16_t*)w3; u.ldb = f; u.b_es = (long)d * f;
  u.C0 = (bf16_t*)h1; u.C1 = (bf16_t*)h3; u.C2 = act; u.ldc = f;
  u.cached = w.cached = cached_experts(d, f);
  u.off = offsets; u.sched = sched; u.e_cnt = e_cnt; u.N = f; u.K = d; u.save_h = (h1 && h3) ? 1 : 0;
  const bool decide = route == COUNTS_DECIDE;
  int rc = decide ? launch_gg_or_few<UP>(u, d, f, s) : launch_gg<UP>(u, s);
  if (rc) return rc;
  w.A0 = w.A1 = act; w.lda = f;
  w.B0 = w.B1 = (const bf16_t*)w2; w.ldb = d; w.b_es = (long)f * d;
  w.C0 = (bf16_t*)o; w.ldc = d;
  w.off = offsets; w.sched = sched + 16; w.e_cnt = e_cnt; w.N = d; w.K = f;
  return decide ? launch_gg_or_few<DOWN>(w, d, f, s) : launch_gg<DOWN>(w, s);
}

int launch_expert_bwd_bf16(const void* xp, const void* h1, const void* h3, const void* a_in, const void* d_o, int cap,
                           int d, int f, int e_cnt, const int32_t* offsets, const void* w1,
                           const void* w3, const void* w2, void* dxp, void* dw1, void* dw3, void* dw2,
                           int accumulate, void* ws, hipStream_t s) {
  if (e_cnt == 0) return MOE_OK;
  bf16_t* a = (bf16_t*)ws;
  bf16_t* dh1 = a + (size_t)cap * f;
  bf16_t* dh3 = dh1 + (size_t)cap * f;
  int32_t* sched = sched_area(ws, 3 * (size_t)cap * f * 2);
  int32_t* plans = sched + 64;                                   // two plans of MOE_MAX_LOCAL words
  float* partials = reinterpret_cast<float*>(reinterpret_cast<char*>(sched) + 256 + WGRAD_PLAN_BYTES);
  const size_t split_bytes = wgrad_split_bytes(d, f);
  const long mn = (long)d * f;
  hipLaunchKernelGGL(zero_words, dim3(1), dim3(64), 0, s, sched, 64);
  HIP_CHECK_LAUNCH();
  GArgs g = {};   // dA = d_o W2^T, epilogue -> a, dH1, dH3
  g.A0 = g.A1 = (const bf16_t*)d_o; g.lda = d;
  g.B0 = g.B1 = (const bf16_t*)w2; g.ldb = d; g.b_es = (long)f * d;
  g.C0 = a_in ? nullptr : a; g.C1 = dh1; g.C2 = dh3; g.ldc = f;
  g.H1 = (const bf16_t*)h1; g.H3 = (const bf16_t*)h3;
  g.off = offsets; g.sched = sched; g.e_cnt = e_cnt; g.N = f; g.K = d;
  GArgs x = {};   // dxp = dH1 W1^T + dH3 W3^T
  x.A0 = dh1; x.A1 = dh3; x.lda = f;
  x.B0 = (const bf16_t*)w1; x.B1 = (const bf16_t*)w3; x.ldb = f; x.b_es = (long)d * f;
  x.C0 = (bf16_t*)dxp; x.ldc = d;
  x.off = offsets; x.sched = sched + 16; x.e_cnt = e_cnt; x.N = d; x.K = f;
  GArgs w = {};   // dW2 = a^T d_o
  w.A0 = w.A1 = a_in ? (const bf16_t*)a_in : a; w.lda = f;
  w.B0 = w.B1 = (const bf16_t*)d_o; w.ldb = d;
  w.C0 = (bf16_t*)dw2; w.ldc = d; w.c_es = (long)f * d;
  w.off = offsets; w.sched = sched + 32; w.e_cnt = e_cnt; w.M = f; w.N = d; w.accumulate = accumulate;
  w.P0 = partials; w.p_stride = mn; w.split_budget = (int)(split_bytes / (mn * 4)); w.plan = plans;
  GArgs v = {};   // dW1|dW3 = xp^T [dH1|dH3]
  v.A0 = v.A1 = (const bf16_t*)xp; v.lda = d;
  v.B0 = dh1; v.B1 = dh3; v.ldb = f;
  v.C0 = (bf16_t*)dw1; v.C1 = (bf16_t*)dw3; v.ldc = f; v.c_es = (long)d * f;
  v.off = offsets; v.sched = sched + 48; v.e_cnt = e_cnt; v.M = d; v.N = f; v.accumulate = accumulate;
  v.P0 = partials; v.p_stride = 2 * mn; v.split_budget = (int)(split_bytes / (2 * mn * 4)); v.plan = plans + MOE_MAX_LOCAL;
  // Order and pairing.  dW2 needs a and d_o, dX and dW1|dW3 need what dA's epilogue writes (dH1, dH3).  With the
  // forward's a at hand dA and dW2 are independent, dX and dW1|dW3 always are, and independent GEMMs may share a
  // launch (gg_pair).  That pays while the first GEMM's tail -- its last round of whole tiles -- is a visible part
  // of it; the second GEMM's workgroups then start out of step, and the panels that the 32 workgroups of an XCD
  // would share through their L2 while walking k together are fetched more often (a quarter more L2 misses
  // measured).  Measured break-even: about a dozen rounds of tiles per workgroup in the first GEMM (a pair gains
  // 2.5-4 % at 8-9 rounds and loses 1-2.5 % at 29-31), counted from the capacity bound since the row counts are
  // on the device.  The fp32 partial tiles of cut experts are one buffer: dW2's are added up before dW1|dW3
  // writes its own.
  int rc;
  const int red_grid = 4 * device_cu_count();
  const auto rounds = [&](int n_cols) {     // tiles of a ragged-M GEMM with n_cols output columns, per workgroup
    const long long m_tiles = (cap + BM - 1) / BM + e_cnt / 2;
    return m_tiles * ((n_cols + BN - 1) / BN) / device_cu_count();
  };
  constexpr int PAIR_MAX_ROUNDS = 12;
  if (cap == 0) {            // no rows at all: only the gradients are written (zeros unless accumulating)
    if ((rc = launch_gg<WG>(w, s))) return rc;
  } else if (a_in && rounds(f) <= PAIR_MAX_ROUNDS) {
    if ((rc = launch_pair<DA, WG>(g, w, MOE_K_DA_WG, s))) return rc;
  } else {
    if ((rc = launch_gg<DA>(g, s))) return rc;
    if ((rc = launch_gg<WG>(w, s))) return rc;
  }
  {
    ProfScope prof(MOE_K_WGRAD_REDUCE, s);
    hipLaunchKernelGGL(wgrad_reduce, dim3(red_grid), dim3(256), 0, s, plans, e_cnt, partials, mn, mn, 1, (bf16_t*)dw2,
                       (bf16_t*)dw2, mn, accumulate);
  }
  HIP_CHECK_LAUNCH();
  if (cap == 0) {
    if ((rc = launch_gg<WGD>(v, s))) return rc;
  } else if (rounds(d) <= PAIR_MAX_ROUNDS) {
    if ((rc = launch_pair<DX, WGD>(x, v, MOE_K_DX_WGD, s))) return rc;
  } else {
    if ((rc = launch_gg<DX>(x, s))) return rc;
    if ((rc = launch_gg<WGD>(v, s))) return rc;
  }
  {
    ProfScope prof(MOE_K_WGRAD_REDUCE, s);
    hipLaunchKernelGGL(wgrad_reduce, dim3(red_grid), dim3(256), 0, s, plans + MOE_MAX_LOCAL, e_cnt, partials, 2 * mn, mn, 2,
                       (bf16_t*)dw1, (bf16_t*)dw3, mn, accumulate);
  }
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}

// ---- trainable router on the matrix cores (bf16, E % 64 == 0, d % 64 == 0) ----------------
// ws layout of the backward: [0,256) ticket counters; then dl as bf16 [T,E]; then the fp32 chunk sums [S,d,E], or in the
// same bytes the streaming weight gradient's operand (pieces of dl) and its sums.  The forward's range tiles start at 256.
// Into how many chunks of tokens the router's weight gradient is cut: the split whose schedule is
// shortest, counted in k-tiles per workgroup: rounds of the chip's CUs times (k-tiles per chunk +
// what a tile costs besides its k loop, about 16 k-tiles for its first loads and its fp32 stores).
constexpr int SPLIT_OVERHEAD_KTILES = 16;
int router_dw_splits(int T, int d, int E) {
  const long long tiles = (long long)((d + BM - 1) / BM) * ((E + BN - 1) / BN);
  const int cus = device_cu_count();
  const int max_by_rows = (T + 4 * BK - 1) / (4 * BK);      // at least four k-tiles per chunk
  int best = 1;
  long long best_cost = -1;
  for (int s = 1; s <= 32 && s <= max_by_rows; ++s) {
    const long long rounds = (tiles * s + cus - 1) / cus;
    const long long cost = rounds * (((T + s - 1) / s + BK - 1) / BK + SPLIT_OVERHEAD_KTILES);
    if (best_cost < 0 || cost < best_cost) { best = s; best_cost = cost; }
  }
  return best;
}

// Into how many ranges the router's forward GEMM cuts its contraction over d: with few experts
// the [T, E] logits are fewer tiles than the chip has CUs, so each tile's k loop is shared out.
// The same cost model as above, in pairs of k-tiles (a range is a whole number of pairs).
int router_fwd_splits(int T, int d, int E) {
  const long long tiles = (long long)((T + BM - 1) / BM) * ((E + BN - 1) / BN);
  const int cus = device_cu_count();
  const int pairs = d / (2 * BK);
  int best = 1;
  long long best_cost = -1;
  for (int s = 1; s <= 8 && s <= pairs / 4; ++s) {
    const long long rounds = (tiles * s + cus - 1) / cus;
    const long long cost = rounds * (2 * ((pairs + s - 1) / s) + SPLIT_OVERHEAD_KTILES);
    if (best_cost < 0 || cost < best_cost) { best = s; best_cost = cost; }
  }
  // no empty range: as many ranges as the rounded-up range length needs
  const int per = (pairs + best - 1) / best;
  return (pairs + per - 1) / per;
}

// partials: fp32 [splits, T, E] when the contraction is cut (splits > 1), else unused; the caller adds them up
int launch_router_fwd_bf16(const void* x, const void* wr, int T, int d, int E, float* logits, float* partials,
                           int splits, int32_t* sched, hipStream_t s) {
  if (T == 0) return MOE_OK;
  hipLaunchKernelGGL(zero_words, dim3(1), dim3(64), 0, s, sched, 8);
  HIP_CHECK_LAUNCH();
  GArgs g = {};
  g.A0 = g.A1 = (const bf16_t*)x; g.lda = d;
  g.B0 = g.B1 = (const bf16_t*)wr; g.ldb = E; g.b_es = 0;
  g.F0 = splits > 1 ? partials : logits; g.ldc = E; g.c_es = (long)T * E;
  g.off = nullptr; g.rows = T; g.chunk = T; g.sched = sched; g.e_cnt = 1; g.N = E;
  const int pairs = d / (2 * BK);
  g.ksplit = splits; g.k_total = d; g.K = splits > 1 ? (pairs + splits - 1) / splits * 2 * BK : d;
  return launch_gg<RL>(g, s);
}

int launch_router_dw_bf16(const void* x, const void* dl_bf16, int T, int d, int E, float* partials, int splits,
                          int32_t* sched, hipStream_t s) {
  GArgs g = {};
  g.A0 = g.A1 = (const bf16_t*)x; g.lda = d;
  g.B0 = g.B1 = (const bf16_t*)dl_bf16; g.ldb = E;
  g.F0 = partials; g.ldc = E; g.c_es = (long)d * E;
  g.off = nullptr; g.rows = T; g.chunk = (((T + splits - 1) / splits + BK - 1) / BK) * BK;
  g.sched = sched; g.e_cnt = splits; g.M = d; g.N = E;
  return launch_gg<RW>(g, s);
}

int launch_router_dx_bf16(const void* dl_bf16, const void* wr, int T, int d, int E, void* dx, int accumulate,
                          int32_t* sched, hipStream_t s) {
  GArgs g = {};
  g.A0 = g.A1 = (const bf16_t*)dl_bf16; g.lda = E;
  g.B0 = g.B1 = (const bf16_t*)wr; g.ldb = E; g.b_es = 0;
  g.C0 = (bf16_t*)dx; g.ldc = d;
  g.off = nullptr; g.rows = T; g.chunk = T; g.sched = sched; g.e_cnt = 1; g.N = d; g.K = E; g.accumulate = accumulate;
  return launch_gg<RX>(g, s);
}

// fp32 partial tiles for weight gradients cut along the rows: room for up to 32 pieces of the
// larger (two-output) gradient, at most 512 MB
size_t wgrad_split_bytes(int d, int f) {
  const size_t piece = 2 * (size_t)d * f * 4;
  size_t b = 32 * piece;
  const size_t cap = (size_t)512 << 20;
  if (b > cap) b = cap / piece * piece;
  return b;
}
size_t expert_bwd_extra_ws_bytes(int d, int f) { return 256 + WGRAD_PLAN_BYTES + wgrad_split_bytes(d, f); }
