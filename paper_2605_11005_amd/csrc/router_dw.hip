// Weight gradient of the trainable router, dWr = x^T dlogits, in bf16 for 32 to 256 experts: a stream over x.
//
// Bound by reading x once (T d 2 bytes).  A block owns 128 columns of x, all experts and a range of tokens; its four wavefronts
// hold 64 columns by half of the experts each as 32x32 blocks of sums.  Pieces of 32 tokens pass through a ring in LDS, four to
// eight of them, so that 30 to 56 KB of x per CU are on their way: x in its own layout, read by the transposing LDS reads, the
// dlogits as router_dl_operands lays them out, tokens contiguous.  The fp32 sums of a range go to memory and reduce_chunks adds
// them up; one block per CU keeps those few.
//
// A chain of matrix instructions does not round to nearest: its error grows with its length, and faster than that of additions.  So a
// range is summed in several chains, added up in fp32, as many as leave no shape further off than the kernels that had it before, and
// the chain of the dlogits' first terms is free of the others (E = 160, whose registers do not hold both, is exact enough without).
// Error of dWr against 64 bits before it is rounded to bf16, of sqrt(T) times the operands' size (rms, 1e-8; exact sums of zero): the
// kernels before / one chain per range / now:
//   T = 16384, d = 4096, E = 128  13.4 / 25.9 / 12.1    T = 16384, d = 512, E = 64   9.2 / 18.4 / 9.1     T = 8192, d = 1024, E = 32    9.9 / 18.4 / 8.8
//   T = 9001, d = 2880, E = 128   9.7 / 15.9 / 9.0      T = 9001, d = 2880, E = 64   8.5 / 16.0 / 8.5     T = 30000, d = 7168, E = 32   35.9 / 100 / 20.9
//   T = 3000, d = 4096, E = 128   7.3 / 10.4 / 7.0      T = 16384, d = 4096, E = 192  18.4 / 25.9 / 15.0  T = 8192, d = 2048, E = 96    38.0 / 30.3 / 11.8
//   T = 9001, d = 2880, E = 256   12.3 / 15.9 / 10.0    T = 2000, d = 4096, E = 256  7.1 / 8.5 / 7.1      T = 8192, d = 2048, E = 160   45.4 / 41.4 / 41.4
// It costs up to 3 us (E = 256, T = 9001, d = 2880 50.5 -> 53.6); E = 32, 96 and 160 nothing or 1.
#include "common.h"
#include "kernels.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int NT = 256, COLS = 128, PIECE = 32;

// NE: experts / 32; PLANES: terms per dlogit (1: rounded to bf16, 3: their sum keeps all 24 bits)
template <int NE, int PLANES> struct Shape {
  static constexpr int E = 32 * NE;
  static constexpr int X_BYTES = COLS * PIECE * 2, STAGE = X_BYTES + PLANES * E * PIECE * 2;
  static constexpr int STAGES = 155 * 1024 / STAGE < 8 ? 155 * 1024 / STAGE : 8;
  static constexpr int DL_LOADS = PLANES * E / 16, PER_WAVE = (DL_LOADS + 3) / 4, LOADS = 2 + PER_WAVE;      // of 1 KB, per stage
  static constexpr int BLOCKS = (NE + 1) / 2;       // of 32 experts, per wavefront
  static constexpr int PARTS = PLANES > 1 && NE < 5 ? 2 : 1;       // chains at a time: of the first plane, of the others
  static constexpr int CHAINS = NE <= 2 ? 8 : NE == 3 ? 2 : NE == 4 ? 5 : NE == 5 ? 1 : 3;      // one after the other in a range
  static_assert((STAGES - 2) * LOADS < 64 && STAGES >= 3, "the wait counter holds 63");
};

// 32 columns from n on of the [32 tokens][64 columns] tile at p, k-step s of 16 tokens; chunk' = chunk ^ (4*((token>>1)&1))
__device__ __forceinline__ bf16x8 x_fragment(const char* p, int n, int s, int lane) {
  const int i = lane & 15, g = lane >> 4;
  const int t = 8 * (g >> 1) + (i >> 2), c = n + 16 * (g & 1) + 4 * (i & 3);
  const char* q = p + s * 2048 + t * 128 + (((c >> 3) ^ (4 * ((t >> 1) & 1))) << 4) + ((c & 4) << 1);
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)q);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(q + 512));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// (64 and 96 experts: bounds that leave the sums no accumulation registers, which an addition cannot read: E = 96 38.2 -> 37.2 us, T = 8192,
// d = 2048.  E = 32 is 7 to 11 % faster with them.)
template <int NE, int PLANES>
__global__ __launch_bounds__(NT, NE == 2 || NE == 3 ? 2 : 1) void router_dw_stream(const bf16_t* __restrict__ x, const bf16_t* __restrict__ dl,
                                                         const float* __restrict__ dlogits, float* __restrict__ sums, int T, int d,
                                                         int n_cols, int per_range) {
  using S = Shape<NE, PLANES>;
  extern __shared__ __align__(16) char lds[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wc = wave >> 1, we = wave & 1;
  const int range = blockIdx.x / n_cols, c0 = (blockIdx.x - range * n_cols) * COLS;
  const int first = range * per_range, n = min(per_range, (T + PIECE - 1) / PIECE - first);       // pieces
  const uint32_t base = lds_addr(lds);

  // stage s: piece first + s, in place s % STAGES; past the end the last piece again, so that the number of loads stays the same
  auto issue = [&](int s) {
    const int piece = first + min(s, n - 1), t0 = min(piece * PIECE, T - PIECE);      // (the last piece ends at the last token)
    const uint32_t at = base + s % S::STAGES * S::STAGE;
#pragma unroll
    for (int j = 0; j < 2; ++j) {         // 8 tokens of 64 columns
      const int id = 2 * wave + j, t = 8 * (id & 3) + (lane >> 3), chunk = (lane & 7) ^ (4 * ((lane >> 4) & 1));
      const int c = min(c0 + 64 * (id >> 2) + 8 * chunk, d - 8);
      lds_load16(x + (size_t)t0 * d, (uint32_t)((t * d + c) * 2), at + id * 1024);
    }
#pragma unroll
    for (int j = 0; j < S::PER_WAVE; ++j) {      // 16 experts of a plane: chunk' = chunk ^ ((expert>>2)&3)
      const int id = min(wave * S::PER_WAVE + j, S::DL_LOADS - 1);
      lds_load16(dl + (size_t)piece * PLANES * S::E * PIECE, (uint32_t)(id * 1024 + (lane >> 2) * 64 + (((lane & 3) ^ ((lane >> 4) & 3)) << 4)),
                 at + S::X_BYTES + id * 1024);
    }
  };
  f32x16 acc[S::PARTS][2][S::BLOCKS], total[2][S::BLOCKS];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int b = 0; b < S::BLOCKS; ++b) {
      total[m][b] = f32x16{};
      acc[S::PARTS - 1][m][b] = f32x16{};
    }
  int expert[S::BLOCKS];                  // of this lane; past the last one it again (never stored)
#pragma unroll
  for (int b = 0; b < S::BLOCKS; ++b) expert[b] = min((we * S::BLOCKS + b) * 32 + (lane & 31), S::E - 1);

#pragma unroll
  for (int s = 0; s < S::STAGES - 1; ++s) issue(s);
  const int per_chain = max(2, (n + S::CHAINS - 1) / S::CHAINS);
  for (int chain = 0; chain < n; chain += per_chain) {
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int b = 0; b < S::BLOCKS; ++b) acc[0][m][b] = f32x16{};
    for (int s = chain; s < min(n, chain + per_chain); ++s) {
      // stage s has landed once those after it are all that is on its way; and everyone is done with the one whose place is filled next
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"((S::STAGES - 2) * S::LOADS) : "memory");
      __builtin_amdgcn_s_barrier();
      issue(s + S::STAGES - 1);
      const char* const stage = lds + s % S::STAGES * S::STAGE;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const bf16x8 f0 = x_fragment(stage + wc * 4096, 0, k, lane), f1 = x_fragment(stage + wc * 4096, 32, k, lane);
#pragma unroll
        for (int p = 0; p < PLANES; ++p)
#pragma unroll
          for (int b = 0; b < S::BLOCKS; ++b) {
            const int row = p * S::E + expert[b], h = p < S::PARTS ? p : S::PARTS - 1;
            const bf16x8 g = *reinterpret_cast<const bf16x8*>(stage + S::X_BYTES + row * 64 + (((2 * k + (lane >> 5)) ^ ((row >> 2) & 3)) << 4));
            acc[h][0][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f0, g, acc[h][0][b], 0, 0, 0);
            acc[h][1][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f1, g, acc[h][1][b], 0, 0, 0);
          }
      }
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int b = 0; b < S::BLOCKS; ++b) total[m][b] += acc[0][m][b];
  }
  if (S::PARTS > 1)
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int b = 0; b < S::BLOCKS; ++b) total[m][b] += acc[S::PARTS - 1][m][b];
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  float* const out = sums + (size_t)range * d * S::E;
  float probe = 0.f;
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    const int col = c0 + 64 * wc + 32 * m + 4 * (lane >> 5);
    if (col >= d) continue;               // d % 64 == 0: 32 columns at a time
#pragma unroll
    for (int b = 0; b < S::BLOCKS; ++b) {
      const int e = (we * S::BLOCKS + b) * 32 + (lane & 31);
      if (e >= S::E) continue;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        out[(size_t)(col + 8 * (r >> 2) + (r & 3)) * S::E + e] = PLANES == 1 ? total[m][b][r] : total[m][b][r] * DL_UNSCALE;
        probe += total[m][b][r] * 0.f;
      }
    }
  }
  if (probe == 0.f) return;
  // Zeros that stand for no product, a dlogit's empty terms and the overlap of the last piece, make NaN of an infinite x, and an
  // infinite dlogit's terms are no sum.  Sums that are no numbers are formed again, in plain fp32, where that can be the reason.
  if (PLANES == 1 && (T % PIECE == 0 || (first + n) * PIECE < T)) return;
  const int end = min(T, (first + n) * PIECE);
#pragma unroll 1
  for (int i = 0; i < 2 * S::BLOCKS * 16; ++i) {
    const int r = i % 16, col = c0 + 64 * wc + 32 * (i / (S::BLOCKS * 16)) + 4 * (lane >> 5) + 8 * (r >> 2) + (r & 3);
    const int e = (we * S::BLOCKS + i / 16 % S::BLOCKS) * 32 + (lane & 31);
    if (col >= d || e >= S::E) continue;
    const size_t at = (size_t)col * S::E + e;
    if (fabsf(out[at]) < INFINITY) continue;
    float sum = 0.f;
    for (int t0 = first * PIECE; t0 < end && sum == sum; t0 += 8) {
      float a[8], g[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const size_t t = min(t0 + k, end - 1);
        a[k] = bf16_to_f32(x[t * d + col]);
        g[k] = dlogits[t * S::E + e];
        if (PLANES == 1) g[k] = bf16lo(pack_bf16x2(g[k], 0.f));
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) sum += t0 + k < end ? a[k] * g[k] : 0.f;
    }
    out[at] = sum;
  }
}

template <int NE, int PLANES>
int launch(const bf16_t* x, const bf16_t* dl, const float* dlogits, float* sums, int T, int d, int ranges, hipStream_t s) {
  using S = Shape<NE, PLANES>;
  constexpr int LDS = S::STAGES * S::STAGE;
  static bool attr_set[64] = {};         // a per-device attribute of the kernel
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MOE_EHIP;
  if (!attr_set[dev]) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&router_dw_stream<NE, PLANES>), hipFuncAttributeMaxDynamicSharedMemorySize,
                            LDS) != hipSuccess)
      return MOE_EHIP;
    attr_set[dev] = true;
  }
  const int n_cols = (d + COLS - 1) / COLS, per = ((T + PIECE - 1) / PIECE + ranges - 1) / ranges;
  ProfScope prof(MOE_K_ROUTER_DW, s);
  hipLaunchKernelGGL((router_dw_stream<NE, PLANES>), dim3((unsigned)(ranges * n_cols)), dim3(NT), LDS, s, x, dl, dlogits, sums, T, d,
                     n_cols, per);
  HIP_CHECK_LAUNCH();
  return MOE_OK;
}

}  // namespace

// Into how many ranges of tokens, one sum each, the weight gradient of a shape is cut here with room for max_sums of them; 0: other
// kernels are faster, or there is no room.  splits: of the product that takes the shape otherwise.  Weight gradient alone (operands,
// product, reduction), us, the streaming kernel of few rows (E = 32, 64 and, up to T d = 2^26, 128), big tiles (E = 128 beyond, 192, 256) or
// plain fp32 products (E = 96, 160) / this one:
//   T = 16384, d = 4096, E = 128  61 / 46     T = 9001, d = 2880, E = 128  37 / 35       T = 4096, d = 2048, E = 64    19.0 / 17.5
//   T = 8192, d = 2048, E = 32    32 / 25     T = 30000, d = 7168, E = 32  229 / 132     T = 8192, d = 2048, E = 96    113 / 37
//   T = 2000, d = 4096, E = 256   53 / 40     T = 9000, d = 7168, E = 256  76 / 72       T = 16384, d = 7168, E = 256  103 / 114
// Small x are the others' (their sums are fewer; E = 128, T = 2048, d = 4096 25.3 / 26.0, 4096, 2048 26.1 / 25.9, 6000, 2048 29.7 / 29.0; E = 96,
// T = 100, d = 2048 12.4 / 13.2, 1000, 256 16.7 / 15.2; E = 160, T = 1000, d = 256 17.1 / 18.0, 3000, 128 27.7 / 23.2), 192 and more experts of a
// large x the big tiles', which read the dlogits half as often per column.
// A block per CU, but at least 12 pieces in a range (8 for E = 32; 4 for E = 96 and 160, whose alternative is slow): every range is one more
// sum to write and read.  4 / 8 / 12 / 16 pieces: T = 4096, d = 1024, E = 64 20.1 / 17.1 / 16.1 / 16.0; 2048, 2048, E = 256 40.7 / 39.4 / 38.0 /
// 38.5; 4096, 1024, E = 32 21.2 / 17.1 / 17.4 / 18.0, 1024, 4096, E = 32 13.6 / 13.3 / 15.7 / 15.7; 512, 2048, E = 160 20.5 / 23 / 28.6 / 28.6.
// Where T is large beside d the operand takes the room of the sums.  Few long ranges are slower than the big tiles' many, than the few
// rows' two blocks per range (E = 128) or eight wavefronts per block (E = 64), and than many more of plain products:
//   E = 128: T = 20000, d = 512 (12 ranges, tiles 32) 33.5 / 38     30000, 1024 (17) 46 / 41.5     70000, 1536 (9) 106 / 125
//   E = 192: T = 16384, d = 512 (16) 52 / 41    24000, 512 (8) 59.5 / 62    50000, 1024 (7) 87 / 115    E = 256: 60000, 1024 (2) 105 / 461
//   E = 64: T = 60000, d = 1536 (12) 58 / 53    24000, 512 (8) 33.4 / 36.1    60000, 1024 (2) 150 / 209
//   E = 96: T = 16384, d = 4096 (2, plain products 8) 409 / 176    E = 160: 12000, 4096 (1, 6) 457 / 347
//   E = 32: T = 20000, d = 512 (5, 64) 100 / 56    21000, 512 (2, 64) 77 / 120
// Two pieces per barrier were no faster (E = 256 slower).
int router_dw_ranges(int T, int d, int E, long long max_sums, int splits) {
  if (T < PIECE || d % 64 || max_sums < 1) return 0;
  const long long x = (long long)T * d;
  long long least = 1ll << 22, most = 1ll << 40;      // of T d
  int pieces_per_range = 12;
  double longer = 2.25;                               // as many pieces in a range as the alternative's, at most, where there is little room
  switch (E) {
    case 32: pieces_per_range = 8; longer = 14; break;
    case 64: longer = 2.75; break;
    case 96: least = 7 << 15; pieces_per_range = 4; longer = 9; break;
    case 128: least = (1 << 23) + 1; break;
    case 160: least = 5 << 16; pieces_per_range = 4; longer = 6; break;
    case 192: case 256: most = 1ll << 26; break;
    default: return 0;
  }
  if (x < least || x > most) return 0;
  const int n_cols = (d + COLS - 1) / COLS, pieces = (T + PIECE - 1) / PIECE;
  int ranges = device_cu_count() / n_cols;
  if (ranges > pieces / pieces_per_range) ranges = pieces / pieces_per_range;
  if (ranges > max_sums) {
    if (splits > longer * max_sums) return 0;
    ranges = (int)max_sums;
  }
  if (ranges < 1) ranges = 1;
  const int per = (pieces + ranges - 1) / ranges;
  return (pieces + per - 1) / per;
}
// dl: pieces of router_dl_operands, one plane where E % 64 == 0, three of 32, 96 or 160 experts, these times DL_SCALE; T >= 32.
// sums: [ranges][d][E]
int launch_router_dw_stream(const void* x, const void* dl, const float* dlogits, int T, int d, int E, float* sums, int ranges, hipStream_t s) {
  const bf16_t *a = (const bf16_t*)x, *b = (const bf16_t*)dl;
  switch (E / 32) {
    case 1: return launch<1, 3>(a, b, dlogits, sums, T, d, ranges, s);
    case 2: return launch<2, 1>(a, b, dlogits, sums, T, d, ranges, s);
    case 3: return launch<3, 3>(a, b, dlogits, sums, T, d, ranges, s);
    case 4: return launch<4, 1>(a, b, dlogits, sums, T, d, ranges, s);
    case 5: return launch<5, 3>(a, b, dlogits, sums, T, d, ranges, s);
    case 6: return launch<6, 1>(a, b, dlogits, sums, T, d, ranges, s);
    default: return launch<8, 1>(a, b, dlogits, sums, T, d, ranges, s);
  }
}
