// Few-token GEMM on 4-bit normal-float weights: out[M, N] = x w^T for M <= 256 stacked tokens, w = bf16(level[code] * max), for
// projections with many weights (which: gemm_codes_plan; the others look their codes up in gemm_bf16_kernel).
//
// What bounds it: the look-up (three vector instructions and an LDS read per weight), the matrix instructions and, where the runs
// are short, the partial sums.  gemm_bf16_kernel looks every weight up once per 128 tokens and puts it into LDS, in turn with its
// matrix instructions; here
//   * a wave owns 32 of a tile's 256 features for all tokens, so a weight is looked up once, straight into the fragment registers
//     of the wave that multiplies with it, and no dequantised weight goes through LDS;
//   * the look-up of the next K-step stands between the matrix instructions of this one (written out: the compiler reads, waits
//     and multiplies in turn);
//   * the list of (feature tile, K-tile) pairs is dealt to at most one persistent block per CU (three quarters of them where that ends
//     runs with their tiles) in equal runs, as in gemm_stream.hip, and the raw sums go to the same reductions.
// 7B shape, 192 tokens, in the model: gate and up 92 -> 61 us (their reduction 7.5 -> 12.6), Q|K|V 58 -> 45 (5.9 -> 9.1); two blocks
// over 192 tokens 508 -> 454 us.  Of whole runs from 32 to 128 K-tiles a K-tile takes a CU 1.1 / 1.3 / 1.6 / 2.0 us (64 / 128 / 192 / 256 tokens; its
// matrix instructions 0.25 to 1.0), the rest of the launch with the partial sums and their reduction 15 / 20 / 22 / 31; a block that ends one
// tile and begins the next stores two partial sums and ends some 8 us later.
#include "gemm_tile.h"
#include "fetch.h"
#include <type_traits>

namespace mpz {
namespace {

// the level of code number e of a word: a word of LDS (sixteen words lie in sixteen banks)
__device__ __forceinline__ float nf4_level_of(uint32_t c, int e, const float* level) { return level[(c >> (4 * e)) & 15u]; }
__device__ __forceinline__ uint32_t nf4_pair(float lo, float hi, float am) { return pack_bf16x2(__fmul_rn(lo, am), __fmul_rn(hi, am)); }
// eight codes of a row -> the fragment of a K-step: the level times the block maximum, rounded once
__device__ __forceinline__ u32x4 nf4_frag(uint32_t c, float am, const float* level) {
  u32x4 r;
#pragma unroll
  for (int p = 0; p < 4; ++p) r[p] = nf4_pair(nf4_level_of(c, 2 * p, level), nf4_level_of(c, 2 * p + 1, level), am);
  return r;
}

// One wave instruction fetches 64 words, one per lane, into 256 bytes of LDS
__device__ __forceinline__ void fetch_words(i32x4 rsrc, uint32_t voff, uint32_t soff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %3\n\ts_nop 4\n\tbuffer_load_dword %0, %1, %2 offen lds" ::"v"(voff), "s"(rsrc), "s"(soff), "s"(lds) : "memory");
}

// One K-step of 32: the fragments `now` times NJ token tiles, and between the matrix instructions the look-up of the fragments
// `next` from the codes c.  The order is written out (and pinned): left to itself the compiler reads, waits and multiplies in turn.
template <int NJ, typename Fetch>
__device__ __forceinline__ void codes_phase(f32x4 (&acc)[2][NJ], const u32x4 (&now)[2], const unsigned char* px, u32x4 (&next)[2],
                                            const uint32_t (&c)[2], const float (&am)[2], const float* level, Fetch&& fetch) {
  constexpr int LAG = NJ >= 8 ? 2 : 1, AHEAD = 3;
  bf16x8 fx[AHEAD + 1];
  float lo[8], hi[8];
#pragma unroll
  for (int j = 0; j < AHEAD; ++j) fx[j] = as_frag(*(const u32x4*)(px + j * 2048));
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    if (j + AHEAD < NJ) fx[(j + AHEAD) % (AHEAD + 1)] = as_frag(*(const u32x4*)(px + (j + AHEAD) * 2048));
    acc[0][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_frag(now[0]), fx[j % (AHEAD + 1)], acc[0][j], 0, 0, 0);
#pragma unroll
    for (int p = 0; p < 8; ++p)
      if (p * (NJ - LAG) / 8 == j) {                     // pair p of the sixteen codes: its two levels are requested
        lo[p] = nf4_level_of(c[p / 4], p % 4 * 2, level);
        hi[p] = nf4_level_of(c[p / 4], p % 4 * 2 + 1, level);
      }
    __builtin_amdgcn_sched_barrier(0);
    acc[1][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_frag(now[1]), fx[j % (AHEAD + 1)], acc[1][j], 0, 0, 0);
#pragma unroll
    for (int p = 0; p < 8; ++p)
      if (p * (NJ - LAG) / 8 + LAG == j) next[p / 4][p % 4] = nf4_pair(lo[p], hi[p], am[p / 4]);
    __builtin_amdgcn_sched_barrier(0);
    fetch(j);
    __builtin_amdgcn_sched_barrier(0);
  }
}


// Per-copy low-rank term of the wave's 32 features: [B_hi | B_lo] of a copy against the bottleneck activations [t | t], the operands
// of 64 tokens requested together.  Copies are whole multiples of 32 rows, segments of 128 columns.
template <int NJ>
__device__ __forceinline__ void codes_low_rank(const MfmaGemmArgs& a, f32x4 (&acc)[2][NJ], int nw, int lane) {
  const int l16 = lane & 15, lq = lane >> 4;
  const u32x4 zero = {0u, 0u, 0u, 0u};
  for (int s = 0; s < a.n_seg; ++s) {
    const MfmaLoraSeg& sg = a.seg[s];
    if (nw < sg.col_begin || nw >= sg.col_end) continue;
    for (int ks = 0; ks < sg.rp; ks += 32) {
      const bool here = ks + lq * 8 < sg.rp;             // (rank <= 8: the upper half of the K-step is zero)
      const int k8 = here ? ks + lq * 8 : 0;
#pragma unroll
      for (int j0 = 0; j0 < NJ; j0 += 4) {
        u32x4 x[4], w[2][2];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          int m = (j0 + j) * 16;
          m = m < a.M ? m : 0;                           // tokens past the end: their sums are not stored
          x[j] = *(const u32x4*)((const uint16_t*)sg.tp + (size_t)(m + l16) * sg.rp + k8);
          if (j % 2 == 0) {
            const uint16_t* bp = (const uint16_t*)sg.bp + (size_t)(m / a.rows_per_copy) * sg.copy_stride + k8;
#pragma unroll
            for (int i = 0; i < 2; ++i) w[j / 2][i] = *(const u32x4*)(bp + (size_t)(nw + i * 16 + l16 - sg.col_begin) * sg.rp);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int i = 0; i < 2; ++i)
            acc[i][j0 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_frag(here ? w[j / 2][i] : zero), as_frag(here ? x[j] : zero), acc[i][j0 + j], 0, 0, 0);
      }
    }
  }
}

template <int BM, int SX, int SC>
__global__ void __launch_bounds__(512, 1) gemm_codes_kernel(MfmaGemmArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ __align__(128) float level[32];
  constexpr int BN = kCodesTile, NJ = BM / 16, FX = BM / 32;         // (fetches of x of a wave per K-tile)
  constexpr uint32_t XSTAGE = BM * 128, CSTAGE = 8192 + 1024, CODES = SX * XSTAGE;   // x rows; codes, then block maxima
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, lq = lane >> 4;
  const int nk = a.K / 64, U = a.stream_units;
  const int units = (a.N + BN - 1) / BN * nk;
  const int u0 = blockIdx.x * U, u1 = u0 + U < units ? u0 + U : units;
  const size_t row_b = (size_t)a.K * 2, row_c = (size_t)a.K / 2, row_a = (size_t)nk * 4;
  // Waves 0-3 fetch x, waves 4-7 codes and block maxima: a wave's fetches land in order, and those of x (in L2) would wait for the
  // codes (from memory) requested before them.
  const bool codes_wave = wave >= 4;
  const int w4 = wave & 3;
  uint32_t voff[2];                                      // of the first two fetches of x; the others are 16, 32, .. rows further down
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int r = codes_wave ? (w4 * 2 + t) * 32 + (lane >> 1) : (w4 * FX + t) * 8 + (lane >> 3);
    voff[t] = codes_wave ? (uint32_t)r * (uint32_t)row_c + (lane & 1) * 16
                         : (uint32_t)r * (uint32_t)row_b + (uint32_t)(((lane & 7) ^ ((r >> 1) & 7)) * 16);
  }
  const uint32_t voffA = (uint32_t)(w4 * 64 + lane) * (uint32_t)row_a;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  // The wave's stream of requests, in the order of the block's units; past the last unit it repeats that one, so that the count of
  // fetches in flight is the same everywhere.  Everything is carried along: divisions per K-tile cost 10 % of the kernel.
  const uint32_t first = codes_wave ? lds0 + CODES : lds0, size = codes_wave ? CSTAGE : XSTAGE;
  const uint32_t end = first + (codes_wave ? SC : SX) * size;
  int left = u1 - 1 - u0, kt_f = u0 % nk, rows = a.w_rows - u0 / nk * BN;
  uint32_t at = first;                                   // stage that the next request goes to
  const char* tile_c = (const char*)a.w + (size_t)(u0 / nk) * BN * row_c;
  const char* tile_a = (const char*)a.w_absmax + (size_t)(u0 / nk) * BN * row_a;
  auto records = [&](size_t row) { return (size_t)(rows < BN ? rows : BN) * row; };
  i32x4 rsrc = codes_wave ? buffer_of(tile_c, records(row_c)) : buffer_of(a.x, (size_t)a.M * row_b);
  i32x4 rsrcA = buffer_of(tile_a, records(row_a));
  auto fetch = [&] {
    if (codes_wave) {
#pragma unroll
      for (int t = 0; t < 2; ++t) fetch_rows<4>(rsrc, voff[t], (uint32_t)kt_f * 32u, at + (uint32_t)(w4 * 2 + t) * 1024u);
      fetch_words(rsrcA, voffA, (uint32_t)kt_f * 4u, at + 8192u + (uint32_t)w4 * 256u);
    } else {
#pragma unroll
      for (int t = 0; t < FX; ++t) fetch_rows<4>(rsrc, voff[t & 1], (uint32_t)kt_f * 128u + (uint32_t)(t / 2 * 16) * (uint32_t)row_b, at + (uint32_t)(w4 * FX + t) * 1024u);
    }
    at = at + size == end ? first : at + size;
    if (left > 0) {
      --left;
      if (++kt_f == nk) {
        kt_f = 0;
        if (codes_wave) {
          rows -= BN; tile_c += BN * row_c; tile_a += BN * row_a;
          rsrc = buffer_of(tile_c, records(row_c)); rsrcA = buffer_of(tile_a, records(row_a));
        }
      }
    }
  };
  if (tid < 16) {
    constexpr float kLevel[16] = {-1.0f, -0.6961928009986877f, -0.5250730514526367f, -0.39491748809814453f,
                                  -0.28444138169288635f, -0.18477343022823334f, -0.09105003625154495f, 0.0f,
                                  0.07958029955625534f, 0.16093020141124725f, 0.24611230194568634f,
                                  0.33791524171829224f, 0.44070982933044434f, 0.5626170039176941f,
                                  0.7229568362236023f, 1.0f};
    level[tid] = kLevel[tid];
  }
  __syncthreads();

  f32x4 acc[2][NJ];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const uint32_t baseX = (uint32_t)l16 * 128u + (uint32_t)(lq ^ ((l16 >> 1) & 7)) * 16u;
  const uint32_t baseC = CODES + (uint32_t)(wave * 32 + l16) * 32u + (uint32_t)lq * 4u;
  const uint32_t baseA = CODES + 8192u + (uint32_t)(wave * 32 + l16) * 4u;

  int xs = 0, cs = 0, kt = kt_f, tile = u0 / nk;         // stages, K-tile and tile of unit u
  // FX fetches a K-tile of x, three of codes: all but the `ahead` youngest K-tiles' have landed, for the block
  auto landed = [&](auto x_ahead, auto c_ahead) {
    if (codes_wave) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(c_ahead)::value * 3) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(x_ahead)::value * FX) : "memory");
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  };
  for (int t = 0; t < (codes_wave ? SC : SX) - 1; ++t) fetch();
  landed(std::integral_constant<int, SX - 1>{}, std::integral_constant<int, SC - 2>{});      // the first unit's codes
  uint32_t c0[2], c1[2];
  float am[2], am_next[2];
  u32x4 fw0[2], fw1[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    am[i] = *(const float*)(smem + baseA + i * 64);
    fw0[i] = nf4_frag(*(const uint32_t*)(smem + baseC + i * 512), am[i], level);
  }
  for (int u = u0; u < u1; ++u) {
    // x of this unit and the codes of the next one have landed; behind the barrier every wave is done with the stages that the
    // next fetches overwrite
    landed(std::integral_constant<int, SX - 2>{}, std::integral_constant<int, SC - 3>{});
    const unsigned char* px = smem + (uint32_t)xs * XSTAGE;
    const unsigned char* pc = smem + (uint32_t)cs * CSTAGE;
    xs = xs + 1 == SX ? 0 : xs + 1;
    cs = cs + 1 == SC ? 0 : cs + 1;
    const unsigned char* pn = smem + (uint32_t)cs * CSTAGE;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      c1[i] = *(const uint32_t*)(pc + baseC + i * 512 + 16);
      c0[i] = *(const uint32_t*)(pn + baseC + i * 512);
      am_next[i] = *(const float*)(pn + baseA + i * 64);
    }
    __builtin_amdgcn_sched_barrier(0);
    codes_phase<NJ>(acc, fw0, px + baseX, fw1, c1, am, level, [&](int j) {
      if (j == 1) fetch();
    });
    codes_phase<NJ>(acc, fw1, px + (baseX ^ 64u), fw0, c0, am_next, level, [](int) {});
    am[0] = am_next[0]; am[1] = am_next[1];
    if (u + 1 == u1 || kt + 1 == nk) {                   // the block's part of this tile ends here
      const int nw = tile * BN + wave * 32, first_u = tile * nk;
      if (u0 <= first_u) codes_low_rank<NJ>(a, acc, nw, lane);   // the block that began the tile adds the low-rank term
      // (tokens past M fall outside the buffer, features past N are aimed outside: 256 rows stay below 2^31 bytes, codes_supported)
      const int slot = (int)blockIdx.x - first_u / U;
      const uint32_t row_p = (uint32_t)a.ldp * 4u;
      const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(a.partial + (size_t)slot * a.M * a.ldp, 0, (int)((uint32_t)a.M * row_p), 0x00020000);
      int off[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int n = nw + i * 16 + lq * 4;
        off[i] = n < a.N ? (int)(l16 * row_p + n * 4u) : (int)0x80000000;
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i)
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[i][j]), out, off[i] + (int)(j * 16 * row_p), 0, 0);   // (no scalar offset: fetch.h)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[0][j] = acc[1][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      ++tile;
    }
    kt = kt + 1 == nk ? 0 : kt + 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // (the repeated requests: LDS is the block's until they have landed)
}

template <int BM, int SX, int SC>
hipError_t launch_codes(hipStream_t st, const MfmaGemmArgs& a, int grid) {
  static_assert(SC >= 4, "the next unit's codes land with this unit's x");
  constexpr size_t lds = (size_t)SX * BM * 128 + (size_t)SC * 9216;
  static_assert(lds + 128 <= 160 * 1024, "one block per CU");
  static const hipError_t attr_status = hipFuncSetAttribute((const void*)gemm_codes_kernel<BM, SX, SC>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (attr_status != hipSuccess) return attr_status;
  gemm_codes_kernel<BM, SX, SC><<<grid, 512, lds, st>>>(a);
  return hipSuccess;
}

// (gate and up come as one product over their 2 N rows)
bool codes_supported(const MfmaGemmArgs& a) {
  return !a.dual && a.w_absmax != nullptr && a.M <= 256 && a.K % 64 == 0 && a.N % 4 == 0 && a.N < 1 << 20 && fetch_aligned(a);
}

// K-tiles per block: equal runs for 256 CUs, of at least four; 0 = the partial sums would not fit `capacity` floats
int codes_units(const MfmaGemmArgs& a, size_t capacity) {
  const int nk = a.K / 64;
  const long units = (long)((a.N + kCodesTile - 1) / kCodesTile) * nk;
  long U = (units + 255) / 256;
  U = U < 4 ? 4 : U;
  // runs a third longer that end with their tiles leave a quarter fewer partial sums
  for (long V = U; 3 * V <= 4 * U && V <= nk; ++V)
    if (nk % V == 0) { U = V; break; }
  while (U < nk && (size_t)stream_slots(nk, (int)U) * a.M * a.N > capacity) ++U;
  return (size_t)stream_slots(nk, (int)U) * a.M * a.N <= capacity ? (int)U : 0;
}

// Are runs of U K-tiles faster than shares of K in `share_blocks` blocks (two per CU) of gemm_bf16_kernel, which looks every code up once per
// 128 tokens?  A run pays its partial sum of 256 features, 16 KB per 16 tokens, and the start of the stream with the look-ups it saves: those
// of the second 128 tokens, and below that only what the look-up in the fragment registers saves.  Runs that do not end with their
// tiles store more of them (see above), and shares that fill their rounds are at their best.  Shares / here, 64, 128, 192, 256 tokens:
// whole runs of 8: 0.82 - 0.95, 0.83 - 0.98, 0.77 - 0.91, 0.75 - 0.84; 12: 0.92 - 0.93, 0.95 - 0.99, 1.09 - 1.13, 0.89 - 0.99; 14 to 17: 0.87 - 0.98, 0.93 - 1.03,
// 1.08 - 1.19, 0.97 - 1.09; 18 to 24: 0.98 - 1.01, 1.03 - 1.06, 1.19 - 1.23, 1.07 - 1.12; 32 and more: 1.01 - 1.11, 1.03 - 1.15, 1.45 - 1.53, 1.29 - 1.35.
// Runs that cross tiles, against full shares: 11 to 13: 0.85 - 0.89, 0.86 - 0.90, 0.94 - 1.11, 0.74 - 0.91; 17: 0.89, 0.93, 1.09, 0.95; 21: 0.91, 0.97;
// against shares that leave CUs idle: 18 to 22: 1.00 - 1.16, 0.99 - 1.11, 1.20 - 1.56, 1.06 - 1.33.
bool codes_pay(const MfmaGemmArgs& a, int U, long share_blocks) {
  const int nk = a.K / 64;
  const long units = (long)((a.N + kCodesTile - 1) / kCodesTile) * nk;
  if (units <= 191L * U || U < (a.M <= 128 ? 18 : a.M <= 192 ? 12 : 14)) return false;       // (fewer blocks: only little room makes them)
  const bool idle = share_blocks * 16 <= (share_blocks + 511) / 512 * 512 * 15;
  return nk % U == 0 || idle || (a.M > 128 && a.M <= 192) || U >= (a.M <= 128 ? 32 : 18);
}

}  // namespace

int gemm_codes_plan(const MfmaGemmArgs& a, size_t capacity, bool forced) {
  if (!codes_supported(a)) return 0;
  const int U = codes_units(a, capacity);
  return U > 0 && (forced || codes_pay(a, U, mfma_gemm_split_blocks(a, capacity))) ? U : 0;
}

hipError_t launch_gemm_codes(hipStream_t st, const MfmaGemmArgs& a) {
  const long units = (long)((a.N + kCodesTile - 1) / kCodesTile) * (a.K / 64);
  const int grid = (int)((units + a.stream_units - 1) / a.stream_units);
  if (a.M <= 64) return launch_codes<64, 6, 8>(st, a, grid);
  if (a.M <= 128) return launch_codes<128, 4, 8>(st, a, grid);
  if (a.M <= 192) return launch_codes<192, 3, 8>(st, a, grid);
  return launch_codes<256, 3, 6>(st, a, grid);
}

}  // namespace mpz
