// Few-token GEMM: out[M, N] = x w^T for M <= 256 stacked tokens, bf16 weights streamed once.
//
// What bounds it: the weight stream.  A kernel that only reads gets 5.2 TB/s from HBM on this chip; with about 2 us between a
// request and its data that takes some 40 KB in flight per CU, all the time and on all CUs:
//   * the work is the list of (128-feature tile, K-tile of 64) pairs, dealt to one persistent block per CU in equal
//     contiguous runs, so no CU has a round more than another, whatever N and K (a block's run may end one tile and begin
//     the next; a tile's sums come from as many blocks as its K-tiles fall on);
//   * the tiles are fetched straight into a ring of LDS stages, two to five K-tiles ahead, across the tile borders of a
//     run; one block barrier per K-tile;
//   * each block leaves the raw fp32 sums of its part of a tile in its slot of the partial buffer; the reduction kernels add
//     the slots of a tile in block order (deterministic) and apply the epilogue.
// Measured alone with cold weights, 128 tokens, features x K = 12288 x 4096 and 22016 x 4096: 28.5 and 46.8 us (3.5 and 3.9 TB/s;
// 33.5 and 52.3 with four waves instead of eight, 27 and 43 with neither activations nor matrix instructions).  Which shapes take
// it, and their times with the reduction against equal shares of K: plan_stream (mpz_api.hip).  Two 7B-shaped blocks over 128
// tokens: 343 us with these two projections streamed, 348 with all four.
#include "gemm_tile.h"
#include "fetch.h"

namespace mpz {
namespace {

// BM tokens (64, 128, 256: all of them), ST stages of 128 weight rows and BM token rows, eight waves (WGM along the tokens): two
// per SIMD, so that one's matrix instructions run under the other's wait, LDS reads and barrier
template <int BM, int ST, int WGM>
__global__ void __launch_bounds__(512, 1) gemm_stream_kernel(MfmaGemmArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int BN = 128, BK = 64;
  constexpr int WGN = 8 / WGM, NI = BN / WGN / 16, NJ = BM / WGM / 16;
  constexpr int FW = 2, FX = BM / 64, PER = FW + FX;     // fetches of a wave per K-tile: 8 rows of 128 bytes each
  constexpr uint32_t WBYTES = BN * BK * 2, STAGE = WBYTES + BM * BK * 2;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wvn = wave / WGM, wvm = wave % WGM, l16 = lane & 15, lq = lane >> 4;
  const int nk = a.K / BK, U = a.stream_units;
  const int units = (a.N + BN - 1) / BN * nk;
  const int u0 = blockIdx.x * U, u1 = u0 + U < units ? u0 + U : units;

  // byte offsets of this lane inside a tile's rows (buffers hold the tile's rows: rows past
  // N or M fall outside, what they accumulate is never stored); 16-byte chunks in the order c ^ ((row / 2) % 8)
  const size_t row_b = (size_t)a.K * 2;
  uint32_t voffW[FW], voffX[FX];
#pragma unroll
  for (int t = 0; t < FW; ++t) {
    const int r = (wave * FW + t) * 8 + (lane >> 3);
    voffW[t] = (uint32_t)r * (uint32_t)row_b + (uint32_t)(((lane & 7) ^ ((r >> 1) & 7)) * 16);
  }
#pragma unroll
  for (int t = 0; t < FX; ++t) {
    const int r = (wave * FX + t) * 8 + (lane >> 3);
    voffX[t] = (uint32_t)r * (uint32_t)row_b + (uint32_t)(((lane & 7) ^ ((r >> 1) & 7)) * 16);
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const i32x4 rsrcX = buffer_of(a.x, (size_t)a.M * row_b);
  auto fetch = [&](int u, int st) {
    const int n0 = u / nk * BN, kt = u % nk;
    const i32x4 rsrcW = buffer_of((const char*)a.w + (size_t)n0 * row_b, (size_t)(a.N - n0 < BN ? a.N - n0 : BN) * row_b);
    const uint32_t soff = (uint32_t)kt * (BK * 2), base = lds0 + (uint32_t)st * STAGE;
#pragma unroll
    for (int t = 0; t < FW; ++t) fetch_rows<4>(rsrcW, voffW[t], soff, base + (uint32_t)(wave * FW + t) * 1024u);
#pragma unroll
    for (int t = 0; t < FX; ++t) fetch_rows<4>(rsrcX, voffX[t], soff, base + WBYTES + (uint32_t)(wave * FX + t) * 1024u);
  };
  // fragment bases inside a stage; K-step of 32: xor 64
  const uint32_t sw = (uint32_t)(lq ^ ((l16 >> 1) & 7)) * 16u;
  const uint32_t baseW = (uint32_t)(wvn * NI * 16 + l16) * 128u + sw, baseX = WBYTES + (uint32_t)(wvm * NJ * 16 + l16) * 128u + sw;

  f32x4 acc[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  int ahead = u0;                                        // next unit to fetch
  for (; ahead < u1 && ahead < u0 + ST - 1; ++ahead) fetch(ahead, (ahead - u0) % ST);
  int st = 0;
  for (int u = u0; u < u1; ++u) {
    // this wave's part of the unit has landed (the younger fetches may still travel); behind the barrier that holds for the
    // block, and every wave is done with the stage of the unit before, which the next fetch overwrites
    wait_fetched<PER, ST - 2>(u1 - 1 - u);
    if (ahead < u1) { fetch(ahead, st == 0 ? ST - 1 : st - 1); ++ahead; }
    const unsigned char* sp = smem + (uint32_t)st * STAGE;
    st = st + 1 == ST ? 0 : st + 1;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      bf16x8 fw[NI], fx[NJ];
#pragma unroll
      for (int i = 0; i < NI; ++i) fw[i] = as_frag(*(const u32x4*)(sp + i * 2048 + (baseW ^ (kk * 64u))));
#pragma unroll
      for (int j = 0; j < NJ; ++j) fx[j] = as_frag(*(const u32x4*)(sp + j * 2048 + (baseX ^ (kk * 64u))));
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[i], fx[j], acc[i][j], 0, 0, 0);
    }
    if (u + 1 == u1 || (u + 1) % nk == 0) {              // the block's part of this tile ends here
      const int tile = u / nk, n0 = tile * BN, first_u = tile * nk;
      if (u0 <= first_u)                                 // the block that began the tile adds the low-rank term
        add_low_rank_16<NI, NJ>(a, acc, 0, n0, wvm * NJ * 16, wvn * NI * 16, lane);
      float* out = a.partial + (size_t)(blockIdx.x - first_u / U) * a.M * a.ldp;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int m = (wvm * NJ + j) * 16 + l16;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          const int n = n0 + (wvn * NI + i) * 16 + lq * 4;
          if (m < a.M && n < a.N) *(f32x4*)(out + (size_t)m * a.ldp + n) = acc[i][j];
          acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
    }
  }
}

template <int BM, int ST, int WGM>
hipError_t launch_stream(hipStream_t st, const MfmaGemmArgs& a, int blocks) {
  constexpr size_t lds = (size_t)ST * (128 + BM) * 128;
  static const hipError_t attr_status = hipFuncSetAttribute((const void*)gemm_stream_kernel<BM, ST, WGM>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (attr_status != hipSuccess) return attr_status;
  gemm_stream_kernel<BM, ST, WGM><<<blocks, 512, lds, st>>>(a);
  return hipSuccess;
}

}  // namespace

hipError_t launch_gemm_stream(hipStream_t st, const MfmaGemmArgs& a) {
  const long units = (long)((a.N + 127) / 128) * (a.K / 64);
  const int blocks = (int)((units + a.stream_units - 1) / a.stream_units);
  if (a.M <= 64) return launch_stream<64, 6, 2>(st, a, blocks);
  if (a.M <= 128) return launch_stream<128, 5, 4>(st, a, blocks);
  return launch_stream<256, 3, 4>(st, a, blocks);
}

// K-tiles per block: one run for each of 256 CUs, of at least 8; 0 = the partial sums would not fit `capacity` floats
int gemm_stream_units(const MfmaGemmArgs& a, size_t capacity) {
  if (a.M > 256 || a.K % 64 || a.N % 4 || a.w_scale != nullptr || a.w_absmax != nullptr || !fetch_aligned(a)) return 0;
  const int nk = a.K / 64;
  const long units = (long)((a.N + 127) / 128) * nk;
  long U = (units + 255) / 256;
  U = U < 8 ? 8 : U;
  while (U < nk && (size_t)stream_slots(nk, (int)U) * a.M * a.N > capacity) ++U;
  return (size_t)stream_slots(nk, (int)U) * a.M * a.N <= capacity ? (int)U : 0;
}

}  // namespace mpz
