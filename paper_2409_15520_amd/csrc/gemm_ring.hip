// The GEMM of small outputs: bf16 weights, 32 x 32 tiles, no split of K.
//
// What bounds it: with about one 64 x 64 tile per CU or fewer, each block walks K alone, and its time is what its CU can fetch
// (some 90 GB/s, whether through registers or straight into LDS) of a tile's operands.  A quarter of the tile is half the bytes
// per block on four times the blocks: all of them are resident at once (three per CU), K-tiles of 128 halve the barriers, and
// the tiles go straight into a ring of three LDS stages.  (64 x 64 tiles fetched that way are slower than through registers:
// 6.6 against 5.4 us for the first shape below.)  384 x 768 x 768: 5.4 -> 4.4 us, 384 x 768 x 3072: 15.8 -> 10.4 us
// (tokens x features x K; 64 x 64 tiles before).  Every sum is taken in the order of gemm_bf16_kernel: the same bits.
#include "gemm_tile.h"
#include "fetch.h"

namespace mpz {
namespace {

constexpr int BN = 32, BM = 32, BK = 128, ST = 3;

// four waves, one 16 x 16 tile each
__global__ void __launch_bounds__(256, 3) gemm_ring_kernel(MfmaGemmArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int CPR = BK / 8, RPF = 64 / CPR;                            // 16-byte chunks per tile row, rows per fetch
  constexpr int FW = BN / RPF / 4, FX = BM / RPF / 4, PER = FW + FX;     // fetches of a wave per K-tile
  constexpr uint32_t ROW = BK * 2, WBYTES = BN * ROW, STAGE = WBYTES + BM * ROW;

  // tile order: see gemm_bf16_kernel
  const int tiles_n = (a.N + BN - 1) / BN, tiles_m = (a.M + BM - 1) / BM;
  const int nblk = tiles_n * tiles_m;
  int pid = blockIdx.x;
  {
    const int per = nblk / 8, rem = nblk % 8, xcd = pid % 8, idx = pid / 8;
    pid = xcd * per + (xcd < rem ? xcd : rem) + idx;
  }
  constexpr int GM = 8;
  const int group = pid / (GM * tiles_n), first_m = group * GM;
  const int gsz = tiles_m - first_m < GM ? tiles_m - first_m : GM;
  const int rr = pid - group * GM * tiles_n;
  const int m0 = (first_m + rr % gsz) * BM, n0 = rr / gsz * BN;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, lq = lane >> 4;
  const int wn = (wave >> 1) * (BN / 2), wm = (wave & 1) * (BM / 2);

  // buffers hold the tile's rows: rows past N or M fall outside, and what they accumulate is never stored.  16-byte chunk c of
  // row r lies at c ^ (r % 16), so that 16 rows read at one chunk meet all banks
  const uint32_t row_b = (uint32_t)a.K * 2u;
  const i32x4 rsrcW = buffer_of((const char*)a.w + (size_t)n0 * row_b, (size_t)(a.N - n0 < BN ? a.N - n0 : BN) * row_b);
  const i32x4 rsrcX = buffer_of((const char*)a.x + (size_t)m0 * row_b, (size_t)(a.M - m0 < BM ? a.M - m0 : BM) * row_b);
  uint32_t voffW[FW], voffX[FX];
#pragma unroll
  for (int t = 0; t < FW; ++t) {
    const int r = (wave * FW + t) * RPF + lane / CPR;
    voffW[t] = (uint32_t)r * row_b + (uint32_t)((lane % CPR) ^ (r & 15)) * 16u;
  }
#pragma unroll
  for (int t = 0; t < FX; ++t) {
    const int r = (wave * FX + t) * RPF + lane / CPR;
    voffX[t] = (uint32_t)r * row_b + (uint32_t)((lane % CPR) ^ (r & 15)) * 16u;
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const int nk = a.K / BK;
  auto fetch = [&](int kt, int st) {
    const uint32_t soff = (uint32_t)kt * ROW, base = lds0 + (uint32_t)st * STAGE;
#pragma unroll
    for (int t = 0; t < FW; ++t) fetch_rows<4>(rsrcW, voffW[t], soff, base + (uint32_t)(wave * FW + t) * 1024u);
#pragma unroll
    for (int t = 0; t < FX; ++t) fetch_rows<4>(rsrcX, voffX[t], soff, base + WBYTES + (uint32_t)(wave * FX + t) * 1024u);
  };

  f32x4 acc[1][1] = {{f32x4{0.f, 0.f, 0.f, 0.f}}};
  const uint32_t sw = (uint32_t)(lq ^ l16) * 16u;     // (wave tiles begin at multiples of 16 rows); K-step s: xor 64 s
  const uint32_t baseW = (uint32_t)(wn + l16) * ROW + sw, baseX = WBYTES + (uint32_t)(wm + l16) * ROW + sw;
#pragma unroll
  for (int t = 0; t < ST - 1; ++t)
    if (t < nk) fetch(t, t);
  int st = 0;
  for (int kt = 0; kt < nk; ++kt) {
    // K-tile kt has landed (younger fetches may still travel) and every wave is done with the stage of the tile before, which
    // the next fetch overwrites
    wait_fetched<PER, ST - 2>(nk - 1 - kt);
    if (kt + ST - 1 < nk) fetch(kt + ST - 1, st == 0 ? ST - 1 : st - 1);
    const unsigned char* sp = smem + (uint32_t)st * STAGE;
    st = st + 1 == ST ? 0 : st + 1;
    bf16x8 fw[BK / 32], fx[BK / 32];
#pragma unroll
    for (int s = 0; s < BK / 32; ++s) {
      fw[s] = as_frag(*(const u32x4*)(sp + (baseW ^ (s * 64u))));
      fx[s] = as_frag(*(const u32x4*)(sp + (baseX ^ (s * 64u))));
    }
#pragma unroll
    for (int s = 0; s < BK / 32; ++s) acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[s], fx[s], acc[0][0], 0, 0, 0);
  }
  add_low_rank_16<1, 1>(a, acc, m0, n0, wm, wn, lane);

  // epilogue: the tile turns around in LDS, so that consecutive lanes take consecutive features of a token
  constexpr int EPS = BN + 4;
  float* ep = (float*)smem;
  __syncthreads();
  *(f32x4*)(ep + (wm + l16) * EPS + wn + lq * 4) = acc[0][0];
  __syncthreads();
  const int row = tid / 8, m = m0 + row, n = n0 + tid % 8 * 4;
  if (m >= a.M || n >= a.N) return;
  const size_t o = (size_t)m * a.ldo + n;
  f32x4 v = *(const f32x4*)(ep + row * EPS + tid % 8 * 4);
  if (a.bias != nullptr) v += *(const f32x4*)(a.bias + n);
  if (a.act == MPZ_ACT_RELU) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
  } else if (a.act == MPZ_ACT_GELU_ERF) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = gelu_erf_call(v[e]);
  }
  if (a.residual != nullptr) v += *(const f32x4*)(a.residual + o);
  if (a.out_f32) *(f32x4*)((float*)a.out + o) = v;
  else *(u32x2*)((uint16_t*)a.out + o) = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
}

}  // namespace

bool gemm_ring_supported(const MfmaGemmArgs& a) {
  return a.w_scale == nullptr && a.w_absmax == nullptr && a.k_splits <= 1 && !a.dual && a.rope_cos == nullptr && a.ce_max == nullptr &&
         a.K % BK == 0 && fetch_aligned(a);
}

hipError_t launch_gemm_ring(hipStream_t st, const MfmaGemmArgs& a) {
  gemm_ring_kernel<<<(unsigned)(((a.N + BN - 1) / BN) * ((a.M + BM - 1) / BM)), 256, ST * (BN + BM) * BK * 2, st>>>(a);
  return hipSuccess;
}

}  // namespace mpz
