// bf16 models, copies whose rows are no multiple of 32: the adapted linears and the LoRA bottleneck with the sums, bit for bit,
// of the shape-agnostic kernels (linear_kernel and lora_down_kernel of simple_kernels.hip), on the fp32 matrix instructions.
// Every sum is one binary32 chain, sum = fma(x_k, w_k, sum) for k = 0, 1, ..., K - 1: v_mfma_f32_32x32x2 and v_mfma_f32_16x16x4
// take their 2 and 4 products one after another in that order, each fused and rounded to nearest (bf16, fp32, 2^-30 ... 2^30
// and subnormal operands: every bit of 1024 chains of 512).  The bf16 matrix instructions add in another order; on such
// batches a step's two-point differences (small copies: few tokens, so little averages out) moved by more than the 1e-3 that
// a step's masters are held to.
// Bound by the fp32 matrix rate (256 FLOP per clock and CU, a sixteenth of bf16) and, few tokens, by the chain: K / 2 dependent
// instructions of 64 clocks.  A 1.1B-shaped block, 8 copies of 231 rows, adapters on all four projections: 2157 us with the
// shape-agnostic kernels, 637 us with these (1848 x 2560 x 2048: 222 us, 87 TFLOP/s; the bottleneck of three targets 30 us).
#include "common.h"
#include "fetch.h"
#include "../../include/mpz.h"

namespace mpz {
namespace {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

// two factors as the contraction sees them: bf16 hi + lo of the fp32 values
__device__ __forceinline__ void factors(float& a, float& b) {
  const uint32_t h = pack_bf16x2(a, b);
  const float ha = __uint_as_float(h << 16), hb = __uint_as_float(h & 0xFFFF0000u);
  const uint32_t l = pack_bf16x2(a - ha, b - hb);
  a = ha + __uint_as_float(l << 16);
  b = hb + __uint_as_float(l & 0xFFFF0000u);
}

// out = epilogue(x W^T): a block of four waves, 32 tokens x 32 features each; K-tiles of 64 go straight into a ring of three LDS
// stages.  (Operands read by each wave for itself, a piece of 32 rows per instruction: 338 us a launch against 204, the two
// adapted projections of that block together.)  Both halves of a wave read the same eight k of a row: the lower half takes the even ones, the
// upper half the odd ones, which is the order in which the instruction adds.  MFMA layout: lane l holds A[l % 32][l / 32],
// B[l / 32][l % 32] and, of the result, D[8 (r / 4) + 4 (l / 32) + r % 4][l % 32], r = 0..15: rows are tokens, columns features.
__global__ void __launch_bounds__(256) linear_ordered_kernel(LinearArgs a) {
  constexpr int BK = 64, ST = 3, PER = 4;                  // k per stage, stages, fetches of a wave per stage (8 rows of 128 bytes each)
  constexpr uint32_t HALF_STAGE = 64 * BK * 2, STAGE = 2 * HALF_STAGE;
  __shared__ __align__(16) unsigned char smem[ST * STAGE];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, half = lane >> 5;
  // XCD-aware tile order, groups of 8 token tiles per feature tile: see gemm_bf16_kernel
  const int tiles_n = gridDim.x, tiles_m = gridDim.y, nblk = tiles_n * tiles_m;
  int pid = blockIdx.y * tiles_n + blockIdx.x;
  {
    const int per = nblk / 8, rem = nblk % 8, xcd = pid % 8;
    pid = xcd * per + (xcd < rem ? xcd : rem) + pid / 8;
  }
  constexpr int GM = 8;
  const int group = pid / (GM * tiles_n), first_m = group * GM;
  const int gsz = tiles_m - first_m < GM ? tiles_m - first_m : GM;
  const int rr = pid - group * GM * tiles_n;
  const int bm = (first_m + rr % gsz) * 64, bn = rr / gsz * 64;
  const int m0 = bm + (wave >> 1) * 32, n0 = bn + (wave & 1) * 32;

  // buffers hold the tile's rows: rows past M or N fall outside (zeros), and their results are not stored.  Waves 0 and 1 fetch the
  // token rows, 2 and 3 the weight rows; 16-byte chunk c of row r lies at c ^ ((r / 2) % 8)
  const size_t row_b = (size_t)a.K * 2;
  const bool weights = wave >= 2;
  const int r_first = weights ? bn : bm, r_end = weights ? a.N : a.M, left = r_end - r_first < 64 ? r_end - r_first : 64;
  const i32x4 rsrc = buffer_of((const char*)(weights ? a.w : a.x) + (size_t)r_first * row_b, (size_t)left * row_b);
  uint32_t voff[PER];
#pragma unroll
  for (int t = 0; t < PER; ++t) {
    const int r = ((wave & 1) * PER + t) * 8 + (lane >> 3);
    voff[t] = (uint32_t)r * (uint32_t)row_b + (uint32_t)(((lane & 7) ^ ((r >> 1) & 7)) * 16);
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem + (uint32_t)wave * (PER * 1024u);
  auto fetch = [&](int kt, int st) {
#pragma unroll
    for (int t = 0; t < PER; ++t) fetch_rows<4>(rsrc, voff[t], (uint32_t)kt * (BK * 2), lds0 + (uint32_t)st * STAGE + (uint32_t)t * 1024u);
  };
  const uint32_t sw = (uint32_t)((l32 >> 1) & 7) * 16u;
  const uint32_t baseX = (uint32_t)((wave >> 1) * 32 + l32) * 128u, baseW = HALF_STAGE + (uint32_t)((wave & 1) * 32 + l32) * 128u;
  const uint32_t sel = half ? 0x07060c0cu : 0x05040c0cu;   // of two bf16 the one of this half's k, as fp32
  auto take = [&](uint32_t two) { return __uint_as_float(__builtin_amdgcn_perm(two, 0u, sel)); };

  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  const int nk = a.K / BK;
#pragma unroll
  for (int t = 0; t < ST - 1; ++t)
    if (t < nk) fetch(t, t);
  int st = 0;
  for (int kt = 0; kt < nk; ++kt) {
    // K-tile kt has landed for the whole block, and every wave is done with the stage that the next fetch overwrites
    wait_fetched<PER, ST - 2>(nk - 1 - kt);
    if (kt + ST - 1 < nk) fetch(kt + ST - 1, st == 0 ? ST - 1 : st - 1);
    const unsigned char* sp = smem + (uint32_t)st * STAGE;
    st = st + 1 == ST ? 0 : st + 1;
#pragma unroll
    for (int c = 0; c < BK / 8; ++c) {
      const u32x4 x = *(const u32x4*)(sp + baseX + ((uint32_t)c * 16u ^ sw)), w = *(const u32x4*)(sp + baseW + ((uint32_t)c * 16u ^ sw));
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(take(x[e]), take(w[e]), acc, 0, 0, 0);
    }
  }
  if (m0 >= a.M || n0 >= a.N) return;                      // (no barriers below)
  const int mrow = m0 + l32 < a.M ? m0 + l32 : a.M - 1;
  const int n = n0 + l32;

  // per-copy low-rank term: a chain of its own over the rank, for every copy that has rows in the tile; its sum goes to the
  // rows of that copy alone (a result row depends on its own row of t only)
  const int last_row = m0 + 31 < a.M ? m0 + 31 : a.M - 1;
  const int first_copy = m0 / a.rows_per_copy, last_copy = last_row / a.rows_per_copy;
  for (int s = 0; s < a.n_seg; ++s) {
    const LoraSeg& sg = a.seg[s];
    if (n0 + 31 < sg.col_begin || n0 >= sg.col_end) continue;
    const int kout = sg.col_end - sg.col_begin;
    const bool in = n >= sg.col_begin && n < sg.col_end;
    const bf16_t* t = (const bf16_t*)sg.t + (int64_t)mrow * sg.t_stride + sg.t_off;
    for (int copy = first_copy; copy <= last_copy; ++copy) {
      const float* B = sg.Bc + (int64_t)copy * sg.copy_stride + (in ? n - sg.col_begin : 0);
      f32x16 dl;
#pragma unroll
      for (int e = 0; e < 16; ++e) dl[e] = 0.f;
      for (int r = half; r < a.rank + half; r += 4) {      // (ranks are multiples of 4)
        float b0 = B[(int64_t)r * kout], b1 = B[(int64_t)(r + 2) * kout];
        factors(b0, b1);
        dl = __builtin_amdgcn_mfma_f32_32x32x2f32(bf16_to_f32(t[r]), b0, dl, 0, 0, 0);
        dl = __builtin_amdgcn_mfma_f32_32x32x2f32(bf16_to_f32(t[r + 2]), b1, dl, 0, 0, 0);
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int m = m0 + 8 * (e / 4) + 4 * half + e % 4;
        acc[e] = in && m / a.rows_per_copy == copy ? acc[e] + dl[e] : acc[e];
      }
    }
  }

  if (n >= a.N) return;
  const float bias = a.bias != nullptr ? a.bias[n] : 0.f;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int m = m0 + 8 * (e / 4) + 4 * half + e % 4;
    if (m >= a.M) continue;
    float v = acc[e];
    if (a.bias != nullptr) v += bias;
    if (a.act == MPZ_ACT_RELU) v = v > 0.f ? v : 0.f;
    const int64_t o = (int64_t)m * a.N + n;
    if (a.residual != nullptr) v += a.residual[o];
    if (a.out_kind == 0) ((bf16_t*)a.out)[o] = f32_to_bf16(v);
    else ((float*)a.out)[o] = v;                           // (bf16 models stage in fp32)
  }
}

// LoRA bottleneck t = bf16(scale * x A_c): a wave per 16 rows of one copy and 16 bottleneck columns.  Bound by the latency of its
// chain: K / 4 dependent instructions of 32 clocks.  Lane l holds x[l % 16][k = l / 16] and A[k = l / 16][column l % 16] of every
// four k and, of the result, D[4 (l / 16) + r][l % 16], r = 0..3.
__global__ void __launch_bounds__(64) lora_down_ordered_kernel(LoraDownArgs a, int tiles_per_copy, int col_tiles) {
  constexpr int CH = 4, AHEAD = 6;                         // pieces of 8 k in a register set, sets in flight
  const int lane = threadIdx.x, l16 = lane & 15, lq = lane >> 4, R = a.n_targets * a.rank;
  const int col_tile = blockIdx.x % col_tiles, rest = blockIdx.x / col_tiles;
  const int copy = rest / tiles_per_copy, r0 = rest % tiles_per_copy * 16;   // first row inside the copy
  const int row = r0 + l16 < a.rows_per_copy ? r0 + l16 : a.rows_per_copy - 1;
  const u32x4* px = (const u32x4*)((const uint16_t*)a.x + (int64_t)(copy * (int64_t)a.rows_per_copy + row) * a.K);
  const int j = col_tile * 16 + l16, jj = j < R ? j : R - 1;
  const float* A = a.Ac[jj / a.rank] + (int64_t)copy * a.copy_stride + (int64_t)lq * a.rank + jj % a.rank;
  const uint32_t sel = 0x00000c0cu | (uint32_t)(2 * lq) << 16 | (uint32_t)(2 * lq + 1) << 24;    // element lq of four bf16
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  const int chunks = a.K / (8 * CH);
  u32x4 rx[AHEAD][CH];
  float rf[AHEAD][2 * CH];
  auto request = [&](u32x4 (&x)[CH], float (&f)[2 * CH], int c) {
    c = c < chunks ? c : chunks - 1;                       // (past the end: the last piece again, never multiplied)
#pragma unroll
    for (int i = 0; i < CH; ++i) x[i] = px[c * CH + i];
#pragma unroll
    for (int i = 0; i < 2 * CH; ++i) f[i] = A[(int64_t)(c * 8 * CH + 4 * i) * a.rank];
  };
#pragma unroll
  for (int u = 0; u < AHEAD; ++u) request(rx[u], rf[u], u);
  for (int c0 = 0; c0 < chunks; c0 += AHEAD)
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      if (c0 + u >= chunks) break;                         // (uniform)
#pragma unroll
      for (int i = 0; i < 2 * CH; i += 2) factors(rf[u][i], rf[u][i + 1]);
#pragma unroll
      for (int i = 0; i < 2 * CH; ++i) {
        const float x = __uint_as_float(__builtin_amdgcn_perm(rx[u][i / 2][i % 2 * 2 + 1], rx[u][i / 2][i % 2 * 2], sel));
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x, rf[u][i], acc, 0, 0, 0);
      }
      request(rx[u], rf[u], c0 + u + AHEAD);
      __builtin_amdgcn_sched_barrier(0);
    }
  if (j >= R) return;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int rc = r0 + 4 * lq + r;
    if (rc < a.rows_per_copy) ((bf16_t*)a.t)[(copy * (int64_t)a.rows_per_copy + rc) * R + j] = f32_to_bf16(acc[r] * a.scale);
  }
}

}  // namespace

// whole K-tiles, operands that begin on 16 bytes and stay below 2 GiB per tile of 64 rows, no GELU (its erff would be contracted in
// other surroundings)
bool launch_linear_ordered(hipStream_t st, const LinearArgs& a) {
  if (a.dtype != MPZ_DTYPE_BF16 || a.K % 64 || a.K < 64 || a.K >= 1 << 24 || a.act == MPZ_ACT_GELU_ERF || (((uintptr_t)a.x | (uintptr_t)a.w) & 15)) return false;
  linear_ordered_kernel<<<dim3((a.N + 63) / 64, (a.M + 63) / 64), 256, 0, st>>>(a);
  return true;
}

bool launch_lora_down_ordered(hipStream_t st, const LoraDownArgs& a) {
  if (a.dtype != MPZ_DTYPE_BF16 || a.K % 32 || a.K < 32 || ((uintptr_t)a.x & 15) || a.T % a.rows_per_copy) return false;
  const int tiles = (a.rows_per_copy + 15) / 16, cols = (a.n_targets * a.rank + 15) / 16;
  const int64_t blocks = (int64_t)(a.T / a.rows_per_copy) * tiles * cols;
  if (blocks * 64 > (int64_t)UINT32_MAX) return false;
  lora_down_ordered_kernel<<<(unsigned)blocks, 64, 0, st>>>(a, tiles, cols);
  return true;
}

}  // namespace mpz
