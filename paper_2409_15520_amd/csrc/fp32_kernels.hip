// The two heavy operations of fp32 models on the matrix cores and the wave: linears with 64-bit sums (v_mfma_f64_16x16x4),
// and the LoRA bottleneck.  Operands are fp32 values widened exactly, sums are binary64 as in the shape-agnostic kernels of
// simple_kernels.hip (another order of the same 64-bit sum), and every stored value is rounded once.
#include "common.h"
#include "../../include/mpz.h"

namespace mpz {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) double f64x4;

// out = epilogue(x W^T) on tiles of 16 WT x 16 WT, one block per tile, its four waves a quarter of K each.  Bound by latency at
// the sizes of the tiny models (a whole step of 2 blocks of d = 128 over 256 rows: 485 us with the shape-agnostic kernels, 107 us
// with those of this file; a 125M-shaped block over 768 rows: 1346 us, 360 us) and by the fp64 matrix rate
// (72 TFLOP/s in the library) above: 768 x 2304 x 768.  Splitting K over the waves of a block, and not tiles, is what gives
// small outputs enough wavefronts; operands come straight from L2 (a 32 x 32 tile needs 16 bytes per clock and CU).
// MFMA layout: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16] and, of the result, D[l / 16 + 4 r][l % 16], r = 0..3.  Of
// every 16 consecutive k a lane takes the four from 4 (l / 16) on, one per step: 16-byte loads, and the same k on both operands.
template <int WT>
__global__ void __launch_bounds__(256) linear_f64_kernel(LinearArgs a) {
  constexpr int BT = 16 * WT;
  __shared__ double part[4][BT][BT + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, lq = lane >> 4;
  const int m0 = blockIdx.y * BT, n0 = blockIdx.x * BT;
  const float* px[WT];
  const float* pw[WT];
#pragma unroll
  for (int t = 0; t < WT; ++t) {                           // rows past the end read the last one; their results are not stored
    const int m = m0 + t * 16 + l16, n = n0 + t * 16 + l16;
    px[t] = (const float*)a.x + (size_t)(m < a.M ? m : a.M - 1) * a.K;
    pw[t] = (const float*)a.w + (size_t)(n < a.N ? n : a.N - 1) * a.K;
  }
  f64x4 acc[WT][WT];
#pragma unroll
  for (int i = 0; i < WT; ++i)
#pragma unroll
    for (int j = 0; j < WT; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  const int steps = (a.K + 15) / 16, s0 = steps * wave / 4, s1 = steps * (wave + 1) / 4;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 cx[WT], cw[WT], nx[WT], nw[WT];
  auto fetch = [&](int s, f32x4 (&x)[WT], f32x4 (&w)[WT]) {
    const int k = s * 16 + lq * 4;                         // (K % 4 == 0: a piece is inside the row or past it)
#pragma unroll
    for (int t = 0; t < WT; ++t) {
      x[t] = k < a.K ? *(const f32x4*)(px[t] + k) : zero;
      w[t] = k < a.K ? *(const f32x4*)(pw[t] + k) : zero;
    }
  };
  if (s0 < s1) fetch(s0, cx, cw);
  for (int s = s0; s < s1; ++s) {
    if (s + 1 < s1) fetch(s + 1, nx, nw);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < WT; ++i)
#pragma unroll
        for (int j = 0; j < WT; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)cx[i][e], (double)cw[j][e], acc[i][j], 0, 0, 0);
#pragma unroll
    for (int t = 0; t < WT; ++t) { cx[t] = nx[t]; cw[t] = nw[t]; }
  }
#pragma unroll
  for (int i = 0; i < WT; ++i)
#pragma unroll
    for (int j = 0; j < WT; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) part[wave][i * 16 + r * 4 + lq][j * 16 + l16] = acc[i][j][r];
  __syncthreads();
  for (int idx = tid; idx < BT * BT; idx += 256) {
    const int row = idx / BT, col = idx % BT, m = m0 + row, n = n0 + col;
    if (m >= a.M || n >= a.N) continue;
    double v = ((part[0][row][col] + part[1][row][col]) + part[2][row][col]) + part[3][row][col];
    for (int s = 0; s < a.n_seg; ++s) {
      const LoraSeg& sg = a.seg[s];
      if (n < sg.col_begin || n >= sg.col_end) continue;
      const int kout = sg.col_end - sg.col_begin;
      const float* t = (const float*)sg.t + (size_t)m * sg.t_stride + sg.t_off;
      const float* B = sg.Bc + (size_t)(m / a.rows_per_copy) * sg.copy_stride + (n - sg.col_begin);
      double dl = 0.0;
      for (int r = 0; r < a.rank; ++r) dl += (double)t[r] * (double)B[(size_t)r * kout];
      v += dl;
    }
    if (a.bias != nullptr) v += (double)a.bias[n];
    if (a.act == MPZ_ACT_RELU) v = v > 0.0 ? v : 0.0;
    else if (a.act == MPZ_ACT_GELU_ERF) v = 0.5 * v * (1.0 + erf(v * 0.70710678118654752440));
    const size_t o = (size_t)m * a.N + n;
    if (a.residual != nullptr) v += (double)a.residual[o];
    if (a.out_kind == 2) ((double*)a.out)[o] = v;
    else ((float*)a.out)[o] = (float)v;
  }
}

// LoRA bottleneck t = fp32(scale * x A_c): a wave per row and four columns, its lanes along K (the shape-agnostic kernel has a
// thread per column walk K alone: 768 rows, K = 768, 16 columns 85 us)
__global__ void __launch_bounds__(256) lora_down_f64_kernel(LoraDownArgs a) {
  const int groups = a.rank / 4, R = a.n_targets * a.rank;
  const int per_row = a.n_targets * groups;
  for (int64_t item = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); item < (int64_t)a.T * per_row; item += (int64_t)gridDim.x * 4) {
    const int m = (int)(item / per_row), g = (int)(item % per_row), tgt = g / groups, j0 = (g % groups) * 4, lane = threadIdx.x & 63;
    const float* A = a.Ac[tgt] + (int64_t)(m / a.rows_per_copy) * a.copy_stride + j0;
    const float* x = (const float*)a.x + (int64_t)m * a.K;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int k = lane; k < a.K; k += 64) {
      const f32x4 av = *(const f32x4*)(A + (int64_t)k * a.rank);
      const double xv = (double)x[k];
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] += xv * (double)av[e];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] += __shfl_xor(s[e], o, 64);
    if (lane < 4) {
      const double v = lane == 0 ? s[0] : lane == 1 ? s[1] : lane == 2 ? s[2] : s[3];
      ((float*)a.t)[(int64_t)m * R + tgt * a.rank + j0 + lane] = (float)(v * (double)a.scale);
    }
  }
}

}  // namespace

// 32 x 32 tiles once they give every CU a block, 16 x 16 below (256 x 128 x 128: 32 against 128 blocks)
bool launch_linear_f64(hipStream_t st, const LinearArgs& a) {
  if (a.dtype != MPZ_DTYPE_F32 || a.K % 4 || (((uintptr_t)a.x | (uintptr_t)a.w) & 15)) return false;
  const long big = (long)((a.N + 31) / 32) * ((a.M + 31) / 32);
  if (big >= 256) linear_f64_kernel<2><<<dim3((a.N + 31) / 32, (a.M + 31) / 32), 256, 0, st>>>(a);
  else linear_f64_kernel<1><<<dim3((a.N + 15) / 16, (a.M + 15) / 16), 256, 0, st>>>(a);
  return true;
}

bool launch_lora_down_f64(hipStream_t st, const LoraDownArgs& a) {
  if (a.dtype != MPZ_DTYPE_F32 || a.rank % 4 || a.copy_stride % 4) return false;
  for (int t = 0; t < a.n_targets; ++t)
    if ((uintptr_t)a.Ac[t] & 15) return false;
  const int64_t items = (int64_t)a.T * a.n_targets * (a.rank / 4);
  const int64_t blocks = (items + 3) / 4, most = UINT32_MAX / 256;   // (a launch holds fewer than 2^32 threads; the waves walk the rest)
  lora_down_f64_kernel<<<(unsigned)(blocks < most ? blocks : most), 256, 0, st>>>(a);
  return true;
}

}  // namespace mpz
