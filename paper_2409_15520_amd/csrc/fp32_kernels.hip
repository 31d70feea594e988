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
// the sizes of the tiny models and by the fp64 matrix rate (72 TFLOP/s in the library) above: 768 x 2304 x 768.  Splitting K over
// the waves of a block, and not tiles, is what gives small outputs enough wavefronts; operands come straight from L2 (a 32 x 32 tile
// needs 16 bytes per clock and CU), AHEAD steps of 16 k ahead.  The fp64 matrix instructions run on the vector lanes: nothing else
// does meanwhile, so a step's operands are widened together, addresses are scalar, and wider tiles widen less per product (768 x 768 x 768 34 -> 26 us,
// 768 x 768 x 3072 112 -> 72, 768 x 3072 x 768 87 -> 74, Q|K|V with adapters 82 -> 77).
// MFMA layout: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16] and, of the result, D[l / 16 + 4 r][l % 16], r = 0..3.  Of
// every 16 consecutive k a lane takes the four from 4 (l / 16) on, one per step: 16-byte loads, and the same k on both operands.
template <int WT>
__global__ void __launch_bounds__(256, 2) linear_f64_kernel(LinearArgs a) {
  constexpr int BT = 16 * WT, AHEAD = WT == 3 ? 2 : 3;
  __shared__ double part[4][BT][BT + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, lq = lane >> 4;
  const int m0 = blockIdx.y * BT, n0 = blockIdx.x * BT;
  // buffers hold the tile's rows: rows past the end fall outside (zeros); their results are not stored
  auto rows_of = [&](const void* p, int first, int end) {
    const int left = end - first < BT ? end - first : BT;
    return __builtin_amdgcn_make_buffer_rsrc((float*)p + (size_t)first * a.K, 0, (int)((size_t)left * a.K * 4), 0x00020000);
  };
  const __amdgpu_buffer_rsrc_t rx = rows_of(a.x, m0, a.M), rw = rows_of(a.w, n0, a.N);
  int voff[WT];
#pragma unroll
  for (int t = 0; t < WT; ++t) voff[t] = ((t * 16 + l16) * a.K + lq * 4) * 4;
  f64x4 acc[WT][WT];
#pragma unroll
  for (int i = 0; i < WT; ++i)
#pragma unroll
    for (int j = 0; j < WT; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  const int steps = (a.K + 15) / 16, s0 = steps * wave / 4, s1 = steps * (wave + 1) / 4;
  f32x4 x[AHEAD + 1][WT], w[AHEAD + 1][WT];
  const bool outside = a.K % 16 != 0 && lq * 4 >= a.K % 16;   // of a last step that is not whole (K % 4 == 0), this lane's piece
  auto fetch = [&](int s, int slot) {
#pragma unroll
    for (int t = 0; t < WT; ++t) {
      const int v = s == steps - 1 && outside ? (int)0x80000000 : voff[t];
      x[slot][t] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rx, v, s * 64, 0));
      w[slot][t] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rw, v, s * 64, 0));
    }
  };
#pragma unroll
  for (int u = 0; u < AHEAD; ++u)
    if (s0 + u < s1) fetch(s0 + u, u);
  for (int sb = s0; sb < s1; sb += AHEAD + 1)
#pragma unroll
    for (int u = 0; u <= AHEAD; ++u) {
      const int s = sb + u;
      if (s >= s1) break;                                  // (uniform)
      if (s + AHEAD < s1) fetch(s + AHEAD, (u + AHEAD) % (AHEAD + 1));
      __builtin_amdgcn_sched_barrier(0);
      double dx[WT][4], dw[WT][4];
#pragma unroll
      for (int t = 0; t < WT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) { dx[t][e] = (double)x[u][t][e]; dw[t][e] = (double)w[u][t][e]; }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
          for (int j = 0; j < WT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(dx[i][e], dw[j][e], acc[i][j], 0, 0, 0);
    }
  // per-copy low-rank term, a sum of its own over the rank, tile by tile in turn by the waves: for every copy that has rows in the
  // 16 x 16 tile; its sum goes to the rows of that copy alone.  (A thread per element walking the rank took 20 us of 82.)
#pragma unroll
  for (int i = 0; i < WT; ++i)
#pragma unroll
    for (int j = 0; j < WT; ++j) {
      const int mi = m0 + i * 16, nj = n0 + j * 16;
      if ((i * WT + j) % 4 != wave || mi >= a.M || nj >= a.N) continue;          // (uniform)
      const int last_row = mi + 15 < a.M ? mi + 15 : a.M - 1, n = nj + l16;
      for (int s = 0; s < a.n_seg; ++s) {
        const LoraSeg& sg = a.seg[s];
        if (nj + 15 < sg.col_begin || nj >= sg.col_end) continue;
        const int kout = sg.col_end - sg.col_begin;
        const bool in = n >= sg.col_begin && n < sg.col_end;
        const float* t = (const float*)sg.t + (size_t)(mi + l16 < a.M ? mi + l16 : a.M - 1) * sg.t_stride + sg.t_off;
        for (int copy = mi / a.rows_per_copy; copy <= last_row / a.rows_per_copy; ++copy) {
          const float* B = sg.Bc + (size_t)copy * sg.copy_stride + (in ? n - sg.col_begin : 0);
          f64x4 dl = {0.0, 0.0, 0.0, 0.0};
          for (int r = lq; r < a.rank + lq; r += 4)
            dl = __builtin_amdgcn_mfma_f64_16x16x4f64(r < a.rank ? (double)t[r] : 0.0, r < a.rank ? (double)B[(size_t)r * kout] : 0.0, dl, 0, 0, 0);
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[i][j][r] = in && (mi + lq + 4 * r) / a.rows_per_copy == copy ? acc[i][j][r] + dl[r] : acc[i][j][r];
        }
      }
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

// value of the lane N to the left in its row of 16 (rotated)
template <int N>
__device__ __forceinline__ double row_rotated(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (uint32_t)b, 0x120 + N, 0xF, 0xF, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (uint32_t)(b >> 32), 0x120 + N, 0xF, 0xF, false);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ double row_max(double v) {
  auto larger = [](double a, double b) { return b > a ? b : a; };
  v = larger(v, row_rotated<1>(v));
  v = larger(v, row_rotated<2>(v));
  v = larger(v, row_rotated<4>(v));
  return larger(v, row_rotated<8>(v));
}
__device__ __forceinline__ double row_sum(double v) {
  v += row_rotated<1>(v);
  v += row_rotated<2>(v);
  v += row_rotated<4>(v);
  return v + row_rotated<8>(v);
}

// Causal attention of up to 128 tokens: a block of four waves per sequence, head and 16 queries.  Scores of 16 keys at a time on the
// fp64 matrix instructions (a wave takes every fourth tile of keys), maxima and sums over the waves in LDS, probabilities through
// LDS into the layout of the product with V (a wave per 16 columns of the head).  What was rounded to fp32 stays so: the score, the
// probability, the result; sums are binary64.  Keys behind a query never enter its sums: in the tile of keys that holds the
// queries themselves the product with V is a masked sum.  Bound by the chain scores -> maximum -> exponentials -> sums (96 tokens, 12 heads of 64, eight
// sequences: 51 -> 15 us; tiny model, 32 tokens: 12 -> 6.5.  With branches around the requests 20 to 32 us and 10 to 12: the waits
// behind a branch are for everything).
template <int DH, int MAXT>
__global__ void __launch_bounds__(256) attention_f64_kernel(const float* __restrict__ qkv, int stride, float* __restrict__ out, int S, int H, int Hkv,
                                                            float scale, const int32_t* __restrict__ cu, int E, int rows_per_copy) {
  constexpr int NF = DH / 16, U = (MAXT + 3) / 4;           // (MAXT: tiles of 16 keys)
  __shared__ __align__(16) float P[16][MAXT * 16 + 4];
  __shared__ double red[2][4][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, lq = lane >> 4;
  const int tiles = (S + 15) / 16, qt = tiles - 1 - (int)(blockIdx.x % tiles), head = (int)(blockIdx.x / tiles % H);
  const int64_t seq = blockIdx.x / ((int64_t)tiles * H);
  int64_t row0 = seq * S;
  int len = S;
  if (cu != nullptr) {                                     // packed batch: S is the longest sequence, this one may be shorter
    const int e = (int)(seq % E);
    row0 = (seq / E) * rows_per_copy + cu[e];
    len = cu[e + 1] - cu[e];
    if (qt * 16 >= len) return;                            // (uniform)
  }
  const int d = H * DH, dkv = Hkv * DH, kvh = head / (H / Hkv);
  const float* base = qkv + row0 * stride;
  auto at = [&](int i, int col) { return base + ((uint32_t)(i < len ? i : len - 1) * (uint32_t)stride + (uint32_t)col); };
  f32x4 q[NF];
#pragma unroll
  for (int k = 0; k < NF; ++k) q[k] = *(const f32x4*)at(qt * 16 + l16, head * DH + k * 16 + lq * 4);
  // all requests at once and without branches (they return in order, the keys before the values); tiles behind the queries' own
  // read rows that exist and are not used
  f32x4 kf[U][NF];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int k = 0; k < NF; ++k) kf[u][k] = *(const f32x4*)at((u * 4 + wave) * 16 + l16, d + kvh * DH + k * 16 + lq * 4);
  const int c = wave * 16 + l16, vcol = d + dkv + kvh * DH + (c < DH ? c : 0);         // this lane's column of the head in the product with V
  float v[MAXT - 1][4], own[16];                           // of every tile of keys before the queries' own, and of that one
#pragma unroll
  for (int t = 0; t < MAXT - 1; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) v[t][e] = *at(t * 16 + lq * 4 + e, vcol);
#pragma unroll
  for (int j = 0; j < 16; ++j) own[j] = *at(qt * 16 + j, vcol);
  __builtin_amdgcn_sched_barrier(0);

  double s[U][4], mx[4] = {-1e30, -1e30, -1e30, -1e30};
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int t = u * 4 + wave;
    if (t > qt) continue;                                  // (uniform)
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < NF; ++k)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)q[k][e], (double)kf[u][k][e], acc, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {                          // query lq + 4 r, key l16 of the tiles
      s[u][r] = (double)(float)acc[r] * (double)scale;
      const bool seen = t < qt || l16 <= lq + 4 * r;
      mx[r] = seen && s[u][r] > mx[r] ? s[u][r] : mx[r];
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) mx[r] = row_max(mx[r]);
  if (l16 == 0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) red[0][wave][lq + 4 * r] = mx[r];
  }
  __syncthreads();
  double sum[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const double other = red[0][w][lq + 4 * r];
      mx[r] = other > mx[r] ? other : mx[r];
    }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int t = u * 4 + wave;
    if (t > qt) continue;                                  // (uniform)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool seen = t < qt || l16 <= lq + 4 * r;
      const float p = seen ? (float)exp(s[u][r] - mx[r]) : 0.f;
      P[lq + 4 * r][t * 16 + l16] = p;
      sum[r] += (double)p;
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) sum[r] = row_sum(sum[r]);
  if (l16 == 0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) red[1][wave][lq + 4 * r] = sum[r];
  }
  __syncthreads();
  if (wave >= NF) return;
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int t = 0; t < MAXT - 1; ++t) {
    if (t >= qt) continue;                                 // (uniform)
    const f32x4 p = *(const f32x4*)&P[l16][t * 16 + lq * 4];
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)p[e], (double)v[t][e], acc, 0, 0, 0);
  }
#pragma unroll
  for (int j = 0; j < 16; ++j) {                           // the queries' own tile
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r] = j <= lq + 4 * r ? fma((double)P[lq + 4 * r][qt * 16 + j], (double)own[j], acc[r]) : acc[r];
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = qt * 16 + lq + 4 * r;
    const double total = ((red[1][0][lq + 4 * r] + red[1][1][lq + 4 * r]) + red[1][2][lq + 4 * r]) + red[1][3][lq + 4 * r];
    if (i < len) out[(row0 + i) * d + head * DH + c] = (float)(acc[r] / total);
  }
}

}  // namespace

// Heads of 32 and 64 and up to 128 tokens (eight tiles of keys, which the registers hold); 16-byte rows.  Eight tokens at least: of shorter
// sequences most of a tile of queries is empty (2 / 4 tokens, 4 sequences of 12 heads: 4.3 / 4.4 us with a wave per query, 5.6 / 5.6 here; 256
// sequences: 8.4 / 15.1 against 17.2 / 17.5).  From there to 16 many sequences gain what few lose (8 / 16 tokens, 4 sequences: 4.9 / 5.8 against
// 5.7 / 5.9; 256: 29.9 / 68.1 against 18.7 / 20.9); the line is drawn by the tokens alone, so that a pass of one copy and a pass of all take the
// same kernel and give the same bits.
bool attention_f64_supported(const float* qkv, int qkv_stride, int n_seq, int S, int H, int dh) {
  return (dh == 32 || dh == 64) && S >= 8 && S <= 128 && qkv_stride % 4 == 0 && qkv_stride < 1 << 24 && ((uintptr_t)qkv & 15) == 0 &&
         (int64_t)n_seq * H * ((S + 15) / 16) * 256 <= (int64_t)UINT32_MAX;
}

bool launch_attention_f64(hipStream_t st, const float* qkv, int qkv_stride, float* out, int n_seq, int S, int H, int Hkv, int dh, const int32_t* cu,
                          int E, int rows_per_copy) {
  if (!attention_f64_supported(qkv, qkv_stride, n_seq, S, H, dh)) return false;
  const int64_t blocks = (int64_t)n_seq * H * ((S + 15) / 16);
  const float scale = (float)(1.0 / sqrt((double)dh));
#define MPZ_ATT(DH, MAXT) attention_f64_kernel<DH, MAXT><<<(unsigned)blocks, 256, 0, st>>>(qkv, qkv_stride, out, S, H, Hkv, scale, cu, E, rows_per_copy)
  if (dh == 64) { if (S <= 32) MPZ_ATT(64, 2); else if (S <= 64) MPZ_ATT(64, 4); else MPZ_ATT(64, 8); }
  else { if (S <= 32) MPZ_ATT(32, 2); else if (S <= 64) MPZ_ATT(32, 4); else MPZ_ATT(32, 8); }
#undef MPZ_ATT
  return true;
}

// 16 x 16 tiles below a block of 32 x 32 per CU (256 x 128 x 128: 32 against 128 blocks).  Above, the tile whose blocks, dealt to 256
// CUs, leave the fullest of them the least work: 768 x 768 is 2.25 blocks of 32 x 32 (three on some) or one of 48 x 48 per CU
bool launch_linear_f64(hipStream_t st, const LinearArgs& a) {
  if (a.dtype != MPZ_DTYPE_F32 || a.K % 4 || a.K >= 1 << 22 || (((uintptr_t)a.x | (uintptr_t)a.w) & 15)) return false;
  auto tiles = [&](int t) { return dim3((unsigned)((a.N + t - 1) / t), (unsigned)((a.M + t - 1) / t)); };
  auto work = [&](int t) { return ((long)tiles(t).x * tiles(t).y + 255) / 256 * t * t; };
  if ((long)tiles(32).x * tiles(32).y < 256) linear_f64_kernel<1><<<tiles(16), 256, 0, st>>>(a);
  else if (work(48) <= work(32)) linear_f64_kernel<3><<<tiles(48), 256, 0, st>>>(a);
  else linear_f64_kernel<2><<<tiles(32), 256, 0, st>>>(a);
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
