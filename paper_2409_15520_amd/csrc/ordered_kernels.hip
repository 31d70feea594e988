// bf16 models, copies whose rows are no multiple of 32: the adapted linears and the LoRA bottleneck with the sums, bit for bit,
// of the shape-agnostic kernels (linear_kernel and lora_down_kernel of simple_kernels.hip), on the fp32 matrix instructions.
// Every sum is one binary32 chain, sum = fma(x_k, w_k, sum) for k = 0, 1, ..., K - 1: v_mfma_f32_32x32x2 and v_mfma_f32_16x16x4
// take their 2 and 4 products one after another in that order, each fused and rounded to nearest (bf16, fp32, 2^-30 ... 2^30
// and subnormal operands: every bit of 1024 chains of 512).  The bf16 matrix instructions add in another order; on such
// batches a step's two-point differences (small copies: few tokens, so little averages out) moved by more than the 1e-3 that
// a step's masters are held to.
// Bound by the fp32 matrix instructions, which run on the vector lanes (256 FLOP per clock and CU, a sixteenth of bf16; no other
// vector instruction runs beside them, on any wave of the SIMD: loops of theirs with one v_perm each, one in turn / eight in turn,
// reach 104 / 129 TFLOP/s with one wave per SIMD, 115 / 133 with four, 155 without).  So the operands of a step are widened together,
// addresses are constants, and the next step's operands are read before.  1848 x 2560 x 2048: 222 -> 199 us (one instruction of
// 32 x 32 x 2 and its two v_perm in turn: 87 TFLOP/s); a 1.1B-shaped block, 8 copies of 231 rows, adapters on all four
// projections: 2157 us with the shape-agnostic kernels, 631 -> 567 us with these.
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

// out = epilogue(x W^T): a block of four waves, each 16 NT tokens x 16 NT features; K-tiles of 64 go straight into a ring of ST LDS
// stages.  MFMA layout (16x16x4): lane l holds A[l % 16][l / 16], B[l / 16][l % 16] and, of the result, D[4 (l / 16) + r][l % 16],
// r = 0..3: rows are features, columns tokens.  The four lanes of a row read the same eight k and take the ones of their quarter.
template <int NT, int ST>
__global__ void __launch_bounds__(256) linear_ordered_kernel(LinearArgs a, int vec) {
  constexpr int BK = 64, BT = 32 * NT, PER = BT / 16;      // k per stage; rows of either operand; fetches of a wave per stage (8 rows of 128 bytes each)
  constexpr uint32_t HALF_STAGE = BT * BK * 2, STAGE = 2 * HALF_STAGE;
  __shared__ __align__(128) unsigned char smem[ST * STAGE];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, lq = lane >> 4;
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
  const int bm = (first_m + rr % gsz) * BT, bn = rr / gsz * BT;
  const int m0 = bm + (wave >> 1) * 16 * NT, n0 = bn + (wave & 1) * 16 * NT;

  // buffers hold the tile's rows: rows past M or N fall outside (zeros), and their results are not stored.  Waves 0 and 1 fetch the
  // token rows, 2 and 3 the weight rows; 16-byte chunk c of row r lies at c ^ ((r / 2) % 8)
  const size_t row_b = (size_t)a.K * 2;
  const bool weights = wave >= 2;
  const int r_first = weights ? bn : bm, r_end = weights ? a.N : a.M, left = r_end - r_first < BT ? r_end - r_first : BT;
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
  const uint32_t sel = 0x00000c0cu | (uint32_t)(2 * lq) << 16 | (uint32_t)(2 * lq + 1) << 24;    // element lq of four bf16, as fp32
  auto take = [&](uint32_t lo, uint32_t hi) { return __uint_as_float(__builtin_amdgcn_perm(hi, lo, sel)); };
  const unsigned char* px[8];                              // this lane's piece of each eight k of its first row, in stage 0
  const unsigned char* pw[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const uint32_t o = (uint32_t)l16 * 128u + ((uint32_t)c * 16u ^ ((uint32_t)((l16 >> 1) & 7) * 16u));
    px[c] = smem + (wave >> 1) * 16 * NT * 128 + o;
    pw[c] = smem + HALF_STAGE + (wave & 1) * 16 * NT * 128 + o;
  }

  f32x4 acc[NT][NT];                                       // [features][tokens]
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nk = a.K / BK;
#pragma unroll
  for (int t = 0; t < ST - 1; ++t)
    if (t < nk) fetch(t, t);
  for (int k0 = 0; k0 < nk; k0 += ST)
#pragma unroll
    for (int st = 0; st < ST; ++st) {                      // (the stage is a constant: no address arithmetic, see above)
      const int kt = k0 + st;
      if (kt >= nk) break;                                 // (uniform)
      // K-tile kt has landed for the whole block, and every wave is done with the stage that the next fetch overwrites
      wait_fetched<PER, ST - 2>(nk - 1 - kt);
      if (kt + ST - 1 < nk) fetch(kt + ST - 1, (st + ST - 1) % ST);
      u32x4 x[2][NT], w[2][NT];
      auto read = [&](int c) {
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          x[c & 1][j] = *(const u32x4*)(px[c] + st * STAGE + j * 2048);
          w[c & 1][j] = *(const u32x4*)(pw[c] + st * STAGE + j * 2048);
        }
      };
      read(0);
#pragma unroll
      for (int c = 0; c < BK / 8; ++c) {
        __builtin_amdgcn_sched_barrier(0);
        if (c + 1 < BK / 8) read(c + 1);
        float fx[2][NT], fw[2][NT];
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
          for (int j = 0; j < NT; ++j) {
            fx[e][j] = take(x[c & 1][j][2 * e], x[c & 1][j][2 * e + 1]);
            fw[e][j] = take(w[c & 1][j][2 * e], w[c & 1][j][2 * e + 1]);
          }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
          for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[e][i], fx[e][j], acc[i][j], 0, 0, 0);
      }
    }
  // (no barriers below)
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int mj = m0 + j * 16, m = mj + l16, mrow = m < a.M ? m : a.M - 1;
    if (mj >= a.M) continue;                               // (uniform)
    // per-copy low-rank term: a chain of its own over the rank, for every copy that has rows in the tile; its sum goes to the
    // rows of that copy alone (a result column depends on its own row of t only)
    const int last_row = mj + 15 < a.M ? mj + 15 : a.M - 1;
    const int first_copy = mj / a.rows_per_copy, last_copy = last_row / a.rows_per_copy;
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int ni = n0 + i * 16;
      if (ni >= a.N) continue;                             // (uniform)
      for (int s = 0; s < a.n_seg; ++s) {
        const LoraSeg& sg = a.seg[s];
        if (ni + 15 < sg.col_begin || ni >= sg.col_end) continue;
        const int kout = sg.col_end - sg.col_begin, col = ni + l16;
        const bool in = col >= sg.col_begin && col < sg.col_end;
        const bf16_t* t = (const bf16_t*)sg.t + (int64_t)mrow * sg.t_stride + sg.t_off;
        for (int copy = first_copy; copy <= last_copy; ++copy) {
          const float* B = sg.Bc + (int64_t)copy * sg.copy_stride + (in ? col - sg.col_begin : 0);
          f32x4 dl = {0.f, 0.f, 0.f, 0.f};
          for (int r = lq; r < a.rank + lq; r += 4) {      // (ranks are multiples of 4)
            float b0 = B[(int64_t)r * kout], none = 0.f;
            factors(b0, none);
            dl = __builtin_amdgcn_mfma_f32_16x16x4f32(b0, bf16_to_f32(t[r]), dl, 0, 0, 0);
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int n = ni + 4 * lq + e;
            acc[i][j][e] = n >= sg.col_begin && n < sg.col_end && m / a.rows_per_copy == copy ? acc[i][j][e] + dl[e] : acc[i][j][e];
          }
        }
      }
      const int n = ni + 4 * lq;
      if (m >= a.M || n >= a.N) continue;
      const int64_t o = (int64_t)m * a.N + n;
      f32x4 v = acc[i][j];
      if (vec) {                                           // N a multiple of 4, pointers on 16 bytes
        if (a.bias != nullptr) v += *(const f32x4*)(a.bias + n);
        if (a.act == MPZ_ACT_RELU) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
        }
        if (a.residual != nullptr) v += *(const f32x4*)(a.residual + o);
        if (a.out_kind == 0) {
          uint32_t lo = (uint32_t)f32_to_bf16(v[0]).bits | (uint32_t)f32_to_bf16(v[1]).bits << 16;
          uint32_t hi = (uint32_t)f32_to_bf16(v[2]).bits | (uint32_t)f32_to_bf16(v[3]).bits << 16;
          *(uint64_t*)((bf16_t*)a.out + o) = (uint64_t)hi << 32 | lo;
        } else {
          *(f32x4*)((float*)a.out + o) = v;                // (bf16 models stage in fp32)
        }
        continue;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (n + e >= a.N) continue;
        float y = v[e];
        if (a.bias != nullptr) y += a.bias[n + e];
        if (a.act == MPZ_ACT_RELU) y = y > 0.f ? y : 0.f;
        if (a.residual != nullptr) y += a.residual[o + e];
        if (a.out_kind == 0) ((bf16_t*)a.out)[o + e] = f32_to_bf16(y);
        else ((float*)a.out)[o + e] = y;
      }
    }
  }
}

// LoRA bottleneck t = bf16(scale * x A_c): a block of four waves per 64 rows of one copy and 16 columns, a wave per 16 rows.  The columns
// are those of all targets side by side, so ranks below 16 share a tile (a lane fetches four columns, which are one target's); K-tiles of 64 (64 rows of x, 64 x 16 of the factor) go straight into a ring of LDS stages.  The factor's values become
// what the contraction sees one K-tile ahead, in place, a quarter by each wave.  Bound by the chain: K / 4 dependent instructions
// of 32 clocks, and vector instructions do not run beside it (1848 rows, K = 2048: 29 -> 21 us; a wave
// per 16 rows with both operands from memory, converting the factor for itself, waited for its requests).  Lane l holds x[l % 16][k = l / 16] and
// A[k = l / 16][column l % 16] of every four k and, of the result, D[4 (l / 16) + r][l % 16], r = 0..3.  K is a multiple of 32: of a
// last K-tile that is half outside, the chain takes the half inside (what lies behind it in the stage is never multiplied).
struct DownFactors { const float* first; uint32_t bytes, off[4]; };           // the targets' factors of a copy as one buffer
template <int BK, int ST>
__global__ void __launch_bounds__(256) lora_down_ordered_kernel(LoraDownArgs a, DownFactors fa, int tiles_per_copy, int col_tiles) {
  constexpr int FX = BK / 32, FA = BK / 64, PER = FX + FA;                     // fetches of a wave per stage: of x, of the factor
  constexpr uint32_t CPR = BK / 8, RPF = 64 / CPR;                             // 16-byte chunks of a row, rows of a fetch
  constexpr uint32_t XBYTES = 64 * BK * 2, STAGE = XBYTES + BK * 64;
  extern __shared__ __align__(16) unsigned char lora_smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, lq = lane >> 4;
  const int c0 = blockIdx.x % col_tiles * 16, rest = blockIdx.x / col_tiles, R = a.n_targets * a.rank;
  const int copy = rest / tiles_per_copy, r0 = rest % tiles_per_copy * 64;     // first row inside the copy
  const size_t row_b = (size_t)a.K * 2;
  const int rows = a.rows_per_copy - r0 < 64 ? a.rows_per_copy - r0 : 64;      // rows past the copy read zeros and are not stored
  const i32x4 rsrcX = buffer_of((const char*)a.x + ((size_t)copy * a.rows_per_copy + r0) * row_b, (size_t)rows * row_b);
  const i32x4 rsrcA = buffer_of(fa.first + (int64_t)copy * a.copy_stride, fa.bytes);
  const uint32_t row_a = (uint32_t)a.rank * 4u;
  auto swizzle = [](uint32_t row) { return BK == 64 ? row >> 1 & 7u : row & 15u; };          // chunk c of a row lies at c ^ this
  uint32_t voffX[FX];
#pragma unroll
  for (int t = 0; t < FX; ++t) {
    const uint32_t row = (uint32_t)(wave * FX + t) * RPF + lane / CPR;
    voffX[t] = row * (uint32_t)row_b + ((lane % CPR) ^ swizzle(row)) * 16u;
  }
  const int j = c0 + (lane & 3) * 4;                       // the first of this lane's four columns; past the last one: aimed outside (zeros)
  uint32_t voffA = 0x80000000u;
#pragma unroll
  for (int t = 0; t < 4; ++t)
    if (j >= t * a.rank && j < (t + 1) * a.rank && j < R) voffA = fa.off[t] + (uint32_t)(wave * 16 + (lane >> 2)) * row_a + (uint32_t)(j - t * a.rank) * 4u;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lora_smem;
  auto fetch = [&](int kt, int st) {
    const uint32_t base = lds0 + (uint32_t)st * STAGE;
#pragma unroll
    for (int t = 0; t < FX; ++t) fetch_rows<4>(rsrcX, voffX[t], (uint32_t)kt * (BK * 2), base + (uint32_t)(wave * FX + t) * 1024u);
#pragma unroll
    for (int t = 0; t < FA; ++t)
      fetch_rows<4>(rsrcA, voffA, (uint32_t)(kt * BK + t * 64) * row_a, base + XBYTES + (uint32_t)(t * 4 + wave) * 1024u);
  };
  auto convert = [&](int st) {
#pragma unroll
    for (int t = 0; t < FA; ++t) {
      f32x4* p = (f32x4*)(lora_smem + (uint32_t)st * STAGE + XBYTES) + t * 256 + tid;
      f32x4 v = *p;
      float f[4] = {v[0], v[1], v[2], v[3]};
      factors(f[0], f[1]);
      factors(f[2], f[3]);
      *p = f32x4{f[0], f[1], f[2], f[3]};
    }
  };
  const uint32_t sel = 0x00000c0cu | (uint32_t)(2 * lq) << 16 | (uint32_t)(2 * lq + 1) << 24;    // element lq of four bf16
  const uint32_t baseX = (uint32_t)(wave * 16 + l16) * (BK * 2), sw = swizzle(l16) * 16u, baseA = XBYTES + (uint32_t)(lq * 16 + l16) * 4u;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  const int nk = (a.K + BK - 1) / BK;
  const bool half = BK == 64 && a.K % BK != 0;             // the last K-tile has 32 k
#pragma unroll
  for (int t = 0; t < ST - 1; ++t)
    if (t < nk) fetch(t, t);
  wait_fetched<PER, ST - 2>(nk - 1);
  convert(0);
  int st = 0;
  for (int kt = 0; kt < nk; ++kt) {
    // K-tile kt + 1 has landed, the factor of kt is converted (its writes are awaited with the fetches), and every wave is done with
    // the stage that the next fetch overwrites
    wait_fetched<PER, ST - 3>(nk - 2 - kt);
    if (kt + ST - 1 < nk) fetch(kt + ST - 1, st == 0 ? ST - 1 : st - 1);
    const unsigned char* sp = lora_smem + (uint32_t)st * STAGE;
    st = st + 1 == ST ? 0 : st + 1;
    u32x4 x[2][8];
    float f[2][16];
    auto read = [&](int h) {                               // 64 k
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        x[h & 1][c] = *(const u32x4*)(sp + baseX + ((uint32_t)(h * 8 + c) * 16u ^ sw));
#pragma unroll
        for (int e = 0; e < 2; ++e) f[h & 1][2 * c + e] = *(const float*)(sp + baseA + (h * 16 + 2 * c + e) * 256);
      }
    };
    read(0);
    if (kt + 1 < nk) convert(st);
#pragma unroll
    for (int h = 0; h < BK / 64; ++h) {
      __builtin_amdgcn_sched_barrier(0);
      if (h + 1 < BK / 64) read(h + 1);
      float fx[16];
#pragma unroll
      for (int c = 0; c < 8; ++c)
#pragma unroll
        for (int e = 0; e < 2; ++e) fx[2 * c + e] = __uint_as_float(__builtin_amdgcn_perm(x[h & 1][c][2 * e + 1], x[h & 1][c][2 * e], sel));
      __builtin_amdgcn_sched_barrier(0);                   // (the chain without vector instructions between its links)
#pragma unroll
      for (int i = 0; i < 8; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fx[i], f[h & 1][i], acc, 0, 0, 0);
      if (half && kt + 1 == nk) break;                     // (uniform)
#pragma unroll
      for (int i = 8; i < 16; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fx[i], f[h & 1][i], acc, 0, 0, 0);
    }
  }
  if (c0 + l16 >= R) return;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int rc = r0 + wave * 16 + 4 * lq + r;
    if (rc < a.rows_per_copy) ((bf16_t*)a.t)[(copy * (int64_t)a.rows_per_copy + rc) * R + c0 + l16] = f32_to_bf16(acc[r] * a.scale);
  }
}

template <int BK, int ST>
bool launch_down(hipStream_t st, const LoraDownArgs& a, const DownFactors& fa, unsigned blocks, int tiles, int cols) {
  constexpr int lds = ST * (64 * BK * 2 + BK * 64);
  static const hipError_t attr_status = hipFuncSetAttribute((const void*)lora_down_ordered_kernel<BK, ST>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (attr_status != hipSuccess) {                         // (the caller takes the shape-agnostic kernel: same bits)
    (void)hipGetLastError();
    return false;
  }
  lora_down_ordered_kernel<BK, ST><<<blocks, 256, lds, st>>>(a, fa, tiles, cols);
  return true;
}

}  // namespace

// whole K-tiles, operands that begin on 16 bytes and stay below 2 GiB per tile of 64 rows, no GELU (its erff would be contracted in
// other surroundings)
bool launch_linear_ordered(hipStream_t st, const LinearArgs& a) {
  if (a.dtype != MPZ_DTYPE_BF16 || a.K % 64 || a.K < 64 || a.K >= 1 << 24 || a.act == MPZ_ACT_GELU_ERF || (((uintptr_t)a.x | (uintptr_t)a.w) & 15)) return false;
  const int vec = a.N % 4 == 0 && (((uintptr_t)a.out | (uintptr_t)a.residual | (uintptr_t)a.bias) & 15) == 0;
  const long small = (long)((a.N + 31) / 32) * ((a.M + 31) / 32);
  const dim3 g32((a.N + 31) / 32, (a.M + 31) / 32), g64((a.N + 63) / 64, (a.M + 63) / 64);
  // up to two tiles of 64 x 64 per CU's worth of rows and columns, 16 x 16 per wave: a quarter of the chain per wave, four times the
  // waves (154 rows, Q|K|V and O of the 1.1B shape: 136 -> 60 us, 100 in the larger tiles; 3696 rows of the 125M shape: 217 / 206)
  if (small <= 2048) linear_ordered_kernel<1, 3><<<g32, 256, 0, st>>>(a, vec);
  else linear_ordered_kernel<2, 2><<<g64, 256, 0, st>>>(a, vec);
  return true;
}

// whole pieces of 32 k (bf16 models of any such width take their bottleneck here, 32 modulo 64 among them: widths of 96 / 352 / 1312
// with the shape-agnostic kernel, a whole block of 1848 tokens took 4 - 10 / 14 - 24 / 8 - 15 % longer)
int64_t lora_down_ordered_blocks(const LoraDownArgs& a) {
  if (a.dtype != MPZ_DTYPE_BF16 || a.K % 32 || a.K < 32 || a.rank % 4 || a.copy_stride % 4 || ((uintptr_t)a.x & 15) || a.T % a.rows_per_copy) return 0;
  if ((size_t)a.K * 128 >= (size_t)1 << 31) return 0;
  uintptr_t lo = (uintptr_t)a.Ac[0], hi = lo;
  for (int t = 0; t < a.n_targets; ++t) {
    const uintptr_t p = (uintptr_t)a.Ac[t];
    if (p & 15) return 0;
    lo = p < lo ? p : lo; hi = p > hi ? p : hi;
  }
  if (hi - lo + (size_t)a.K * a.rank * 4 >= (size_t)1 << 31) return 0;       // one buffer (a layer's factors lie together)
  const int64_t blocks = (int64_t)(a.T / a.rows_per_copy) * ((a.rows_per_copy + 63) / 64) * ((a.n_targets * a.rank + 15) / 16);
  return blocks * 256 > (int64_t)UINT32_MAX ? 0 : blocks;
}

bool launch_lora_down_ordered(hipStream_t st, const LoraDownArgs& a) {
  const int64_t blocks = lora_down_ordered_blocks(a);
  if (blocks == 0) return false;
  const int tiles = (a.rows_per_copy + 63) / 64, cols = (a.n_targets * a.rank + 15) / 16;
  DownFactors fa{a.Ac[0], 0, {0, 0, 0, 0}};
  for (int t = 1; t < a.n_targets; ++t) fa.first = a.Ac[t] < fa.first ? a.Ac[t] : fa.first;
  for (int t = 0; t < a.n_targets; ++t) {
    fa.off[t] = (uint32_t)((uintptr_t)a.Ac[t] - (uintptr_t)fa.first);
    const uint32_t end = fa.off[t] + (uint32_t)a.K * (uint32_t)a.rank * 4u;
    fa.bytes = end > fa.bytes ? end : fa.bytes;
  }
  // few blocks: twice the bytes in flight and half the barriers (a block has the CU to itself)
  if (blocks <= 256 && a.K % 128 == 0) return launch_down<128, 6>(st, a, fa, (unsigned)blocks, tiles, cols);
  return launch_down<64, 6>(st, a, fa, (unsigned)blocks, tiles, cols);
}

}  // namespace mpz
