// Pieces shared by the bf16 MFMA GEMM kernels: fragment types, the per-copy low-rank term and the epilogue.
#pragma once
#include "common.h"
#include "../../include/mpz.h"

namespace mpz {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;     // 16-byte chunk in registers (native vector type)
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;

__device__ __forceinline__ bf16x8 as_frag(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ float gelu_erf(float v) { return 0.5f * v * (1.0f + erff(v * 0.70710678118654752440f)); }
// the same arithmetic as a real call: where all of a block's accumulators are live around it, inlining erff 128 times
// would cost registers that the common path (no GELU) never needs
__device__ __noinline__ float gelu_erf_call(float v) { return gelu_erf(v); }

// Per-copy low-rank term: extra K-steps with the packed factor [B_hi | B_lo] of a copy against the duplicated
// bottleneck activations [t | t].  Copies are whole multiples of 32 rows, so every 32-row MFMA tile belongs to one copy
// (a block tile may span several); segments are aligned to the block tile.
template <int NI, int NJ>
__device__ __forceinline__ void add_low_rank(const MfmaGemmArgs& a, f32x16 (&acc)[NI][NJ], int m0, int n0, int wm, int wn, int lane) {
  const int lrow = lane & 31, lhalf = lane >> 5;
  for (int s = 0; s < a.n_seg; ++s) {
    const MfmaLoraSeg& sg = a.seg[s];
    if (n0 < sg.col_begin || n0 >= sg.col_end) continue;
    const uint16_t* tp = (const uint16_t*)sg.tp;
    for (int ks = 0; ks < sg.rp; ks += 16) {
      // all fragments of the step first, then its MFMAs: the block waits for L2 once per step, not once per tile
      bf16x8 lx[NJ], lw[NJ][NI];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        int mt = m0 + wm + j * 32;                       // first row of this MFMA tile
        mt = mt < a.M ? mt : a.M - 32;                   // tiles past the end compute discarded values in bounds
        const int copy = mt / a.rows_per_copy;
        const uint16_t* bp = (const uint16_t*)sg.bp + (size_t)copy * sg.copy_stride;
        lx[j] = as_frag(*(const u32x4*)(tp + (size_t)(mt + lrow) * sg.rp + ks + lhalf * 8));
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          const int n = n0 + wn + i * 32 + lrow - sg.col_begin;
          lw[j][i] = as_frag(*(const u32x4*)(bp + (size_t)n * sg.rp + ks + lhalf * 8));
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < NI; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lw[j][i], lx[j], acc[i][j], 0, 0, 0);
    }
  }
}

// The same on 16 x 16 tiles (v_mfma_f32_16x16x32): lane l holds features 4 (l / 16) .. + 3 of token l % 16.
template <int NI, int NJ>
__device__ __forceinline__ void add_low_rank_16(const MfmaGemmArgs& a, f32x4 (&acc)[NI][NJ], int m0, int n0, int wm, int wn, int lane) {
  const int l16 = lane & 15, lq = lane >> 4;
  const u32x4 zero = {0u, 0u, 0u, 0u};
  for (int s = 0; s < a.n_seg; ++s) {
    const MfmaLoraSeg& sg = a.seg[s];
    if (n0 < sg.col_begin || n0 >= sg.col_end) continue;
    for (int ks = 0; ks < sg.rp; ks += 32) {
      const bool here = ks + lq * 8 < sg.rp;               // (rank <= 8: the upper half of the K-step is zero)
      const int k8 = here ? ks + lq * 8 : 0;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int mt = m0 + wm + j * 16;
        if (mt >= a.M) continue;                           // (uniform)
        u32x4 x = *(const u32x4*)((const uint16_t*)sg.tp + (size_t)(mt + l16) * sg.rp + k8);
        x = here ? x : zero;
        const uint16_t* bp = (const uint16_t*)sg.bp + (size_t)(mt / a.rows_per_copy) * sg.copy_stride + k8;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          u32x4 w = *(const u32x4*)(bp + (size_t)(n0 + wn + i * 16 + l16 - sg.col_begin) * sg.rp);
          w = here ? w : zero;
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_frag(w), as_frag(x), acc[i][j], 0, 0, 0);
        }
      }
    }
  }
}

// Fused cross-entropy: the logits never leave the registers.  A lane holds NI * 16 columns of token row lrow (the other
// half of the row's columns sits in lane ^ 32): row maximum, sum of exponentials against it, and the target's logit if it
// falls into this wave tile.
template <int BN, int WGN, int WGM, int NW, int NI, int NJ>
__device__ __forceinline__ void ce_partials(const MfmaGemmArgs& a, f32x16 (&acc)[NW][NI][NJ], int m0, int n0, int wm, int wn, int wave,
                                            int lane) {
  const int lrow = lane & 31, lhalf = lane >> 5;
  constexpr float LOG2E = 1.4426950408889634f;
  const int slot = (n0 / BN) * WGN + wave / WGM;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int m = m0 + wm + j * 32 + lrow;
    const int tg = m < a.M ? a.ce_target[m] : -1;
    float mx = -1e30f, tl = 0.f;
    bool has = false;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int n = n0 + wn + i * 32 + g * 8 + lhalf * 4 + e;
          const float v = acc[0][i][j][g * 4 + e];
          if (n < a.N) mx = v > mx ? v : mx;
          if (n == tg) { tl = v; has = true; }
        }
    const float other = __shfl_xor(mx, 32);
    mx = other > mx ? other : mx;
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int n = n0 + wn + i * 32 + g * 8 + lhalf * 4 + e;
          if (n < a.N) sum += __builtin_amdgcn_exp2f((acc[0][i][j][g * 4 + e] - mx) * LOG2E);
        }
    sum += __shfl_xor(sum, 32);
    if (m < a.M) {
      if (lhalf == 0) {
        a.ce_max[(size_t)slot * a.M + m] = mx;
        a.ce_sum[(size_t)slot * a.M + m] = sum;
      }
      if (has) a.ce_tlogit[m] = tl;
    }
  }
}

// What follows the accumulation: bias, activation or gating, rotary embedding, fused cross-entropy, residual, output
// type.  acc[d][i][j]: MFMA tile i (32 output features) x j (32 tokens) of the wave tile at (n0 + wn, m0 + wm); d = 1:
// the second weight tile of a dual launch.  smem: the block's dynamic LDS, all operand traffic in it finished.
template <int BN, int WGN, int WGM, int NW, int NI, int NJ, int HP>
__device__ __forceinline__ void gemm_epilogue(const MfmaGemmArgs& a, f32x16 (&acc)[NW][NI][NJ], unsigned char* smem, int m0, int n0,
                                              int wm, int wn, int wave, int lane, bool raw, int split) {
  constexpr bool DUAL = NW == 2;
  constexpr int TN = NI * 32;
  const int lrow = lane & 31, lhalf = lane >> 5;
  // Epilogue, part 1 (accumulator layout: a lane holds, for token m = lrow, features nb + g*8 + lhalf*4 + (0..3),
  // g = 0..3, of every MFMA tile): bias, activation or gating, rotary embedding -- everything that needs no
  // other token's data -- written back into acc[0].
  if (!DUAL || !raw) {                                     // (raw sums of one weight tile: plus zero, without a branch around the accumulators)
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      int n = n0 + wn + i * 32 + g * 8 + lhalf * 4;
      n = n < a.N ? n : 0;                                 // columns past N are never stored
      f32x4 bg = {0.f, 0.f, 0.f, 0.f}, bu = bg;
      if (a.bias != nullptr && !raw) {
        bg = *(const f32x4*)(a.bias + n);
        if (DUAL) bu = *(const f32x4*)(a.bias + a.dual_offset + n);
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float v = acc[0][i][j][g * 4 + e] + bg[e];
          if (DUAL) {
            const float u = acc[NW - 1][i][j][g * 4 + e] + bu[e];
            v = silu_mul_f32(v, u);                        // SiLU(gate) * up
          }
          acc[0][i][j][g * 4 + e] = v;
        }
    }
  }
  if (!raw && !DUAL && a.act == MPZ_ACT_RELU) {            // one uniform branch, no select where there is no ReLU
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[0][i][j][e] = !(acc[0][i][j][e] > 0.f) ? 0.f : acc[0][i][j][e];
  }
  if (!raw && !DUAL && a.act == MPZ_ACT_GELU_ERF) {                // rare (no workload of the paper uses it): one cold loop
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[0][i][j][e] = gelu_erf_call(acc[0][i][j][e]);
  }
  if constexpr (HP > 0) {
    static_assert(!DUAL && NI >= 2 * HP && NI % (2 * HP) == 0, "a wave tile must hold whole heads");
    if (!raw && n0 < a.rope_cols) {
      // q / k columns: y_lo = x_lo cos - x_hi sin, y_hi = x_hi cos + x_lo sin with (lo, hi) = columns (c, c + d_head/2)
      const int half = 32 * HP;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        int m = m0 + wm + j * 32 + lrow;
        m = m < a.M ? m : a.M - 1;
        const int pos = a.rope_pos != nullptr ? a.rope_pos[m % a.S] : m % a.S;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          if ((i / HP) % 2 != 0) continue;                  // upper halves are rotated together with their lower half
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int c = (i % HP) * 32 + g * 8 + lhalf * 4;  // column inside the lower half of the head
            const f32x4 cs = *(const f32x4*)(a.rope_cos + (size_t)pos * half + c);
            const f32x4 sn = *(const f32x4*)(a.rope_sin + (size_t)pos * half + c);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float lo = acc[0][i][j][g * 4 + e], hi = acc[0][i + HP][j][g * 4 + e];
              // one rounded product, one fma: the same two operations as the stand-alone rotary kernel, so a pass
              // that takes that kernel (tile too narrow for a whole head) gives the same bits
              acc[0][i][j][g * 4 + e] = fmaf(lo, cs[e], -__fmul_rn(hi, sn[e]));
              acc[0][i + HP][j][g * 4 + e] = fmaf(hi, cs[e], __fmul_rn(lo, sn[e]));
            }
          }
        }
      }
    }
  }

  if (a.ce_max != nullptr) {                               // cross-entropy mode: nothing is stored to `out`
    ce_partials<BN, WGN, WGM, NW, NI, NJ>(a, acc, m0, n0, wm, wn, wave, lane);
    return;
  }

  // Epilogue, part 2: each wave turns its tile around in a private LDS strip, 32 tokens at a time, so that a lane
  // ends up with 4 consecutive features of a token and consecutive lanes with consecutive features: residual reads
  // and output stores then cover whole 128-byte lines (straight from the accumulator layout a store instruction
  // would touch 32 token rows with 16 bytes each).
  constexpr int EPS = TN + 4;                              // strip row stride in floats: conflict-free 16-byte columns
  constexpr int LPR = TN / 4;                              // lanes per token row on the way out
  float* ep = (float*)smem + wave * 32 * EPS;
  __syncthreads();                                         // every wave is done with the operand stages
  // With split K the raw sums of this split go out instead (fp32, no bias / activation / residual; both weight tiles
  // of a dual launch, the second N columns to the right): partial[split][m][d N + n], row stride ldp.
  const int nd = raw ? NW : 1;
  const int ld = raw ? a.ldp : a.ldo;
  float* const praw = raw ? a.partial + (size_t)split * a.M * a.ldp : nullptr;
#pragma unroll
  for (int d = 0; d < NW; ++d) {
  if (d >= nd) break;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 v = {acc[d][i][j][g * 4], acc[d][i][j][g * 4 + 1], acc[d][i][j][g * 4 + 2], acc[d][i][j][g * 4 + 3]};
        *(f32x4*)(ep + lrow * EPS + i * 32 + g * 8 + lhalf * 4) = v;
      }
    // RB pieces at a time: all their residual loads are issued before the first is used (a piece past M or N reads
    // a clamped, in-bounds address and is not stored), and the kind of output is decided outside the loops
    constexpr int R = 32 * LPR / 64, RB = R % 8 == 0 ? 8 : 4;
    static_assert(R % RB == 0, "pieces must deal out evenly to the batches");
#pragma unroll
    for (int r0 = 0; r0 < R; r0 += RB) {
      f32x4 v[RB];
      size_t o[RB];
      bool ok[RB];
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const int idx = (r0 + r) * 64 + lane, row = idx / LPR, c4 = idx % LPR;
        const int m = m0 + wm + j * 32 + row, n = n0 + wn + c4 * 4;
        ok[r] = m < a.M && n < a.N;
        o[r] = (size_t)(m < a.M ? m : a.M - 1) * ld + (n < a.N ? n : 0) + (raw ? d * a.N : 0);
        v[r] = *(const f32x4*)(ep + row * EPS + c4 * 4);
      }
      if (raw) {
#pragma unroll
        for (int r = 0; r < RB; ++r)
          if (ok[r]) *(f32x4*)(praw + o[r]) = v[r];
        continue;
      }
      if (a.residual != nullptr) {
        f32x4 rs[RB];
#pragma unroll
        for (int r = 0; r < RB; ++r) rs[r] = *(const f32x4*)(a.residual + o[r]);
#pragma unroll
        for (int r = 0; r < RB; ++r) v[r] += rs[r];
      }
      if (a.out_f32) {
#pragma unroll
        for (int r = 0; r < RB; ++r)
          if (ok[r]) *(f32x4*)((float*)a.out + o[r]) = v[r];
      } else {
#pragma unroll
        for (int r = 0; r < RB; ++r)
          if (ok[r]) {
            u32x2 pk = {pack_bf16x2(v[r][0], v[r][1]), pack_bf16x2(v[r][2], v[r][3])};
            *(u32x2*)((uint16_t*)a.out + o[r]) = pk;
          }
      }
    }
  }
  }
}

}  // namespace
}  // namespace mpz
