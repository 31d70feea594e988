// The large bf16 GEMM: 256 output features x 256 tokens per tile (SwiGLU: 2 x 128 features), four waves of 128 x 128 (one
// per SIMD), operands fetched straight into LDS, one persistent block per CU.
//
// What bounds it: the matrix cores under the clock the chip holds on real operand bits.  A loop of MFMAs on a 128 x 128
// wave tile with its fragment reads reaches 1780 TFLOP/s here (1612 on the 128 x 64 wave tile of eight waves per block,
// which reads half as many LDS bytes again per MFMA); everything below is there to keep the loop at that rate and to
// take the edges of a tile off the clock.  v_mfma_f32_16x16x32_bf16 gives the bits of two v_mfma_f32_32x32x16_bf16 in a row
// and draws less power: the same kernel built on the 32 x 32 shape is 10-12 % slower (48.7 against 54.6 us per round of 256
// tiles at K = 2048).  Measured in turn with the register-staged 8-wave tile it replaces, one box (bf16 out, M x N x K; boxes differ
// by 5 %): 8192 x 12288 x 4096 718 -> 640 us (1290 TFLOP/s), 8192 x 4096 x 4096 221 -> 191, 8192 x 4096 x 11008 560 -> 491 (1500),
// 32768 x 8192 x 2048 953 -> 798, 65536 x 2560 x 2048 580 -> 502; on another box SwiGLU 65536 x 5632 x 2048 2426 -> 2105 and, with
// the fp32 residual, 65536 x 2048 x 2048 600 -> 487.
//   * A K-tile (64) is four pieces of 128 rows x 128 bytes: weights W0, W1 and tokens X0, X1, each wave owning 64 rows of
//     every piece.  Two LDS stages of four pieces; a piece's slot is free as soon as its fragments are in registers, so
//     a fetch has one and a half K-tiles to arrive, without registers to stage it.
//   * A K-tile is four phases of 16 MFMAs, one per (W piece, X piece), in the order W0 F, W0 S, W1 S, W1 F with (F, S) =
//     (X0, X1) on even and (X1, X0) on odd K-tiles: each phase reads the fragments that the next phase needs into the
//     registers that the previous one has finished with, across the block's two barriers per K-tile as well.
//   * The K order of every accumulator is that of the other tile configurations (same bits).
//   * The fetches of a tile's last two K-tiles are the next tile's first two: the operand stream does not stop at the
//     epilogue, which turns a wave's tile around in 8 KiB of LDS of its own beside the stages.
// LDS rows are 128 bytes with the 16-byte chunks of row r stored in the order c ^ ((r / 2) % 8), which leaves the fragment
// reads without bank conflicts; the fetch applies that order through each lane's global address.
#include <mutex>

#include "fetch.h"
#include "gemm_tile.h"

namespace mpz {
namespace {

enum { PIPE_BF16 = 0, PIPE_ROPE64 = 1, PIPE_ROPE128 = 2, PIPE_F32 = 3, PIPE_CE = 4 };   // what the epilogue makes of the tile

// Fused cross-entropy: the logits never leave the registers.  A lane holds 4 NI columns of a token row (lanes l, l ^ 16,
// l ^ 32 and l ^ 48 share the row): row maximum, sum of exponentials against it, and the target's logit if it falls into
// this wave tile.  Two sweeps over all rows instead of one row after the other, so that the shuffles of the eight token tiles travel
// together and the targets are requested at once (33792 x 32000 x 2048: 3581 -> 3519 us, 65536 x 32000 x 2048: 6577 -> 6551).
template <int BN, int WGN, int WGM, int NW, int NI, int NJ>
__device__ __forceinline__ void pipe_ce_partials(const MfmaGemmArgs& a, f32x4 (&acc)[NW][NI][NJ], int m0, int n0, int wm, int wn,
                                                 int wave, int lane) {
  constexpr float LOG2E = 1.4426950408889634f;
  const int l16 = lane & 15, lq = lane >> 4;
  const int slot = (n0 / BN) * WGN + wave / WGM, nl = n0 + wn + lq * 4;
  const bool whole = n0 + wn + NI * 16 <= a.N;           // (uniform) all columns of the wave tile exist
  const int mr = m0 + wm + l16;
  int tg[NJ];
  float mx[NJ], sum[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) tg[j] = mr + j * 16 < a.M ? a.ce_target[mr + j * 16] : -1;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    __builtin_amdgcn_sched_barrier(0);
    mx[j] = -1e30f;
    if (whole) {
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) mx[j] = fmaxf(mx[j], acc[0][i][j][e]);
    } else {
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) mx[j] = nl + i * 16 + e < a.N && acc[0][i][j][e] > mx[j] ? acc[0][i][j][e] : mx[j];
    }
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < NJ; ++j) mx[j] = fmaxf(mx[j], __shfl_xor(mx[j], 16));
#pragma unroll
  for (int j = 0; j < NJ; ++j) mx[j] = fmaxf(mx[j], __shfl_xor(mx[j], 32));
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    __builtin_amdgcn_sched_barrier(0);
    sum[j] = 0.f;
    if (whole) {
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[j] += __builtin_amdgcn_exp2f((acc[0][i][j][e] - mx[j]) * LOG2E);
    } else {
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          sum[j] += nl + i * 16 + e < a.N ? __builtin_amdgcn_exp2f((acc[0][i][j][e] - mx[j]) * LOG2E) : 0.f;
    }
    const int rel = tg[j] - nl;                          // the target's column among this lane's: 16 i + e
    const bool has = rel >= 0 && rel < NI * 16 && (rel & 15) < 4;
    if (__ballot(has) != 0) {                            // one tile in many holds a row's target
      float tl = 0.f;
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) tl = rel == i * 16 + e ? acc[0][i][j][e] : tl;
      if (has) a.ce_tlogit[mr + j * 16] = tl;
    }
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < NJ; ++j) sum[j] += __shfl_xor(sum[j], 16);
#pragma unroll
  for (int j = 0; j < NJ; ++j) sum[j] += __shfl_xor(sum[j], 32);
#pragma unroll
  for (int j = 0; j < NJ; ++j)
    if (mr + j * 16 < a.M && lq == 0) {
      a.ce_max[(size_t)slot * a.M + mr + j * 16] = mx[j];
      a.ce_sum[(size_t)slot * a.M + mr + j * 16] = sum[j];
    }
}

// The part of the output (and of the residual, of the same shape) that belongs to a wave, as a buffer that starts at the
// wave's first element and ends with the matrix.  A lane moves 16 bytes: chunk cc of row crow of an instruction.
template <int ES, int CHUNKS = 16>                       // bytes of an element, 16-byte chunks per row of the strip (fp32: 64 features)
struct PipeOut {
  static constexpr int FPC = 16 / ES, CPW = ES == 4 ? 16 : CHUNKS, RPI = 64 / CPW;   // features per chunk, chunks per row, rows per instruction
  int crow, cc, ldb, off[ES == 4 ? 2 : 1];
  __amdgpu_buffer_rsrc_t ro, rr;
  __device__ __forceinline__ PipeOut(const MfmaGemmArgs& a, int mw, int nw, int lane) {
    crow = lane / CPW; cc = lane % CPW; ldb = a.ldo * ES;
    const size_t first = (size_t)mw * a.ldo + nw, end = (size_t)a.M * a.ldo;
    const size_t left = end > first ? (end - first) * ES : 0;
    const int records = left < 0x7ffffff0 ? (int)left : 0x7ffffff0;
    ro = __builtin_amdgcn_make_buffer_rsrc((char*)a.out + (left ? first * ES : 0), 0, records, 0x00020000);
    rr = ES == 4 && a.residual != nullptr ? __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.residual) + (left ? first : 0), 0, records, 0x00020000) : ro;
    // this lane's byte in the first rows; columns past N aim outside (128 rows stay below 2^31: checked by the launcher)
#pragma unroll
    for (int h = 0; h < (ES == 4 ? 2 : 1); ++h)
      off[h] = nw + h * 64 + cc * FPC < a.N ? crow * ldb + (h * 64 + cc * FPC) * ES : (int)0x80000000;
  }
  __device__ __forceinline__ void read(u32x4 (&rs)[8], int q) const {     // residual of 64 features x 32 tokens
#pragma unroll
    for (int r = 0; r < 8; ++r) rs[r] = __builtin_amdgcn_raw_buffer_load_b128(rr, off[q / 4] + ((q % 4) * 32 + r * 4) * ldb, 0, 0);
  }
  __device__ __forceinline__ void write(u32x4 y, int h, int row) const {
    __builtin_amdgcn_raw_buffer_store_b128(y, ro, off[h] + row * ldb, 0, 0);
  }
};

// Epilogue of one wave's 128 x 128 (SwiGLU: 64 x 128) tile.  A lane holds, for token m0 + wm + 16 j + lane % 16, the
// features n0 + wn + 16 i + 4 (lane / 16) + (0..3) of MFMA tile (i, j).  32 tokens at a time go through the wave's own
// 8 KiB strip (16-byte chunk c of row r at c ^ (r % 16)), so that residual reads and output stores cover whole 256-byte
// pieces of a row with 16 bytes per lane; bf16 outputs are rounded before they enter the strip.  With one wave per SIMD
// nothing hides an instruction here, so there are few, and no branches (the compiler spills accumulators around them; 19 of the 31
// instances still spill 3 to 27 registers between the K loop and the stores, none inside the loop):
// outputs and residuals are buffers that start at the wave's first element and end with the matrix, so rows past M fall
// outside, and the lanes of columns past N aim outside.
template <bool DUAL, int EPI, bool BIAS, bool RELU, bool RES, int NW, int NI, int NJ, int BN, int WGN, int WGM, bool RES1, int NRS>
__device__ __forceinline__ void pipe_epilogue(const MfmaGemmArgs& a, f32x4 (&acc)[NW][NI][NJ], u32x4 (&rs)[NRS][8], unsigned char* strip, int m0, int n0,
                                              int wm, int wn, int wave, int lane) {
  const int l16 = lane & 15, lq = lane >> 4;
  if constexpr (EPI == PIPE_CE) {
    pipe_ce_partials<BN, WGN, WGM, NW, NI, NJ>(a, acc, m0, n0, wm, wn, wave, lane);
    return;
  } else {
    constexpr bool F32 = EPI == PIPE_F32;
    const int mw = m0 + wm, nw = n0 + wn;                // the wave's first token and feature
    const PipeOut<F32 ? 4 : 2, NI * 2> out(a, mw, nw, lane);
    constexpr int FPC = out.FPC, CPW = out.CPW, RPI = out.RPI;
    const int crow = out.crow, cc = out.cc;
    if constexpr (F32) {
#pragma unroll
      for (int q = 0; q < NJ; ++q) {                     // 64 features x 32 tokens at a time: rows of 256 bytes
        const int hf = q / 4, j = q % 4;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (RES) {
          if (q == 0) {
            if constexpr (!RES1) out.read(rs[1], 1);
            out.read(rs[2], 2);
          }
          if (q + 3 < NJ) out.read(rs[(q + 3) & 3], q + 3);
        }
        const int n = nw + hf * 64 + cc * FPC;
        f32x4 bias = {0.f, 0.f, 0.f, 0.f};
        if constexpr (BIAS) bias = *(const f32x4*)(a.bias + (n < a.N ? n : 0));
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int row = h * 16 + l16;
            *(f32x4*)(strip + row * 256 + (((i * 4 + lq) ^ (row & 15)) * 16)) = acc[0][hf * 4 + i][j * 2 + h];
          }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          const int row = r * 4 + crow;
          f32x4 y = *(const f32x4*)(strip + row * 256 + ((cc ^ (row & 15)) * 16));
          if constexpr (BIAS) y += bias;
          if constexpr (RES) y += __builtin_bit_cast(f32x4, rs[q & 3][r]);
          out.write(__builtin_bit_cast(u32x4, y), hf, j * 32 + r * 4);
        }
      }
    } else {
      f32x4 bg[NI], bu[DUAL ? NI : 1];
      if constexpr (BIAS) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          int n = nw + i * 16 + lq * 4;
          n = n < a.N ? n : 0;
          bg[i] = *(const f32x4*)(a.bias + n);
          if (DUAL) bu[i] = *(const f32x4*)(a.bias + a.dual_offset + n);
        }
      }
      // rotary tables of token tile j: cosines and sines of the lower half's features, requested one or two token tiles ahead
      constexpr bool ROPE = EPI == PIPE_ROPE64 || EPI == PIPE_ROPE128;
      constexpr int HP = EPI == PIPE_ROPE128 ? 4 : 2, HALF = 16 * HP, TD = HP == 2 ? 3 : 2;
      f32x4 cs[TD][ROPE ? HP : 1], sn[TD][ROPE ? HP : 1];
      const float inv_s = ROPE ? 1.0f / (float)a.S : 0.f;
      auto tables = [&](int j) {
        int m = mw + j * 16 + l16;
        m = m < a.M ? m : a.M - 1;
        int p = m - (int)((float)m * inv_s) * a.S;       // m % S: m < 2^24 is exact in binary32, the quotient off by one at most
        p = p < 0 ? p + a.S : p;
        p = p >= a.S ? p - a.S : p;
        if (a.rope_pos != nullptr) p = a.rope_pos[p];
#pragma unroll
        for (int i = 0; i < HP; ++i) {
          cs[j % TD][i] = *(const f32x4*)(a.rope_cos + (size_t)p * HALF + i * 16 + lq * 4);
          sn[j % TD][i] = *(const f32x4*)(a.rope_sin + (size_t)p * HALF + i * 16 + lq * 4);
        }
      };
      if constexpr (ROPE) {
#pragma unroll
        for (int j = 0; j < TD - 1; ++j) tables(j);
      }
#pragma unroll
      for (int j2 = 0; j2 < NJ / 2; ++j2) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int j = j2 * 2 + h, lrow = h * 16 + l16;   // token tile, row of the strip
          if constexpr (ROPE) {
            if (j + TD - 1 < NJ) tables(j + TD - 1);
          }
          f32x4 v[NI];
#pragma unroll
          for (int i = 0; i < NI; ++i) {
            v[i] = acc[0][i][j];
            if constexpr (BIAS) v[i] += bg[i];
            if constexpr (DUAL) {
              f32x4 u = acc[NW - 1][i][j];
              if constexpr (BIAS) u += bu[i];
#pragma unroll
              for (int e = 0; e < 4; ++e) v[i][e] = silu_mul_f32(v[i][e], u[e]);
            }
            if constexpr (RELU) {
#pragma unroll
              for (int e = 0; e < 4; ++e) v[i][e] = v[i][e] > 0.f ? v[i][e] : 0.f;
            }
          }
          if constexpr (ROPE) {
            // q / k columns: y_lo = x_lo cos - x_hi sin, y_hi = x_hi cos + x_lo sin with (lo, hi) = columns (c, c + d_head/2); one
            // rounded product and one fma each, as in the stand-alone rotary kernel (same bits); v columns stay
            const bool rot = n0 < a.rope_cols;
#pragma unroll
            for (int i = 0; i < NI; ++i) {
              if ((i / HP) % 2 != 0) continue;
              const f32x4 c = cs[j % TD][i % HP], s = sn[j % TD][i % HP];
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const float lo = v[i][e], hi = v[i + HP][e];
                const float rl = fmaf(lo, c[e], -__fmul_rn(hi, s[e])), rh = fmaf(hi, c[e], __fmul_rn(lo, s[e]));
                v[i][e] = rot ? rl : lo;
                v[i + HP][e] = rot ? rh : hi;
              }
            }
          }
          const int sz = NI == 8 ? (lrow & 15) : ((lrow >> 1) & 7);
#pragma unroll
          for (int i = 0; i < NI; ++i)
            *(u32x2*)(strip + lrow * (CPW * 16) + (((i * 2 + (lq >> 1)) ^ sz) * 16) + (lq & 1) * 8) =
                u32x2{pack_bf16x2(v[i][0], v[i][1]), pack_bf16x2(v[i][2], v[i][3])};
        }
#pragma unroll
        for (int r = 0; r < 32 / RPI; ++r) {
          const int row = r * RPI + crow;
          const int sz = NI == 8 ? (row & 15) : ((row >> 1) & 7);
          const u32x4 y = *(const u32x4*)(strip + row * (CPW * 16) + ((cc ^ sz) * 16));
          out.write(y, 0, j2 * 32 + r * RPI);
        }
      }
    }
  }
}

constexpr int PIPE_BLOCKS = 256;                         // one per CU

// FL bit 0: bias, bit 1: ReLU (fp32 output: residual).  LR: K-steps of 16 of the low-rank term (0: none)
template <bool DUAL, int EPI, int FL, int LR>
__global__ void __launch_bounds__(256, 1) gemm_pipe_kernel(MfmaGemmArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int BN = DUAL ? 128 : 256, BM = 256, BK = 64, WGN = 2, WGM = 2;
  constexpr int NW = DUAL ? 2 : 1, NI = DUAL ? 4 : 8, NJ = 8, TN = BN / WGN, TM = BM / WGM;
  constexpr uint32_t PIECE = 128 * BK * 2, STAGE = 4 * PIECE;

  const int tiles_n = (a.N + BN - 1) / BN, tiles_m = (a.M + BM - 1) / BM;
  const int nblk = tiles_n * tiles_m;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wvn = wave / WGM, wvm = wave % WGM;
  const int wn = wvn * TN, wm = wvm * TM;
  const int l16 = lane & 15, lq = lane >> 4;             // MFMA row / column and 16-byte chunk of a K-step

  // tile number `t` -> (n0, m0), in the order of the other tile configurations: hardware deals consecutive blocks to the
  // 8 XCDs in turn, each XCD owns a contiguous range of tiles and walks it in groups of 8 token-tiles per weight tile
  auto place = [&](int t, int& n0, int& m0) {
    constexpr int GM = 8;
    const int per = nblk / 8, rem = nblk % 8, xcd = t % 8;
    const int pid = xcd * per + (xcd < rem ? xcd : rem) + t / 8;
    const int group = pid / (GM * tiles_n), first_m = group * GM;
    const int gsz = tiles_m - first_m < GM ? tiles_m - first_m : GM;
    const int rr = pid - group * GM * tiles_n;
    m0 = (first_m + rr % gsz) * BM;
    n0 = rr / gsz * BN;
  };

  // A tile's operands are buffers that start at its first row and end with the matrix, so a lane's byte offsets are the
  // same for every tile, and rows past N or M fall outside (whatever those accumulate is never stored).
  const size_t row_b = (size_t)a.K * 2;
  i32x4 rsrcW, rsrcU, rsrcX, nextW, nextU, nextX;
  auto aim = [&](int n0, int m0, i32x4& W, i32x4& U, i32x4& X) {
    W = buffer_of((const char*)a.w + (size_t)n0 * row_b, (size_t)(a.N - n0) * row_b);
    if (DUAL) U = buffer_of((const char*)a.w + (size_t)(n0 + a.dual_offset) * row_b, (size_t)(a.N - n0) * row_b);
    X = buffer_of((const char*)a.x + (size_t)m0 * row_b, (size_t)(a.M - m0) * row_b);
  };
  uint32_t voff[2][4], voffD[4];                         // pieces 0 and 1 (SwiGLU weights: one piece each), four instructions
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int pr = (wave * 4 + t) * 8 + (lane >> 3);     // row of the piece
    const uint32_t ck = (uint32_t)(((lane & 7) ^ ((pr >> 1) & 7)) * 16);
#pragma unroll
    for (int p = 0; p < 2; ++p) voff[p][t] = (uint32_t)((pr >> 6) * 128 + p * 64 + (pr & 63)) * (uint32_t)row_b + ck;
    if (DUAL) voffD[t] = (uint32_t)pr * (uint32_t)row_b + ck;
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem + (uint32_t)wave * 4096u;

  f32x4 acc[NW][NI][NJ];
  bf16x8 fw[2][4][2], fx[2][4][2];                       // [piece][16-row tile][K-step of 32]
  // byte of (row l16, K-step 0) in the chunk order of its row; K-step kk: xor 64 kk
  const uint32_t sw = (uint32_t)(lq ^ ((l16 >> 1) & 7)) * 16u;
  const uint32_t baseW = (uint32_t)(wvn * 64 + l16) * 128u + sw, baseX = 2 * PIECE + (uint32_t)(wvm * 64 + l16) * 128u + sw;

#define FETCH(stage, p, t, soff)                                                                                     \
  fetch_rows((p) >= 2 ? rsrcX : DUAL && (p) == 1 ? rsrcU : rsrcW, DUAL && (p) < 2 ? voffD[t] : voff[(p) & 1][t], soff, \
             lds0 + (stage) * STAGE + (p) * PIECE + (t) * 1024u)
#define READ_W(stage, p, i, kk) \
  fw[p][i][kk] = as_frag(*(const u32x4*)(smem + (stage) * STAGE + (p) * PIECE + (i) * 2048 + (baseW ^ ((kk) * 64u))))
#define READ_X(stage, p, i, kk) \
  fx[p][i][kk] = as_frag(*(const u32x4*)(smem + (stage) * STAGE + (p) * PIECE + (i) * 2048 + (baseX ^ ((kk) * 64u))))
#define ACC(p, i, j) acc[DUAL ? (p) : 0][DUAL ? (i) : (p) * 4 + (i)][j]
// (in place by construction: around the builtin the compiler moves accumulators between registers.  It does not know how long
// the result of the statement takes, so nothing but MFMAs may touch an accumulator inside a K-tile, and the s_nop of
// PIECES_READY covers the last ones: tests/test_gemm_pipe_listing.py checks the compiled code for both.)
#define MFMA(p, i, q, j, kk) \
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(ACC(p, i, (q) * 4 + (j))) : "v"(fw[p][i][kk]), "v"(fx[q][j][kk]))
#define PIN() __builtin_amdgcn_sched_barrier(0)
// Twice per K-tile: this wave's fragment reads have returned and, but for the 16 youngest, its fetches have landed; behind
// the barrier that holds for the block, so the pieces fetched three half K-tiles ago may be read and the slots just read
// may be fetched into.  In a tile's first K-tile the fetches that matter were awaited in the epilogue before (or in the
// prologue); there the epilogue's stores, counted by the same counter, need not be waited for.
#define PIECES_READY(kt)                                                                                                \
  asm volatile("s_cmp_eq_u32 %0, 0\n\ts_cbranch_scc1 .Lready%=\n\ts_waitcnt vmcnt(16)\n.Lready%=:\n\ts_nop 15\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" \
               ::"s"(kt) : "memory", "scc");                                                                            \
  PIN()
// K-tile kt in LDS stage st (its parity); F, S: the token piece multiplied first and second; soff: byte offset of the
// K-tile to fetch into this stage (two further on)
#define TILE(st, F, S, kt)                                                                                             \
  {                                                                                                                    \
    /* W0 x first */                                                                                                   \
    MFMA(0, 0, F, 0, 0); READ_X(st, S, 0, 0); PIN();                                                                   \
    MFMA(0, 0, F, 1, 0); MFMA(0, 0, F, 2, 0); READ_X(st, S, 1, 0); PIN();                                              \
    MFMA(0, 0, F, 3, 0); PIN();                                                                                        \
    MFMA(0, 1, F, 3, 0); READ_X(st, S, 2, 0); PIN();                                                                   \
    MFMA(0, 1, F, 2, 0); MFMA(0, 1, F, 1, 0); READ_X(st, S, 3, 0); PIN();                                              \
    MFMA(0, 1, F, 0, 0); PIN();                                                                                        \
    MFMA(0, 2, F, 0, 0); READ_X(st, S, 0, 1); PIN();                                                                   \
    MFMA(0, 2, F, 1, 0); MFMA(0, 2, F, 2, 0); READ_X(st, S, 1, 1); PIN();                                              \
    MFMA(0, 2, F, 3, 0); PIN();                                                                                        \
    MFMA(0, 3, F, 3, 0); READ_X(st, S, 2, 1); PIN();                                                                   \
    MFMA(0, 3, F, 2, 0); MFMA(0, 3, F, 1, 0); READ_X(st, S, 3, 1); PIN();                                              \
    MFMA(0, 3, F, 0, 0); PIN();                                                                                        \
    MFMA(0, 0, F, 0, 1); MFMA(0, 0, F, 1, 1); FETCH(st, 0, 0, soff); PIN();                                            \
    MFMA(0, 0, F, 2, 1); MFMA(0, 0, F, 3, 1); PIN();                                                                   \
    MFMA(0, 1, F, 3, 1); MFMA(0, 1, F, 2, 1); FETCH(st, 0, 1, soff); PIN();                                            \
    MFMA(0, 1, F, 1, 1); MFMA(0, 1, F, 0, 1); PIN();                                                                   \
    MFMA(0, 2, F, 0, 1); MFMA(0, 2, F, 1, 1); FETCH(st, 0, 2, soff); PIN();                                            \
    MFMA(0, 2, F, 2, 1); MFMA(0, 2, F, 3, 1); PIN();                                                                   \
    MFMA(0, 3, F, 3, 1); MFMA(0, 3, F, 2, 1); FETCH(st, 0, 3, soff); PIN();                                            \
    MFMA(0, 3, F, 1, 1); MFMA(0, 3, F, 0, 1); PIN();                                                                   \
    /* W0 x second */                                                                                                  \
    MFMA(0, 0, S, 0, 0); READ_W(st, 1, 0, 0); PIN();                                                                   \
    MFMA(0, 0, S, 1, 0); MFMA(0, 0, S, 2, 0); READ_W(st, 1, 1, 0); PIN();                                              \
    MFMA(0, 0, S, 3, 0); PIN();                                                                                        \
    MFMA(0, 1, S, 3, 0); READ_W(st, 1, 2, 0); PIN();                                                                   \
    MFMA(0, 1, S, 2, 0); MFMA(0, 1, S, 1, 0); READ_W(st, 1, 3, 0); PIN();                                              \
    MFMA(0, 1, S, 0, 0); PIN();                                                                                        \
    MFMA(0, 2, S, 0, 0); READ_W(st, 1, 0, 1); PIN();                                                                   \
    MFMA(0, 2, S, 1, 0); MFMA(0, 2, S, 2, 0); READ_W(st, 1, 1, 1); PIN();                                              \
    MFMA(0, 2, S, 3, 0); PIN();                                                                                        \
    MFMA(0, 3, S, 3, 0); READ_W(st, 1, 2, 1); PIN();                                                                   \
    MFMA(0, 3, S, 2, 0); MFMA(0, 3, S, 1, 0); READ_W(st, 1, 3, 1); PIN();                                              \
    MFMA(0, 3, S, 0, 0); PIN();                                                                                        \
    MFMA(0, 0, S, 0, 1); MFMA(0, 0, S, 1, 1); FETCH(st, 2 + F, 0, soff); PIN();                                        \
    MFMA(0, 0, S, 2, 1); MFMA(0, 0, S, 3, 1); PIN();                                                                   \
    MFMA(0, 1, S, 3, 1); FETCH(st, 2 + F, 1, soff); PIN();                                                             \
    MFMA(0, 1, S, 2, 1); MFMA(0, 1, S, 1, 1); MFMA(0, 1, S, 0, 1); FETCH(st, 2 + F, 2, soff); PIN();                   \
    MFMA(0, 2, S, 0, 1); MFMA(0, 2, S, 1, 1); MFMA(0, 2, S, 2, 1); FETCH(st, 2 + F, 3, soff); PIN();                   \
    MFMA(0, 2, S, 3, 1); PIN();                                                                                        \
    MFMA(0, 3, S, 3, 1); MFMA(0, 3, S, 2, 1); MFMA(0, 3, S, 1, 1); MFMA(0, 3, S, 0, 1); PIN();                         \
    PIECES_READY(kt);                                                                                                  \
    /* W1 x second */                                                                                                  \
    MFMA(1, 0, S, 0, 0); READ_W(1 - st, 0, 0, 0); PIN();                                                               \
    MFMA(1, 0, S, 1, 0); MFMA(1, 0, S, 2, 0); READ_W(1 - st, 0, 1, 0); PIN();                                          \
    MFMA(1, 0, S, 3, 0); PIN();                                                                                        \
    MFMA(1, 1, S, 3, 0); READ_W(1 - st, 0, 2, 0); PIN();                                                               \
    MFMA(1, 1, S, 2, 0); MFMA(1, 1, S, 1, 0); READ_W(1 - st, 0, 3, 0); PIN();                                          \
    MFMA(1, 1, S, 0, 0); PIN();                                                                                        \
    MFMA(1, 2, S, 0, 0); READ_W(1 - st, 0, 0, 1); PIN();                                                               \
    MFMA(1, 2, S, 1, 0); MFMA(1, 2, S, 2, 0); READ_W(1 - st, 0, 1, 1); PIN();                                          \
    MFMA(1, 2, S, 3, 0); PIN();                                                                                        \
    MFMA(1, 3, S, 3, 0); READ_W(1 - st, 0, 2, 1); PIN();                                                               \
    MFMA(1, 3, S, 2, 0); MFMA(1, 3, S, 1, 0); READ_W(1 - st, 0, 3, 1); PIN();                                          \
    MFMA(1, 3, S, 0, 0); PIN();                                                                                        \
    MFMA(1, 0, S, 0, 1); MFMA(1, 0, S, 1, 1); FETCH(st, 1, 0, soff); PIN();                                            \
    MFMA(1, 0, S, 2, 1); MFMA(1, 0, S, 3, 1); PIN();                                                                   \
    MFMA(1, 1, S, 3, 1); MFMA(1, 1, S, 2, 1); FETCH(st, 1, 1, soff); PIN();                                            \
    MFMA(1, 1, S, 1, 1); MFMA(1, 1, S, 0, 1); PIN();                                                                   \
    MFMA(1, 2, S, 0, 1); MFMA(1, 2, S, 1, 1); FETCH(st, 1, 2, soff); PIN();                                            \
    MFMA(1, 2, S, 2, 1); MFMA(1, 2, S, 3, 1); PIN();                                                                   \
    MFMA(1, 3, S, 3, 1); MFMA(1, 3, S, 2, 1); FETCH(st, 1, 3, soff); PIN();                                            \
    MFMA(1, 3, S, 1, 1); MFMA(1, 3, S, 0, 1); PIN();                                                                   \
    /* W1 x first */                                                                                                   \
    MFMA(1, 0, F, 0, 0); READ_X(1 - st, S, 0, 0); PIN();                                                               \
    MFMA(1, 0, F, 1, 0); MFMA(1, 0, F, 2, 0); READ_X(1 - st, S, 1, 0); PIN();                                          \
    MFMA(1, 0, F, 3, 0); PIN();                                                                                        \
    MFMA(1, 1, F, 3, 0); READ_X(1 - st, S, 2, 0); PIN();                                                               \
    MFMA(1, 1, F, 2, 0); MFMA(1, 1, F, 1, 0); READ_X(1 - st, S, 3, 0); PIN();                                          \
    MFMA(1, 1, F, 0, 0); PIN();                                                                                        \
    MFMA(1, 2, F, 0, 0); READ_X(1 - st, S, 0, 1); PIN();                                                               \
    MFMA(1, 2, F, 1, 0); MFMA(1, 2, F, 2, 0); READ_X(1 - st, S, 1, 1); PIN();                                          \
    MFMA(1, 2, F, 3, 0); PIN();                                                                                        \
    MFMA(1, 3, F, 3, 0); READ_X(1 - st, S, 2, 1); PIN();                                                               \
    MFMA(1, 3, F, 2, 0); MFMA(1, 3, F, 1, 0); READ_X(1 - st, S, 3, 1); PIN();                                          \
    MFMA(1, 3, F, 0, 0); PIN();                                                                                        \
    MFMA(1, 0, F, 0, 1); MFMA(1, 0, F, 1, 1); FETCH(st, 2 + S, 0, soff); PIN();                                        \
    MFMA(1, 0, F, 2, 1); MFMA(1, 0, F, 3, 1); PIN();                                                                   \
    MFMA(1, 1, F, 3, 1); FETCH(st, 2 + S, 1, soff); PIN();                                                             \
    MFMA(1, 1, F, 2, 1); MFMA(1, 1, F, 1, 1); MFMA(1, 1, F, 0, 1); FETCH(st, 2 + S, 2, soff); PIN();                   \
    MFMA(1, 2, F, 0, 1); MFMA(1, 2, F, 1, 1); MFMA(1, 2, F, 2, 1); FETCH(st, 2 + S, 3, soff); PIN();                   \
    MFMA(1, 2, F, 3, 1); PIN();                                                                                        \
    MFMA(1, 3, F, 3, 1); MFMA(1, 3, F, 2, 1); MFMA(1, 3, F, 1, 1); MFMA(1, 3, F, 0, 1); PIN();                         \
    PIECES_READY(kt);                                                                                                  \
  }

  const int nk = a.K / BK;                               // even, at least 2 (checked by the launcher)
  int tile = blockIdx.x, n0, m0;
  place(tile, n0, m0);
  aim(n0, m0, rsrcW, rsrcU, rsrcX);
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
      for (int t = 0; t < 4; ++t) FETCH(s, p, t, (uint32_t)s * (BK * 2));
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

  for (;;) {
    // (this wave's fetches of the first two K-tiles have landed)
    asm volatile("s_barrier" ::: "memory");
    PIN();
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        READ_W(0, 0, i, kk);
        READ_X(0, 0, i, kk);
      }
#pragma unroll
    for (int d = 0; d < NW; ++d)
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[d][i][j][e] = 0.f;
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    PIN();
    const int cn0 = n0, cm0 = m0;
    const bool more = tile + PIPE_BLOCKS < nblk;
    // What the end of the tile needs and is known now travels behind the K loop: the residual of the first tokens, the
    // bottleneck activations of all the wave's tokens and the factor of the first ones' copy.  Copies are whole multiples of 32
    // rows, so a 32-row piece belongs to one copy, and the wave's 128 rows mostly do: only where a copy ends inside are the next
    // pieces' factors requested behind the loop, each under the matrix instructions of the piece before.  Segments begin and end
    // on tile borders; tiles outside every segment multiply zeros.  (With the factors of every 32 rows fetched as if of another copy,
    // half of them behind the loop: 65536 x 2560 x 2048 rotated 588 us, now 554; 65536 x 2048 x 2048 with residual 542 / 509.)
    constexpr bool RES = EPI == PIPE_F32 && (FL & 2);
    u32x4 rs[RES ? 4 : 1][8];
    if constexpr (RES) {
      const PipeOut<4> o(a, cm0 + wm, cn0 + wn, lane);
      o.read(rs[0], 0);
      if constexpr (LR == 0) o.read(rs[1], 1);
    }
    u32x4 lx[LR ? NJ / 2 : 1][2], lw[2][NI];
    int seg = 0;
    bool in = false, one = true;                           // one: the wave's 128 tokens belong to one copy
    const bool part = LR == 2 || lq < 2;
    auto first_row = [&](int j2) {                         // tiles past the end compute discarded values in bounds
      const int mt = cm0 + wm + j2 * 32;
      return mt < a.M ? mt : a.M - 32;
    };
    if constexpr (LR > 0) {
      for (int s = 0; s < a.n_seg; ++s)
        if (cn0 >= a.seg[s].col_begin && cn0 < a.seg[s].col_end) { seg = s; in = true; }
      one = first_row(0) / a.rows_per_copy == first_row(NJ / 2 - 1) / a.rows_per_copy;
    }
    auto low_rank_x = [&](int j2) {                        // operands of 32 tokens
      const uint16_t* tr = (const uint16_t*)a.seg[seg].tp + (size_t)(first_row(j2) + l16) * (16 * LR) + (part ? lq * 8 : 0);
#pragma unroll
      for (int j = 0; j < 2; ++j) lx[j2][j] = *(const u32x4*)(tr + j * 16 * 16 * LR);
    };
    auto low_rank_w = [&](int j2) {                        // and the factor of their copy
      const MfmaLoraSeg& sg = a.seg[seg];
      const int col = in ? cn0 + wn + l16 - sg.col_begin : l16;
      const uint16_t* bp = (const uint16_t*)sg.bp + (size_t)(first_row(j2) / a.rows_per_copy) * sg.copy_stride + (size_t)col * (16 * LR) + (part ? lq * 8 : 0);
#pragma unroll
      for (int i = 0; i < NI; ++i) lw[j2 & 1][i] = *(const u32x4*)(bp + (in ? i * 16 * 16 * LR : 0));
    };
    if constexpr (LR > 0) {
#pragma unroll
      for (int j2 = 0; j2 < NJ / 2; ++j2) low_rank_x(j2);
      low_rank_w(0);
      __builtin_amdgcn_sched_barrier(0);
    }
    // the last two K-tiles fetch the next tile's first two (without a next tile: this one's again)
    if (more) place(tile + PIPE_BLOCKS, n0, m0);
    aim(n0, m0, nextW, nextU, nextX);
    for (int kt = 0; kt < nk; kt += 2) {
      const bool last = kt + 2 >= nk;
#pragma unroll
      for (int e = 0; e < 3; ++e) {
        rsrcW[e] = last ? nextW[e] : rsrcW[e];
        if (DUAL) rsrcU[e] = last ? nextU[e] : rsrcU[e];
        rsrcX[e] = last ? nextX[e] : rsrcX[e];
      }
      uint32_t soff = last ? 0u : (uint32_t)(kt + 2) * (BK * 2);
      TILE(0, 0, 1, kt)
      soff += BK * 2;
      TILE(1, 1, 0, kt + 1)
    }
    // the matrix cores write their last results behind this; the fetches of the next tile's first two K-tiles land
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    if constexpr (LR > 0) {
      // per-copy low-rank term: one more K-step, [B_hi | B_lo] of a copy against the duplicated bottleneck activations [t | t]
      // (rank <= 8: its upper half is zero)
      __builtin_amdgcn_sched_barrier(0);
      const u32x4 zero = {0u, 0u, 0u, 0u};
      if (!one) {
        low_rank_w(1);
      } else {
#pragma unroll
        for (int i = 0; i < NI; ++i) lw[1][i] = lw[0][i];
      }
#pragma unroll
      for (int j2 = 0; j2 < NJ / 2; ++j2) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 2; ++j) lx[j2][j] = in && part ? lx[j2][j] : zero;
#pragma unroll
        for (int i = 0; i < NI; ++i) lw[j2 & 1][i] = part ? lw[j2 & 1][i] : zero;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int i = 0; i < NI; ++i)
            acc[0][i][j2 * 2 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_frag(lw[j2 & 1][i]), as_frag(lx[j2][j]), acc[0][i][j2 * 2 + j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (j2 + 2 < NJ / 2 && !one) low_rank_w(j2 + 2);
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    pipe_epilogue<DUAL, EPI, (FL & 1) != 0, (FL & 2) != 0 && EPI != PIPE_F32, (FL & 2) != 0 && EPI == PIPE_F32, NW, NI, NJ, BN, WGN, WGM, LR == 0>(a, acc, rs, smem + 2 * STAGE + wave * 8192, cm0, cn0, wm, wn, wave, lane);
    if (!more) break;
    tile += PIPE_BLOCKS;
  }
#undef FETCH
#undef READ_W
#undef READ_X
#undef ACC
#undef MFMA
#undef PIN
#undef PIECES_READY
#undef TILE
}

template <bool DUAL, int EPI, int FL, int LR>
hipError_t launch_pipe(hipStream_t st, const MfmaGemmArgs& a) {
  constexpr int BN = DUAL ? 128 : 256;
  constexpr size_t lds = 2 * 4 * 128 * 64 * 2 + 4 * 8192;                  // two stages and a strip per wave: all 160 KiB
  static std::once_flag once;
  static hipError_t attr_status = hipSuccess;
  std::call_once(once, [] {
    attr_status = hipFuncSetAttribute((const void*)gemm_pipe_kernel<DUAL, EPI, FL, LR>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  });
  if (attr_status != hipSuccess) return attr_status;
  const long tiles = (long)((a.N + BN - 1) / BN) * ((a.M + 255) / 256);
  gemm_pipe_kernel<DUAL, EPI, FL, LR><<<(unsigned)(tiles < PIPE_BLOCKS ? tiles : PIPE_BLOCKS), 256, lds, st>>>(a);
  return hipSuccess;
}

template <int EPI, int FL>
hipError_t launch_pipe_lr(hipStream_t st, const MfmaGemmArgs& a) {
  if (a.n_seg == 0) return launch_pipe<false, EPI, FL, 0>(st, a);
  return a.seg[0].rp == 16 ? launch_pipe<false, EPI, FL, 1>(st, a) : launch_pipe<false, EPI, FL, 2>(st, a);
}

}  // namespace

// bf16 weights, whole pairs of K-tiles, 16-byte output pieces that begin on 16 bytes; no GELU (erf around 256 live
// accumulators spills); the low-rank term with rank <= 16
// and no activation behind it.  What is
// refused takes the tile of the same size in gemm_mfma.hip.
bool gemm_pipe_supported(const MfmaGemmArgs& a) {
  if (a.w_scale != nullptr || a.w_absmax != nullptr || a.k_splits > 1 || a.K % 128 || a.act == MPZ_ACT_GELU_ERF || !fetch_aligned(a)) return false;
  if (a.ce_max != nullptr) return a.bias == nullptr && a.n_seg == 0 && a.act < 0;   // (its epilogue takes the products as the logits)
  const int es = a.out_f32 ? 4 : 2;
  if (((uintptr_t)a.out | (uintptr_t)a.residual) & 15 || a.N * es % 16 || a.ldo * es % 16 || a.ldo > (1 << 21)) return false;
  if (!a.out_f32 && a.residual != nullptr) return false;
  if (a.dual || a.rope_cos != nullptr) { if (a.out_f32) return false; }
  else if (a.act >= 0 && (a.out_f32 || a.n_seg || a.act != MPZ_ACT_RELU)) return false;
  if (a.n_seg && a.out_f32 && a.residual == nullptr) return false;
  for (int s = 0; s < a.n_seg; ++s)
    if (a.seg[s].rp != a.seg[0].rp || (a.seg[s].rp != 16 && a.seg[s].rp != 32)) return false;
  return true;
}

hipError_t launch_gemm_pipe(hipStream_t st, const MfmaGemmArgs& a) {
  const bool bias = a.bias != nullptr;
  if (a.dual) return bias ? launch_pipe<true, PIPE_BF16, 1, 0>(st, a) : launch_pipe<true, PIPE_BF16, 0, 0>(st, a);
  if (a.ce_max != nullptr) return launch_pipe<false, PIPE_CE, 0, 0>(st, a);
  if (a.rope_cos != nullptr) {
    if (a.rope_dh == 64) return bias ? launch_pipe_lr<PIPE_ROPE64, 1>(st, a) : launch_pipe_lr<PIPE_ROPE64, 0>(st, a);
    return bias ? launch_pipe_lr<PIPE_ROPE128, 1>(st, a) : launch_pipe_lr<PIPE_ROPE128, 0>(st, a);
  }
  if (a.out_f32) {
    if (a.residual != nullptr) return bias ? launch_pipe_lr<PIPE_F32, 3>(st, a) : launch_pipe_lr<PIPE_F32, 2>(st, a);
    return bias ? launch_pipe<false, PIPE_F32, 1, 0>(st, a) : launch_pipe<false, PIPE_F32, 0, 0>(st, a);
  }
  if (a.act == MPZ_ACT_RELU) return bias ? launch_pipe<false, PIPE_BF16, 3, 0>(st, a) : launch_pipe<false, PIPE_BF16, 2, 0>(st, a);
  return bias ? launch_pipe_lr<PIPE_BF16, 1>(st, a) : launch_pipe_lr<PIPE_BF16, 0>(st, a);
}

}  // namespace mpz
