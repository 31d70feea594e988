// GEMM tiles between the 128 x 128 ones that are staged through registers and the 256 x 256 one of gemm_pipe.hip, for products of
// one to a few rounds of CUs: 8 waves (two per SIMD), operands fetched straight into LDS, one persistent block per CU.
//
// What bounds it.  The time of such a product is its number of rounds of 256 tiles times the time of a tile: with 128 x 128 and 256 x 256
// tiles alone the last round is often nearly empty.  Inside the K loop the shapes differ little (ns per K-tile of 64 with every CU
// busy, fitted: 192 x 256 1034, 256 x 192 1060, 256 x 128 725, 192 x 128 580, 128 x 128 434: 1240 to 1560 TFLOP/s), because all of them keep two or
// more K-tiles in flight without registers to stage them and meet at one barrier per K-tile; what a smaller tile loses is the operand
// traffic of its CU (90 GB/s at most).  So there are five shapes, and gemm_fit_shape takes the one that fills its rounds.
//   * A K-tile (64) of BN + BM rows of 128 bytes lies in one of ST stages, 16-byte chunk c of row r at c ^ ((r / 2) % 8) (the fetch
//     applies that order through each lane's global address; fragment reads then meet no bank twice).
//   * A K-tile is two K-steps of 32.  Each step's matrix instructions cover the fragment reads of the next.  Behind the first
//     step the block meets: all its fragments of this stage are in registers, so the stage may be fetched into again (K-tile kt + ST), and
//     K-tile kt + 1, whose fetches were issued ST - 1 K-tiles ago, has landed and may be read.
//   * The stream of K-tiles does not stop at a tile's end: its last ST K-tiles fetch the next tile's first ones, and the epilogue's stores
//     are not waited for.  What an epilogue reads comes back in order behind those fetches: the residual, low-rank operands, rotary tables, and in
//     nine of the 89 instances 2 to 26 spilled registers (192 x 256 with fp32 output, int8 256 x 256; none in a K loop).
//   * The outputs leave the accumulators without LDS: two neighbouring 16-feature tiles exchange halves between lanes (one lane swap per
//     dword), so that a lane holds 8 features of a token, and an instruction writes 64 contiguous bytes per token.
// v_mfma_f32_16x16x32_bf16 gives the bits of two chained 32 x 32 x 16 ones and K runs upwards: the sums are those of every other tile.
#pragma once
#include "fetch.h"
#include "gemm_tile.h"

namespace mpz {
namespace {

enum { FIT_BF16 = 0, FIT_ROPE64 = 1, FIT_ROPE128 = 2, FIT_F32 = 3, FIT_DUAL = 4 };   // what the epilogue makes of the tile

// 8 int8 codes -> 8 bf16, exact: |code| <= 128 has at most 8 significant bits
__device__ __forceinline__ uint32_t i8x2_to_bf16(uint32_t v, int lo) {
  return pack_bf16x2((float)(int8_t)(v >> lo), (float)(int8_t)(v >> (lo + 8)));
}

template <int WGN, int WGM, int NI, int NJ, int ST, int EPI, bool LR, bool Q8>
__global__ void __launch_bounds__(64 * WGN * WGM, 2) gemm_fit_kernel(MfmaGemmArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr bool DUAL = EPI == FIT_DUAL, F32 = EPI == FIT_F32;
  constexpr int NWV = WGN * WGM, BN = WGN * NI * 16, BM = WGM * NJ * 16, BK = 64;
  constexpr int CN = DUAL ? BN / 2 : BN, TN = DUAL ? NI * 8 : NI * 16;       // output columns of a tile, of a wave
  constexpr int RPW = Q8 ? 16 : 8, PW = BN / RPW / NWV, PX = BM / 8 / NWV, PER = PW + PX;   // weight rows per fetch; fetches of a wave per K-tile
  static_assert(BN % (RPW * NWV) == 0 && BM % (8 * NWV) == 0, "rows of a K-tile deal out evenly to the waves");
  constexpr uint32_t WROW = Q8 ? 64 : 128, WB = BN * WROW, STAGE = WB + BM * 128, BIAS0 = ST * STAGE;   // behind the stages: biases (and scales) of two tiles

  const int tiles_n = (a.N + CN - 1) / CN, tiles_m = (a.M + BM - 1) / BM, nblk = tiles_n * tiles_m;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wvn = wave / WGM, wvm = wave % WGM, l16 = lane & 15, lq = lane >> 4;   // MFMA row / column and 16-byte chunk of a K-step

  // tile number -> (n0, m0), in the order of the other tile configurations (see gemm_bf16_kernel)
  auto place = [&](int t, int& n0, int& m0) {
    constexpr int GM = 8;
    const int per = nblk / 8, rem = nblk % 8, xcd = t % 8;
    const int pid = xcd * per + (xcd < rem ? xcd : rem) + t / 8;
    const int group = pid / (GM * tiles_n), first_m = group * GM;
    const int gsz = tiles_m - first_m < GM ? tiles_m - first_m : GM;
    const int rr = pid - group * GM * tiles_n;
    m0 = (first_m + rr % gsz) * BM;
    n0 = rr / gsz * CN;
  };

  // A tile's operands are buffers that start at its first row and end with the matrix: a lane's byte offsets are the same for every
  // tile, and rows past the end read as zeros (gate rows past N: rows of up; whatever those accumulate is never stored).
  const uint32_t row_b = (uint32_t)a.K * 2u, wrow_b = Q8 ? (uint32_t)a.K : row_b;
  uint32_t voffW[PW], voffX[PX];
#pragma unroll
  for (int t = 0; t < PW; ++t) {
    const int r = (wave * PW + t) * RPW + lane / (64 / RPW), g = DUAL && r >= CN ? r - CN + a.dual_offset : r;
    voffW[t] = (uint32_t)g * wrow_b + (uint32_t)(Q8 ? ((lane & 3) ^ ((r >> 2) & 3)) * 16 : ((lane & 7) ^ ((r >> 1) & 7)) * 16);
  }
#pragma unroll
  for (int t = 0; t < PX; ++t) {
    const int r = (wave * PX + t) * 8 + (lane >> 3);
    voffX[t] = (uint32_t)r * row_b + (uint32_t)(((lane & 7) ^ ((r >> 1) & 7)) * 16);
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const uint32_t ldsW = lds0 + (uint32_t)(wave * PW) * 1024u, ldsX = lds0 + WB + (uint32_t)(wave * PX) * 1024u;

  // the stream of K-tiles that are fetched: tile, K-tile of it, its buffers (past the last tile: empty ones)
  i32x4 rsrcW, rsrcX;
  int ftile = blockIdx.x, fk = 0;
  const int nk = a.K / BK;
  auto aim = [&]() {
    const bool any = ftile < nblk;
    int n0, m0;
    place(any ? ftile : 0, n0, m0);
    rsrcW = buffer_of((const char*)a.w + (size_t)n0 * wrow_b, any ? (size_t)(a.w_rows - n0) * wrow_b : 0);
    rsrcX = buffer_of((const char*)a.x + (size_t)m0 * row_b, any ? (size_t)(a.M - m0) * row_b : 0);
  };
  auto fetch = [&](int r, uint32_t stage) {              // fetch r of the wave's PER
    const uint32_t soff = (uint32_t)fk * 128u;
    if (r < PW) fetch_rows(rsrcW, voffW[r < PW ? r : 0], Q8 ? soff / 2 : soff, ldsW + stage + (uint32_t)r * 1024u);
    else fetch_rows(rsrcX, voffX[r < PW ? 0 : r - PW], soff, ldsX + stage + (uint32_t)(r - PW) * 1024u);
  };
  auto advance = [&]() {
    if (++fk == nk) {
      fk = 0;
      ftile += (int)gridDim.x;
      aim();
    }
  };
  aim();
#pragma unroll
  for (int s = 0; s < ST; ++s) {
#pragma unroll
    for (int r = 0; r < PER; ++r) fetch(r, s * STAGE);
    advance();
  }

  bf16x8 fw[2][NI], fx[2][NJ];                           // [K-step][16-row tile]
  f32x4 acc[NI][NJ];
  // Feature tile i of a wave: 16 rows of the K-tile from tile_row(wvn, i) on, which are also its columns of the output (gate and up: the
  // second half of the tiles are the up rows of the columns of the first).  Rotated heads are dealt so that a wave has both halves of
  // its columns: with heads of two (four) waves a wave's tiles are every second (fourth) part of either half.
  constexpr bool ROPE = EPI == FIT_ROPE64 || EPI == FIT_ROPE128;
  constexpr int DH = EPI == FIT_ROPE128 ? 128 : 64, WPH = ROPE ? DH / (NI * 16) : 1, NH = NI / 2;
  static_assert(!ROPE || (NI % 2 == 0 && WPH >= 1 && WGN % WPH == 0), "whole heads");
  auto tile_of = [](int i) { return ROPE ? i % NH * 16 + i / NH * (DH / 2) : DUAL && i >= NH ? CN + (i - NH) * 16 : i * 16; };
  const int wcol = ROPE ? wvn / WPH * DH + wvn % WPH * (NI * 8) : wvn * TN;
  const uint32_t sw = (uint32_t)(lq ^ ((l16 >> 1) & 7)) * 16u;
  const uint32_t baseW = (uint32_t)(wcol + l16) * WROW + (Q8 ? (uint32_t)((lq >> 1) ^ (l16 >> 2)) * 16u + (uint32_t)(lq & 1) * 8u : sw);
  const uint32_t baseX = WB + (uint32_t)(wvm * NJ * 16 + l16) * 128u + sw;
  u32x2 raw[Q8 ? NI : 1];                                // int8 codes of the next K-step
  auto read = [&](int r, const unsigned char* sp, int s) {                   // fragment r of NI + NJ, K-step s
    if (r >= NI) fx[s][r < NI ? 0 : r - NI] = as_frag(*(const u32x4*)(sp + (r - NI) * 2048 + (baseX ^ (s * 64u))));
    else if (Q8) raw[Q8 && r < NI ? r : 0] = *(const u32x2*)(sp + tile_of(r) * WROW + (baseW ^ (s * 32u)));
    else fw[s][r < NI ? r : 0] = as_frag(*(const u32x4*)(sp + tile_of(r) * WROW + (baseW ^ (s * 64u))));
  };
  auto widen = [&](int h, int s) {                       // half h of the 2 NI halves of the weight fragments
    const int i = Q8 ? h / 2 : 0;
    u32x4 f = __builtin_bit_cast(u32x4, fw[s][i]);
    const uint32_t v = raw[i][h & 1];
    f[(h & 1) * 2] = i8x2_to_bf16(v, 0);
    f[(h & 1) * 2 + 1] = i8x2_to_bf16(v, 16);
    fw[s][i] = as_frag(f);
  };
  constexpr int NM = NI * NJ, NR = NI + NJ;
#define PIN() __builtin_amdgcn_sched_barrier(0)
#define MFMA(s, m)                                                                                      \
  {                                                                                                     \
    const int i = (m) / NJ, j = (i & 1) ? NJ - 1 - (m) % NJ : (m) % NJ;                                 \
    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[s][i], fx[s][j], acc[i][j], 0, 0, 0);        \
  }

  uint32_t st = 0;                                       // byte of the stage in use
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((ST - 1) * PER) : "memory");
  PIN();
#pragma unroll
  for (int r = 0; r < NR; ++r) read(r, smem, 0);
  if constexpr (Q8) {
#pragma unroll
    for (int h = 0; h < 2 * NI; ++h) widen(h, 0);
  }
  int parity = 0, early = 0;                             // K-tiles of a tile that may leave the tile before's stores on their way
  for (int tile = blockIdx.x; tile < nblk; tile += gridDim.x, parity ^= 1) {
    int n0, m0;
    place(tile, n0, m0);
    // the tile's biases (none: zeros): 1 KiB beside the stages, the other one than the tile before, whose epilogue some waves may
    // still be in (every wave fetches the same bytes, so that their fetches stay in step)
    {
      const int c = lane * 4, col = DUAL && c >= CN ? c - CN + n0 + a.dual_offset : c + n0;
      const uint32_t at = c < BN ? (uint32_t)col * 4u : 0x80000000u;
      fetch_rows<4>(buffer_of(a.bias, a.bias != nullptr ? (size_t)a.w_rows * 4 : 0), at, 0, lds0 + BIAS0 + (uint32_t)parity * 1024u);
      if constexpr (Q8) fetch_rows<4>(buffer_of(a.w_scale, (size_t)a.w_rows * 4), at, 0, lds0 + BIAS0 + 2048u + (uint32_t)parity * 1024u);
    }
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // younger than the fetches of K-tile kt + 1 are those of ST - 2 K-tiles and, in a tile's first ST - 1, the stores (at least S_OUT) of the
    // tile before and the biases
    constexpr int S_OUT = DUAL ? NM / 4 : F32 ? NM : NM / 2, LATE = (ST - 2) * PER, EARLY = LATE + S_OUT + (Q8 ? 2 : 1);
    static_assert(EARLY < 64, "the counter holds 63");
    for (int kt = 0; kt < nk; ++kt) {
      const unsigned char* sp = smem + st;
      const uint32_t nst = st + STAGE == ST * STAGE ? 0 : st + STAGE;
      const unsigned char* np = smem + nst;
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        MFMA(0, m)
#pragma unroll
        for (int r = 0; r < NR; ++r)
          if (r * (NM * 3 / 4) / NR == m) read(r, sp, 1);
        if constexpr (Q8) {
#pragma unroll
          for (int h = 0; h < 2 * NI; ++h)
            if (NM / 2 + h * (NM / 2) / (2 * NI) == m) widen(h, 1);
        }
        PIN();
      }
      asm volatile("s_cmp_lt_i32 %0, %1\n\ts_cbranch_scc1 .Learly%=\n\ts_waitcnt vmcnt(%2)\n\ts_branch .Lmeet%=\n"
                   ".Learly%=:\n\ts_waitcnt vmcnt(%3)\n.Lmeet%=:\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::"s"(kt), "s"(early), "n"(LATE), "n"(EARLY)
                   : "memory", "scc");
      PIN();
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        MFMA(1, m)
#pragma unroll
        for (int r = 0; r < NR; ++r)
          if (r * (NM * 3 / 4) / NR == m) read(r, np, 0);
#pragma unroll
        for (int r = 0; r < PER; ++r)
          if (r * NM / PER == m) fetch(r, st);
        if constexpr (Q8) {
#pragma unroll
          for (int h = 0; h < 2 * NI; ++h)
            if (NM / 2 + h * (NM / 2) / (2 * NI) == m) widen(h, 0);
        }
        PIN();
      }
      advance();
      st = nst;
    }

    early = ST - 1;

    const int mw = m0 + wvm * NJ * 16, nw = n0 + wcol;      // the wave's first token and output column
    if (nk < ST) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (otherwise a wait of the K loop has covered the biases and scales)
    // int8 weights: the accumulators hold x . codes; the per-channel scale turns them into x . W before anything else is added
    // (and rounded there: no fused multiply-add with the bias)
    if constexpr (Q8) {
#pragma clang fp contract(off)
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const f32x4 sc = *(const f32x4*)(smem + BIAS0 + 2048 + parity * 1024 + (wcol + tile_of(i) + lq * 4) * 4);
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] *= sc;
      }
    }
    // Per-copy low-rank term: one more K-step, [B_hi | B_lo] of a copy against the duplicated bottleneck activations [t | t] (rank <= 8:
    // its upper half is zero).  Copies are whole multiples of 32 rows; segments begin and end between wave tiles.
    if constexpr (LR) {
      int seg = -1;
      for (int s = 0; s < a.n_seg; ++s)
        if (nw >= a.seg[s].col_begin && nw < a.seg[s].col_end) seg = s;
      if (seg >= 0) {
        const MfmaLoraSeg& sg = a.seg[seg];
        const bool part = lq * 8 < sg.rp;
        const u32x4 zero = {0u, 0u, 0u, 0u};
        auto row_of = [&](int j) { const int m = mw + j * 16; return m < a.M ? m : a.M - 16; };   // (past the end: discarded, in bounds)
        u32x4 lx[NJ], lw[NI];
        auto factor = [&](int j) {
          const uint16_t* bp = (const uint16_t*)sg.bp + (size_t)(row_of(j) / a.rows_per_copy) * sg.copy_stride + (size_t)(nw + l16 - sg.col_begin) * sg.rp + (part ? lq * 8 : 0);
#pragma unroll
          for (int i = 0; i < NI; ++i) lw[i] = *(const u32x4*)(bp + (size_t)tile_of(i) * sg.rp);
        };
#pragma unroll
        for (int j = 0; j < NJ; ++j) lx[j] = *(const u32x4*)((const uint16_t*)sg.tp + (size_t)(row_of(j) + l16) * sg.rp + (part ? lq * 8 : 0));
        factor(0);
        PIN();
        int copy = row_of(0) / a.rows_per_copy;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int c = row_of(j) / a.rows_per_copy;
          if (c != copy) { factor(j); copy = c; }
#pragma unroll
          for (int i = 0; i < NI; ++i)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_frag(part ? lw[i] : zero), as_frag(part ? lx[j] : zero), acc[i][j], 0, 0, 0);
        }
      }
    }

    // Output: a buffer from the wave's first element to the end of the matrix, so rows past M fall outside; the lanes of columns past N
    // aim outside.  Every store is issued (the waits above count them) and keeps its offset in the vector register.
    constexpr int ES = F32 ? 4 : 2;
    const size_t first = (size_t)mw * a.ldo + nw, end = (size_t)a.M * a.ldo, left = end > first ? (end - first) * ES : 0;
    const int records = left < 0x7ffffff0 ? (int)left : 0x7ffffff0;
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc((char*)a.out + (left ? first * ES : 0), 0, records, 0x00020000);
    const int ldb = a.ldo * ES;
    f32x4 bias[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      bias[i] = *(const f32x4*)(smem + BIAS0 + parity * 1024 + (wcol + tile_of(i) + lq * 4) * 4);
    }
    if constexpr (F32) {
      const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.residual) + (left && a.residual != nullptr ? first : 0), 0,
                                                                          a.residual != nullptr ? records : 0, 0x00020000);
      auto off = [&](int i, int j) { return nw + i * 16 + lq * 4 < a.N ? (j * 16 + l16) * ldb + (i * 16 + lq * 4) * 4 : (int)0x80000000; };
      constexpr int G = NM <= 16 ? NJ : NM <= 24 ? NJ / 2 : 2;
#pragma unroll
      for (int j0 = 0; j0 < NJ; j0 += G) {
        u32x4 rs[G][NI];
#pragma unroll
        for (int j = 0; j < G; ++j)
#pragma unroll
          for (int i = 0; i < NI; ++i)
            if (j0 + j < NJ) rs[j][i] = __builtin_amdgcn_raw_buffer_load_b128(rr, off(i, j0 + j), 0, 0);
        PIN();
#pragma unroll
        for (int j = 0; j < G; ++j)
#pragma unroll
          for (int i = 0; i < NI; ++i)
            if (j0 + j < NJ) {
              const f32x4 y = (acc[i][j0 + j] + bias[i]) + __builtin_bit_cast(f32x4, rs[j][i]);
              __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, y), ro, off(i, j0 + j), 0, 0);
            }
      }
    } else {
      constexpr int NO = DUAL ? NH : NI;
      static_assert(NO % 2 == 0 || NJ % 2 == 0, "tiles in pairs");
      const bool relu = a.act == MPZ_ACT_RELU, rot = ROPE && nw < a.rope_cols;
      const float inv_s = ROPE ? 1.0f / (float)a.S : 0.f;
      auto store = [&](f32x4 v, f32x4 w, int col, int row) {   // this lane's 4 features of two tiles -> 8 of one, at (row, col) of the wave's outputs
        const auto p0 = __builtin_amdgcn_permlane16_swap(pack_bf16x2(v[0], v[1]), pack_bf16x2(w[0], w[1]), false, false);
        const auto p1 = __builtin_amdgcn_permlane16_swap(pack_bf16x2(v[2], v[3]), pack_bf16x2(w[2], w[3]), false, false);
        const int off = nw + col < a.N ? row * ldb + col * 2 : (int)0x80000000;
        __builtin_amdgcn_raw_buffer_store_b128(u32x4{p0[0], p1[0], p0[1], p1[1]}, ro, off, 0, 0);
      };
      f32x4 before[NO % 2 ? NO : 1];                       // outputs of an even token tile whose feature tiles have no pair
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        f32x4 v[NO];
#pragma unroll
        for (int i = 0; i < NO; ++i) {
          v[i] = acc[i][j] + bias[i];
          if constexpr (DUAL) {
            const f32x4 u = acc[NO + i][j] + bias[NO + i];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[i][e] = silu_mul_f32(v[i][e], u[e]);
          } else if constexpr (!ROPE) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[i][e] = relu && !(v[i][e] > 0.f) ? 0.f : v[i][e];
          }
        }
        if constexpr (ROPE) {
          // q / k columns: y_lo = x_lo cos - x_hi sin, y_hi = x_hi cos + x_lo sin with (lo, hi) = columns (c, c + d_head / 2); one rounded
          // product and one fma each, as in the stand-alone rotary kernel (same bits); v columns stay
          int m = mw + j * 16 + l16;
          m = m < a.M ? m : a.M - 1;
          int p = m - (int)((float)m * inv_s) * a.S;     // m % S: m < 2^24 is exact in binary32, the quotient off by one at most
          p = p < 0 ? p + a.S : p;
          p = p >= a.S ? p - a.S : p;
          if (a.rope_pos != nullptr) p = a.rope_pos[p];
          if (rot) {
#pragma unroll
            for (int i = 0; i < NH; ++i) {
              const size_t t = (size_t)p * (DH / 2) + wvn % WPH * (NI * 8) + i * 16 + lq * 4;
              const f32x4 c = *(const f32x4*)(a.rope_cos + t), s = *(const f32x4*)(a.rope_sin + t);
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const float lo = v[i][e], hi = v[(i + NH) % NO][e];
                v[i][e] = fmaf(lo, c[e], -__fmul_rn(hi, s[e]));
                v[(i + NH) % NO][e] = fmaf(hi, c[e], __fmul_rn(lo, s[e]));
              }
            }
          }
        }
        // lane rows 0 / 2 (of 16 lanes) keep their 4 features of the first tile and take the next 4 from row 1 / 3, which take theirs of the second
        if constexpr (NO % 2 == 0) {
#pragma unroll
          for (int i = 0; i < NO; i += 2) store(v[i], v[i + 1], ((lq & 1) ? tile_of(i + 1) : tile_of(i)) + (lq >> 1) * 8, j * 16 + l16);
        } else {
#pragma unroll
          for (int i = 0; i < NO; ++i) {
            if (j % 2) store(before[i], v[i], tile_of(i) + (lq >> 1) * 8, (j - 1 + (lq & 1)) * 16 + l16);
            before[i] = v[i];
          }
        }
      }
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // (fetches past the last tile still write zeros into LDS)
#undef PIN
#undef MFMA
}

template <int WGN, int WGM, int NI, int NJ, int ST, int EPI, bool LR, bool Q8 = false>
hipError_t launch_fit(hipStream_t st, const MfmaGemmArgs& a) {
  constexpr int BN = WGN * NI * 16, BM = WGM * NJ * 16, CN = EPI == FIT_DUAL ? BN / 2 : BN;
  constexpr int lds = ST * (BN * (Q8 ? 64 : 128) + BM * 128) + (Q8 ? 4096 : 2048);
  static_assert(lds <= 160 * 1024, "");
  static const hipError_t attr_status =
      hipFuncSetAttribute((const void*)gemm_fit_kernel<WGN, WGM, NI, NJ, ST, EPI, LR, Q8>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (attr_status != hipSuccess) return attr_status;
  const long tiles = (long)((a.N + CN - 1) / CN) * ((a.M + BM - 1) / BM);
  gemm_fit_kernel<WGN, WGM, NI, NJ, ST, EPI, LR, Q8><<<(unsigned)(tiles < 256 ? tiles : 256), 64 * WGN * WGM, lds, st>>>(a);
  return hipSuccess;
}

}  // namespace
}  // namespace mpz
