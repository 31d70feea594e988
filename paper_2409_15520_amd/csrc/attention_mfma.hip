// Causal self-attention for the stacked copies (every copy is an ordinary batch row here: Section 3,
// the n copies of the input batch travel through the model side by side).  bf16 MFMA for Q K^T and P V,
// fp32 softmax.  Two passes over the keys: the first finds each query's exact row maximum, the second
// recomputes the scores (bit-identical), forms P = bf16(exp(s - max)) and accumulates P V and sum(P).
// Rounding P against the exact maximum makes the result independent of the key tiling, which a running
// ("online") maximum would not be.
//
// One block = one (sequence, head) and 128 or 256 queries, 32 per wave.  MFMA orientation: rows = keys
// (A operand), columns = queries (B operand): a lane owns ONE query, so max / sum are in-lane plus one
// cross-half shuffle, and the score registers are directly the B operand of the P V product
// D[dv, q] = sum_key Vt[dv, key] P[key, q] (the key order inside an MFMA K-step is permuted identically
// on both operands).
#include "common.h"
#include "fetch.h"

namespace mpz {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;

// The score path is one fma and one hardware exp2 per element: exp(scale (s - max)) = exp2(s c - max c) with c = scale log2(e); masking
// only on tiles that touch the diagonal; bf16 rounding in hardware.
//
// K and V go straight into LDS as they lie in memory, in pieces of KC keys that take turns in a ring of NS slots: pass 1 takes the pieces of K,
// pass 2 pairs of K and V.  V is read transposed
// (ds_read_b64_tr_b16: lane i of 16 gets element i of four rows), so the operand V^T of the second product needs neither a transposition
// through registers nor loads that touch a row with 16 bytes.  16-byte chunk c of row r lies at c ^ f(r), where f
// keeps the reads of either operand out of each other's banks (K: 32 rows at one chunk; V: four rows at four chunks).
// WV waves of 32 queries per block.  ONE: all keys fit half the ring (the launcher knows): each piece is fetched once, all at the start, and
// the scores of pass 1 stay in registers.
// What bounds it: no unit by itself.  128 x 512 tokens, heads of 64: a SIMD issues 65 % of the time (vector instructions 37 %: one fma and one
// exp2 at a quarter of the rate per score; scalar 18 %), the matrix cores are busy 28 %, and a wave stands at waits for half of its
// time (256 tokens: 47 %, 15 %; heads of 128: 37 %, 22 %): the chain scores -> exp2 -> P V of the waves that are there.  Few scalar instructions
// matter therefore: constant waits, no bookkeeping of what is on its way (61 a tile instead of 114: 363 -> 343 us).  Against the form that moved K
// and V through registers, with the same bits (us; sequences x tokens, heads over key-value heads of columns): 128 x 512, 32 / 4 of 64 397 -> 330,
// 64 x 256 74 -> 54, 64 x 96 21.6 -> 15.9, 64 x 128, 12 / 12 of 64 14.0 -> 10.8, 16 x 512, 32 / 32 of 128 127 -> 93, 8 x 480, 20 / 20 of 128 51 -> 34.
// FAR: the rows of a sequence span more than the 31 bits that the offsets into one buffer have (attention_far): each piece gets a buffer of its
// own, whose base is computed in 64 bits.  The pieces, their order and the sums are the same.
template <int DH, int KC, int NS, int WV, int MINB, bool ONE, bool FAR = false>
__global__ void __launch_bounds__(64 * WV, MINB) attention_mfma_kernel(const uint16_t* __restrict__ qkv, int qkv_stride,
                                                             uint16_t* __restrict__ out, int S_grid, int H, int Hkv,
                                                             float scale, const int32_t* __restrict__ cu, int E,
                                                             int rows_per_copy) {
  constexpr int QB = 32 * WV;       // queries per block
  constexpr int NJ = DH / 16;       // MFMA K-steps over the head dimension
  constexpr int NT = DH / 32;       // 32-row output tiles over the head dimension
  constexpr int CPR = DH / 8, RPF = 64 / CPR, PER = KC / RPF / WV;           // 16-byte chunks of a row, rows of a fetch, fetches of a wave per piece
  constexpr uint32_t RB = DH * 2, PIECE = KC * RB;
  static_assert(KC % (RPF * WV) == 0 && KC % 32 == 0, "pieces deal out evenly");
  static_assert(!(ONE && FAR), "a sequence of two pieces is near");
  __shared__ __align__(256) unsigned char smem[NS * PIECE];

  // Hardware deals consecutive workgroups round-robin to the 8 XCDs; give each XCD a contiguous range of the
  // (sequence, head, query block) order instead, so that the blocks that read one sequence's K and V (all query
  // blocks, and under grouped-query attention all heads of the group) share an L2.
  // (1.3B-shaped workload, S = 256: 5.4 -> 4.5 ms per step; with a single query block per head and no key sharing
  // there is nothing to share and the plain order is kept)
  int pid = blockIdx.x;
  const int qblocks = (S_grid + QB - 1) / QB;
  if (qblocks * (H / Hkv) > 1) {
    const int nblk = gridDim.x, per = nblk / 8, rem = nblk % 8;
    const int xcd = pid % 8, idx = pid / 8;
    pid = xcd * per + (xcd < rem ? xcd : rem) + idx;
  }
  const int qb = pid % qblocks;
  const int head = (pid / qblocks) % H;
  const int seq = pid / (qblocks * H);
  // padded batch: every sequence holds S_grid rows.  Packed batch: S_grid is the longest sequence; this one starts at
  // its copy's row cu[e] and may be shorter (query blocks past its end leave at once: block-uniform, before any barrier)
  int S = S_grid;
  size_t row0 = (size_t)seq * S_grid;
  if (cu != nullptr) {
    const int e = seq % E;
    const int start = cu[e];
    S = cu[e + 1] - start;
    row0 = (size_t)(seq / E) * rows_per_copy + start;
    if (qb * QB >= S) return;
  }
  const int kvh = head / (H / Hkv);
  const int d = H * DH, dkv = Hkv * DH;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // a scalar: the tile-visibility tests below are wave-uniform
  const int lrow = lane & 31, lhalf = lane >> 5;

  const int q0 = qb * QB + wave * 32;             // first query of this wave
  const int qi = q0 + lrow;                       // this lane's query
  const int qi_c = qi < S ? qi : S - 1;
  const int last_q_block = qb * QB + QB - 1 < S ? qb * QB + QB - 1 : S - 1;
  const int n = __builtin_amdgcn_readfirstlane(last_q_block / KC + 1);       // pieces of K (and of V) that any query of the block can see
  const int wave_last_q = q0 + 31;

  // this head's K as a buffer of S rows, its V dkv columns to the right in it: rows past the end read as zeros (their keys are masked)
  const uint32_t stride_b = (uint32_t)qkv_stride * 2u, v_b = (uint32_t)dkv * 2u;
  const uint16_t* const kbase = qkv + row0 * qkv_stride + d + kvh * DH;
  const i32x4 rsrc = buffer_of(kbase, (size_t)(S - 1) * stride_b + v_b + RB);
  auto swizzle = [](int r) { return DH == 64 ? (r >> 1 & 1) * 4 + (r >> 2 & 1) * 2 + (r >> 3 & 1) : (r & 3) * 4 + (r >> 2 & 3); };
  uint32_t voff[PER];
#pragma unroll
  for (int t = 0; t < PER; ++t) {
    const int r = (wave * PER + t) * RPF + lane / CPR;
    voff[t] = (uint32_t)r * stride_b + (uint32_t)(lane % CPR ^ swizzle(r)) * 16u;
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem + (uint32_t)wave * (PER * 1024u);
  auto fetch = [&](uint32_t soff, uint32_t slot) {
#pragma unroll
    for (int t = 0; t < PER; ++t) fetch_rows(rsrc, voff[t], soff, lds0 + slot + (uint32_t)t * 1024u);
  };
  // Pieces in the order of their use: ONE K_0 K_1 V_0 V_1 (all of them, at once), else K_0 .. K_n-1 and then K_0 V_0 K_1 V_1 ...; past the end
  // nothing is read (an offset outside the buffer, or a buffer of no bytes), so that the waits need not know where the end is
  const uint32_t piece_b = (uint32_t)KC * stride_b;
  auto fetch_piece = [&](int p, uint32_t slot) {
    const int q = p - n;
    if constexpr (FAR) {
      const int rows = __builtin_amdgcn_readfirstlane(S), c = q < 0 ? p : q >> 1, left = c < n ? rows - c * KC : 0;   // (n pieces begin inside the sequence)
      const i32x4 piece = buffer_of(kbase + (size_t)c * KC * qkv_stride + (q >= 0 && (q & 1) ? dkv : 0),
                                    left > 0 ? (size_t)((left < KC ? left : KC) - 1) * stride_b + RB : 0);
#pragma unroll
      for (int t = 0; t < PER; ++t) fetch_rows<4>(piece, voff[t], 0, lds0 + slot + (uint32_t)t * 1024u);
    } else {
      fetch(q < 0 ? (uint32_t)p * piece_b : q < 2 * n ? (uint32_t)(q >> 1) * piece_b + (q & 1 ? v_b : 0u) : 0x7fffff00u, slot);
    }
  };
  if constexpr (ONE) {
#pragma unroll
    for (int c = 0; c < NS; ++c) fetch((c % (NS / 2) < n ? (uint32_t)(c % (NS / 2)) * piece_b : 0x7ff00000u) + (c >= NS / 2 ? v_b : 0u), c * PIECE);
  } else {
#pragma unroll
    for (int c = 0; c < NS - 1; ++c) fetch_piece(c, c * PIECE);
  }

  // Q fragments (B operand): query qi, head-dim elements j*16 + lhalf*8 .. +7
  bf16x8 fq[NJ];
  {
    const uint16_t* qp = qkv + (row0 + qi_c) * qkv_stride + head * DH + lhalf * 8;
#pragma unroll
    for (int j = 0; j < NJ; ++j) fq[j] = __builtin_bit_cast(bf16x8, *(const u32x4*)(qp + j * 16));
    // (used here, so that the wait for them stands here: inside the loops it would wait for the pieces on their way as well.  They are the
    // youngest requests: what has been fetched so far has landed behind this wait, so that the first counted wait below, and the second of
    // ONE, are barriers only.  ONE with one barrier for both passes: 512 sequences of 128 tokens 154 -> 157 us, 32 over 32 heads 250 -> 256)
#pragma unroll
    for (int j = 0; j < NJ; ++j) asm volatile("" : "+v"(fq[j]));
  }

  // byte of this lane's first chunk in a piece of K (row lrow), and of its quarter of four rows of V (row 4 lhalf + i / 4, i = lane % 16; then
  // eight rows on)
  const uint32_t kaddr = (uint32_t)lrow * RB + (uint32_t)(lhalf ^ swizzle(lrow)) * 16u;
  const int ti = lane & 15, vrow = lhalf * 4 + (ti >> 2), vchunk = (lane >> 4 & 1) * 2 + (ti >> 1 & 1);
  const uint32_t vaddr0 = (uint32_t)vrow * RB + (uint32_t)(vchunk ^ swizzle(vrow)) * 16u + (uint32_t)(ti & 1) * 8u;
  const uint32_t vaddr8 = (uint32_t)(vrow + 8) * RB + (uint32_t)(vchunk ^ swizzle(vrow + 8)) * 16u + (uint32_t)(ti & 1) * 8u;

  // raw scores (q . k, unscaled) of one 32-key tile against this wave's 32 queries; lane: query qi,
  // keys kt0 + (e/4)*8 + lhalf*4 + e%4.  Tiles that reach past the diagonal get -inf on the masked entries.
  auto score_tile = [&](f32x16& sacc, const unsigned char* piece, int t, int kt0) {
#pragma unroll
    for (int e = 0; e < 16; ++e) sacc[e] = 0.f;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const bf16x8 fk = __builtin_bit_cast(bf16x8, *(const u32x4*)(piece + t * 32 * RB + (kaddr ^ (j * 32u))));
      sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fk, fq[j], sacc, 0, 0, 0);
    }
    if (kt0 + 31 > q0) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int key = kt0 + (e >> 2) * 8 + lhalf * 4 + (e & 3);
        sacc[e] = key <= qi ? sacc[e] : -INFINITY;
      }
    }
  };

  // ---- pass 1: exact row maximum ----
  float mx = -1e30f;
  constexpr int KEPT = ONE ? NS / 2 * (KC / 32) : 1;
  f32x16 kept[KEPT];                              // ONE: the scores of all tiles, for pass 2
  auto pass1 = [&](int c, uint32_t slot) {
    const unsigned char* piece = smem + slot;
#pragma unroll
    for (int t = 0; t < KC / 32; ++t) {
      const int kt0 = c * KC + t * 32;
      if (kt0 > wave_last_q) continue;            // tile entirely in this wave's future
      f32x16& sc = kept[ONE ? (c * (KC / 32) + t) % KEPT : 0];
      score_tile(sc, piece, t, kt0);
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = fmaxf(mx, sc[e]);
    }
  };
  uint32_t slot = 0;                              // byte of the slot of the piece in use
  if constexpr (ONE) {
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(NS / 2 * PER) : "memory");
#pragma unroll
    for (int c = 0; c < NS / 2; ++c)
      if (c < n) pass1(c, c * PIECE);
  } else {
    for (int c = 0; c < n; ++c) {
      // piece c has landed for the block and every wave is done with the piece before, whose slot is requested again
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NS - 2) * PER) : "memory");
      fetch_piece(c + NS - 1, slot == 0 ? (NS - 1) * PIECE : slot - PIECE);
      pass1(c, slot);
      slot = slot + PIECE == NS * PIECE ? 0 : slot + PIECE;
    }
  }
  mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
  const float c1 = scale * 1.4426950408889634f;   // scale > 0: the maximum of the raw scores is the maximum
  const float mx2 = mx * c1;

  // ---- pass 2: P = bf16(exp(s - max)), O^T += V^T P, l += P ----
  f32x16 oacc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) oacc[t][e] = 0.f;
  float lsum = 0.f;
  const bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3f803f80u);
  auto pass2 = [&](int c, uint32_t kslot, uint32_t vslot) {
    const unsigned char* piece = smem + kslot;
    const unsigned char* vpiece = smem + vslot;
#pragma unroll
    for (int t = 0; t < KC / 32; ++t) {
      const int kt0 = c * KC + t * 32;
      if (kt0 > wave_last_q) continue;
      f32x16& sc = kept[ONE ? (c * (KC / 32) + t) % KEPT : 0];
      if constexpr (!ONE) score_tile(sc, piece, t, kt0);
      uint32_t pw[8];                             // 16 probabilities as bf16 pairs
#pragma unroll
      for (int e = 0; e < 16; e += 2) {
        const float p0 = __builtin_amdgcn_exp2f(fmaf(sc[e], c1, -mx2));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(sc[e + 1], c1, -mx2));
        const uint32_t w = pack_bf16x2(p0, p1);
        pw[e >> 1] = w;
        lsum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), ones, lsum, false);   // the rounded values
      }
      // two MFMA K-steps of 16 keys: step h uses score registers 8h .. 8h+7, i.e. keys
      // kt0 + 16h + lhalf*4 + (0..3) and kt0 + 16h + 8 + lhalf*4 + (0..3)
#pragma unroll
      for (int hstep = 0; hstep < 2; ++hstep) {
        const u32x4 pfrag = {pw[hstep * 4], pw[hstep * 4 + 1], pw[hstep * 4 + 2], pw[hstep * 4 + 3]};
        const bf16x8 fp = __builtin_bit_cast(bf16x8, pfrag);
#pragma unroll
        for (int vt = 0; vt < NT; ++vt) {
          typedef __attribute__((address_space(3))) s16x4 lds4;
          const unsigned char* p = vpiece + (t * 32 + hstep * 16) * RB;
          const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)(p + (vaddr0 ^ (vt * 64u)))));
          const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)(p + (vaddr8 ^ (vt * 64u)))));
          const u32x4 vfrag = {lo[0], lo[1], hi[0], hi[1]};
          oacc[vt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vfrag), fp, oacc[vt], 0, 0, 0);
        }
      }
    }
  };
  if constexpr (ONE) {
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int c = 0; c < NS / 2; ++c)
      if (c < n) pass2(c, c * PIECE, (NS / 2 + c) * PIECE);
  } else {
    static_assert(NS == 4, "two pairs of pieces");
    for (int c = 0; c < n; ++c) {
      // the pair has landed and every wave is done with the pair before, whose slots take the next one (its K is on its way since pass 1
      // when c = 0)
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      const uint32_t vslot = slot == 3 * PIECE ? 0 : slot + PIECE, next = vslot == 3 * PIECE ? 0 : vslot + PIECE, next_v = next == 3 * PIECE ? 0 : next + PIECE;
      if (c > 0) fetch_piece(n + 2 * c + 2, next);
      fetch_piece(n + 2 * c + 3, next_v);
      pass2(c, slot, vslot);
      slot = next;
    }
  }
  lsum += __shfl_xor(lsum, 32, 64);

  // a lane has four elements of every eight of its query's row, its partner (lane ^ 32) the others: they exchange halves of neighbouring
  // eights, so that each stores 16 bytes
  if (qi < S) {
    const float inv = 1.0f / lsum;
    uint16_t* op = out + (row0 + qi) * (size_t)d + head * DH;
#pragma unroll
    for (int vt = 0; vt < NT; ++vt)
#pragma unroll
      for (int g = 0; g < 4; g += 2) {
        const auto a = __builtin_amdgcn_permlane32_swap(pack_bf16x2(oacc[vt][g * 4] * inv, oacc[vt][g * 4 + 1] * inv),
                                                        pack_bf16x2(oacc[vt][g * 4 + 4] * inv, oacc[vt][g * 4 + 5] * inv), false, false);
        const auto b = __builtin_amdgcn_permlane32_swap(pack_bf16x2(oacc[vt][g * 4 + 2] * inv, oacc[vt][g * 4 + 3] * inv),
                                                        pack_bf16x2(oacc[vt][g * 4 + 6] * inv, oacc[vt][g * 4 + 7] * inv), false, false);
        *(u32x4*)(op + vt * 32 + (g + lhalf) * 8) = u32x4{a[0], b[0], a[1], b[1]};
      }
  }
}

}  // namespace

bool attention_mfma_supported(int dh, int qkv_stride, int d) {
  return (dh == 64 || dh == 128) && qkv_stride % 8 == 0 && d % 8 == 0;
}

// Do the rows of a sequence span more than the offsets into one buffer reach?  Offsets are 32 bits of which the ones from 0x7ff00000 on mean
// "past the end" (attention_mfma_kernel), and the last piece's run up to 64 rows past the sequence.  (A piece's own offsets always fit: 64
// rows of 32 MB would be the rows of a model whose Q|K|V weights alone outgrow the memory.)
bool attention_far(int S, int qkv_stride, int dkv) { return ((size_t)S + 64) * qkv_stride * 2 + (size_t)dkv * 2 >= 0x7ff00000u; }

// Do the scores of the first pass stay in registers (ONE)?  Where all keys fit half the ring; heads of 128 that share no keys only unless
// operands and results together outgrow the last-level cache (64 tokens, 20 heads over 20, ONE / twice: 128 sequences, 168 MB, 26.1 / 28; 256, 335 MB,
// 77.9 / 76.3; 512 153.3 / 152.6).  Everywhere else ONE is ahead whatever the size (16 over 2 heads of 128, 920 sequences 149.5 / 173; heads of 64: 32 over
// 4, 256 x 128 tokens 87.7 / 99.7, 32 over 32 128.1 / 139.8, 16 over 8, 768 x 96 100.3 / 116.1).  The same bits either way.
bool attention_keeps_scores(int n_seq, int S, int H, int Hkv, int dh) {
  if (S > (dh == 64 ? 128 : 64)) return false;
  return dh == 64 || H > Hkv || (size_t)n_seq * S * (2 * H + 2 * Hkv) * dh * 2 < (size_t)320 << 20;
}

// Eight waves fetch a key once for 256 queries: heads of 64 whose last 256 are at least three quarters there (128 x 512, 32 over 4 345 -> 330 us, 64 x
// 256 58.8 -> 53.8; 416 tokens 43.3 -> 44.3, 288 11.4 -> 16.6; heads of 128, 512 tokens 93 -> 107).  Not where the blocks are few and the last of every 256 of
// them (one a CU; a CU holds two) are at most half there: twice the blocks of four waves then take as many rounds, of half the work (four waves / eight,
// us, 200 and 512 tokens, 12 over 12: 96 blocks 7.6 / 9.0 and 12.7 / 15.5, 312 12.0 / 13.0 and 20.6 / 22.9, 600 18.7 / 19.7 and 31.7 / 33.4; but 192 9.7 / 9.4 and
// 16.4 / 15.9, 504 15.6 / 14.4 and 26.3 / 24.9; from 768 on it hangs on the keys that the heads share: 832 blocks of 256 tokens 32 over 4 25.4 / 24.5, 852 12
// over 12 27.1 / 27.8).  The same bits either way.
bool attention_eight_waves(int n_seq, int S, int H, int dh) {
  if (dh != 64 || S <= 128 || (S - 1) % 256 < 191) return false;
  const long blocks = (long)n_seq * H * ((S + 255) / 256);
  return blocks > 640 || (blocks - 1) % 256 >= 128;
}

void launch_attention_mfma(hipStream_t st, const void* qkv, int qkv_stride, void* out, int n_seq, int S, int H, int Hkv,
                           int dh, const int32_t* cu, int E, int rows_per_copy) {
  const float scale = (float)(1.0 / sqrt((double)dh));
  const bool one = attention_keeps_scores(n_seq, S, H, Hkv, dh), eight = attention_eight_waves(n_seq, S, H, dh);
#define LAUNCH(DH, KC, NS, WV, MINB, ...)                                                                                    \
  attention_mfma_kernel<DH, KC, NS, WV, MINB, __VA_ARGS__><<<(unsigned)((size_t)n_seq * H * ((S + 32 * WV - 1) / (32 * WV))), 64 * WV, 0, st>>>( \
      (const uint16_t*)qkv, qkv_stride, (uint16_t*)out, S, H, Hkv, scale, cu, E, rows_per_copy)
  if (attention_far(S, qkv_stride, Hkv * dh)) {
    if (dh == 64) LAUNCH(64, 64, 4, 4, 4, false, true);
    else LAUNCH(128, 32, 4, 4, 2, false, true);
  } else if (dh == 64) {
    if (one) LAUNCH(64, 64, 4, 4, 2, true);
    else if (eight) LAUNCH(64, 64, 4, 8, 4, false);
    else LAUNCH(64, 64, 4, 4, 4, false);
  } else {
    if (one) LAUNCH(128, 32, 4, 4, 2, true);
    else LAUNCH(128, 32, 4, 4, 2, false);
  }
#undef LAUNCH
}

}  // namespace mpz
