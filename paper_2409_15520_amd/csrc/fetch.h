// Fetches straight from memory into LDS, counted by the hand-written waits of the kernels that use them.
#pragma once
#include "common.h"

namespace mpz {
namespace {

typedef __attribute__((ext_vector_type(4))) int32_t i32x4;

// One wave instruction fetches 8 rows of 128 bytes (64 lanes x 16 bytes) from a raw buffer into 1 KiB of LDS at byte
// `lds`, in lane order.  It has no destination register; its completion is counted by vmcnt.  (The builtin is not used:
// the compiler would make every later LDS read wait for the fetch.)
// The s_nop: one wait state between the write of m0 and the fetch that reads it; five (NOP = 4) where the scalars may have been
// written by a vector instruction right before.
template <int NOP = 0>
__device__ __forceinline__ void fetch_rows(i32x4 rsrc, uint32_t voff, uint32_t soff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %3\n\ts_nop %4\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(voff), "s"(rsrc), "s"(soff), "s"(lds), "n"(NOP)
               : "memory");
}

// Everything but the youngest min(newer, N) groups of PER fetches has landed, for the whole block
template <int PER, int N>
__device__ __forceinline__ void wait_fetched(int newer) {
  if (N == 0 || newer >= N) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N * PER) : "memory");
  else wait_fetched<PER, N == 0 ? 0 : N - 1>(newer);
}

__device__ __forceinline__ i32x4 buffer_of(const void* p, size_t bytes) {
  const uint64_t b = (uint64_t)p;
  i32x4 r;
  r[0] = (int)(uint32_t)b;
  r[1] = (int)((uint32_t)(b >> 32) & 0xFFFFu);
  r[2] = (int)(uint32_t)bytes;
  r[3] = 0x00020000;
  return r;
}

// Stores through such a buffer (__builtin_amdgcn_raw_buffer_store_b128) keep the whole offset in the vector register and 0 in the
// scalar one.  A store of 16 bytes reads its last registers some cycles after it was issued; the compiler waits for that before it
// overwrites them, but not behind a store whose scalar offset is a register: sums that were cleared right behind such stores went to
// memory as zeros, in one launch of a hundred.

}  // namespace
}  // namespace mpz
