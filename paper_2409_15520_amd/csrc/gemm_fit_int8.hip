// The tiles of gemm_fit.h with int8 weights.  The codes are fetched into LDS as they are and widened by the wave that reads them, between the
// matrix instructions of the K-step before; waves are dealt along the features, because every wave along the tokens widens the same codes
// again.  (Widened on the way into LDS through registers, the codes cost the fetch its two K-tiles in flight and every store its wait.)
#include "gemm_fit.h"

namespace mpz {

hipError_t launch_gemm_fit_int8(hipStream_t st, const MfmaGemmArgs& a, int shape) {
#define SHAPES(EPI, LR)                                                    \
  switch (shape) {                                                         \
    case 1: return launch_fit<4, 2, 4, 6, 3, EPI, LR, true>(st, a);        \
    case 3: return launch_fit<4, 2, 2, 6, 4, EPI, LR, true>(st, a);        \
    case 4: return launch_fit<4, 2, 4, 4, 4, EPI, LR, true>(st, a);        \
    case 6: return launch_fit<4, 2, 4, 8, 3, EPI, LR, true>(st, a);        \
    default: return launch_fit<4, 2, 2, 4, 5, EPI, LR, true>(st, a);       \
  }
  if (a.dual) { SHAPES(FIT_DUAL, false) }
  if (a.rope_cos != nullptr) {
    if (a.rope_dh == 128) { if (a.n_seg) { SHAPES(FIT_ROPE128, true) } SHAPES(FIT_ROPE128, false) }
    if (a.n_seg) { SHAPES(FIT_ROPE64, true) }
    SHAPES(FIT_ROPE64, false)
  }
  if (a.out_f32) {
    if (a.n_seg) { SHAPES(FIT_F32, true) }
    SHAPES(FIT_F32, false)
  }
  if (a.n_seg) { SHAPES(FIT_BF16, true) }
  SHAPES(FIT_BF16, false)
#undef SHAPES
}

}  // namespace mpz
