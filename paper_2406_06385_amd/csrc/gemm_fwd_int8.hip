// Instantiations of the GEMM (gemm_impl.h): forward on the int8 MFMA (W4A8, per-channel scales).
#include "gemm_impl.h"

namespace lrqat {

hipError_t launch_fwd_int8(bool q8, bool zp, const GemmArgs& p, hipStream_t st) {
  if (q8) return zp ? launch_variant<kFwd, kActI8, false, kOptQ8 | kOptZ>(p, st) : launch_variant<kFwd, kActI8, false, kOptQ8>(p, st);
  return zp ? launch_variant<kFwd, kActI8, false, kOptZ>(p, st) : launch_variant<kFwd, kActI8, false, 0>(p, st);
}

}  // namespace lrqat
