// Instantiations of the bf16 MFMA GEMM (gemm_impl.h): dW GEMM with the G epilogue, per-channel scales.
#include "gemm_impl.h"

namespace lrqat {

hipError_t launch_dw_pc(const GemmArgs& p, hipStream_t st) { return launch_dw<false>(p, st); }

}  // namespace lrqat
