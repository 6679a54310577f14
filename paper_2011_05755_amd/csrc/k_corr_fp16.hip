// FP16 instantiations of the correlation kernel.
#include "corr_impl.h"

namespace mra {

// variant 0: particle operand read once per row tile and resident; 1: re-read
// per reference tile (the runner-up pass: resident).
void corr_dispatch_fp16(int variant, const CorrArgs& a, int mode, hipStream_t st) {
  if (variant == 0 || mode == kRunnerUp) corr_dispatch_16<kFP16, true>(a, mode, st);
  else corr_dispatch_16<kFP16, false>(a, mode, st);
}
void corr_dispatch_fp16(int variant, const CorrBatch& b, hipStream_t st) {
  if (variant == 0) corr_dispatch_16<kFP16, true>(b, kArgmax, st);
  else corr_dispatch_16<kFP16, false>(b, kArgmax, st);
}

}  // namespace mra
