// FP32 instantiations of the correlation kernel.
#include "corr_impl.h"

namespace mra {

// variant 0: 8 waves, particle operand resident; 1: 4 waves, resident,
// R4 <= 12; 2: 8 waves, streamed.  The runner-up pass takes the 8-wave form
// that reads the operand the first pass read (resident or slot-major).
void corr_dispatch_fp32(int variant, const CorrArgs& a, int mode, hipStream_t st) {
  if (mode == kRunnerUp && variant == 1) variant = 2;
  if (variant == 0) return corr_go<Cfg<kFP32, 8, 9, true, false>>(a, mode, st);
  if (variant == 1) return corr_go<Cfg<kFP32, 4, 12, true, false>>(a, mode, st);
  return corr_go<Cfg<kFP32, 8, 16, false, false>>(a, mode, st);
}

}  // namespace mra
