// FP32 instantiations of the correlation kernel.
#include "corr_impl.h"

namespace mra {

// variant 0: 8 waves, particle operand resident, the ring count compiled in
// (one form for 1 to 9 rings per lane group loads and masks the operands of 9:
// 1500 particles x 25 shifts, 40 references, whole call: 3 rings 1170 against 787
// us, 15 rings 1411 / 1024, 28 rings 1722 / 1542, 36 rings 1955 / 1882); 1: 4 waves,
// resident, R4 <= 12; 2: 8 waves, streamed.  The runner-up pass takes the 8-wave form
// that reads the operand the first pass read (resident or slot-major).
template <class Args>
static void argmax_resident(const Args& a, hipStream_t st) {
  switch (first_piece(a).R4) {
    case 1: return launch_mode<Cfg<kFP32, 8, 1, true, true>, kArgmax>(a, st);
    case 2: return launch_mode<Cfg<kFP32, 8, 2, true, true>, kArgmax>(a, st);
    case 3: return launch_mode<Cfg<kFP32, 8, 3, true, true>, kArgmax>(a, st);
    case 4: return launch_mode<Cfg<kFP32, 8, 4, true, true>, kArgmax>(a, st);
    case 5: return launch_mode<Cfg<kFP32, 8, 5, true, true>, kArgmax>(a, st);
    case 6: return launch_mode<Cfg<kFP32, 8, 6, true, true>, kArgmax>(a, st);
    case 7: return launch_mode<Cfg<kFP32, 8, 7, true, true>, kArgmax>(a, st);
    case 8: return launch_mode<Cfg<kFP32, 8, 8, true, true>, kArgmax>(a, st);
    default: return launch_mode<Cfg<kFP32, 8, 9, true, true>, kArgmax>(a, st);
  }
}

void corr_dispatch_fp32(int variant, const CorrArgs& a, int mode, hipStream_t st) {
  if (mode == kRunnerUp && variant == 1) variant = 2;
  if (variant == 0 && mode == kArgmax) return argmax_resident(a, st);
  if (variant == 0) return launch_mode<Cfg<kFP32, 8, 9, true, false>, kRunnerUp>(a, st);
  if (variant == 1) return corr_go<Cfg<kFP32, 4, 12, true, false>>(a, mode, st);
  return corr_go<Cfg<kFP32, 8, 16, false, false>>(a, mode, st);
}

void corr_dispatch_fp32(int variant, const CorrBatch& b, hipStream_t st) {
  if (variant == 0) return argmax_resident(b, st);
  if (variant == 1) return corr_go<Cfg<kFP32, 4, 12, true, false>>(b, kArgmax, st);
  return corr_go<Cfg<kFP32, 8, 16, false, false>>(b, kArgmax, st);
}

}  // namespace mra
