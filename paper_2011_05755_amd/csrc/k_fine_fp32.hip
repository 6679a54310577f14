// FP32 instantiations of the evaluation kernel.
#include "fine_impl.h"

namespace mra {

void fine_dispatch_fp32(const FineLaunch& f) {
  if (f.R4max <= 8) return fine_go<kFP32, 8, false>(f);
  if (f.R4max <= 9) return fine_go<kFP32, 9, false>(f);
  if (f.R4max <= 12) return fine_go<kFP32, 12, false>(f);
  return fine_go<kFP32, 16, false>(f);
}

}  // namespace mra
