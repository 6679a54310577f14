// FP16 instantiations of the evaluation kernel, and the tightening of FP32 bounds with it.
#include "fine_impl.h"

namespace mra {

void fine_dispatch_fp16(const FineLaunch& f) { fine_dispatch_16<kFP16, false>(f); }

// tightening of FP32 bounds
void fine_dispatch_tighten(const FineLaunch& f) { fine_dispatch_16<kFP16, true>(f); }

}  // namespace mra
