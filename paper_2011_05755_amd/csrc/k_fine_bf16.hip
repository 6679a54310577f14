// BF16 instantiations of the evaluation kernel.
#include "fine_impl.h"

namespace mra {

void fine_dispatch_bf16(const FineLaunch& f) { fine_dispatch_16<kBF16, false>(f); }

}  // namespace mra
