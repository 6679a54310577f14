// FP16 instantiations of the evaluation kernel, and the tightening of FP32 bounds with it.
#include "fine_impl.h"

namespace mra {

void fine_dispatch_fp16(FineMode mode, int R4max, const FineArgs* a, const FineBatch* b, const FineOver& over, int grid,
                        size_t lds, hipStream_t st) {
  fine_dispatch_16<kFP16, false>(mode, R4max, a, b, over, grid, lds, st);
}

// tightening of FP32 bounds
void fine_dispatch_tighten(int R4max, const FineArgs* a, const FineBatch* b, const FineOver& over, int grid,
                           size_t lds, hipStream_t st) {
  fine_dispatch_16<kFP16, true>(kFineTighten, R4max, a, b, over, grid, lds, st);
}

}  // namespace mra
