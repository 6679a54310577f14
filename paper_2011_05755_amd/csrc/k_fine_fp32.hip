// FP32 instantiations of the evaluation kernel.
#include "fine_impl.h"

namespace mra {

void fine_dispatch_fp32(FineMode mode, int R4max, const FineArgs* a, const FineBatch* b, const FineOver& over, int grid,
                        size_t lds, hipStream_t st) {
  if (R4max <= 8) return fine_go<kFP32, 8, false>(mode, a, b, over, grid, lds, st);
  if (R4max <= 9) return fine_go<kFP32, 9, false>(mode, a, b, over, grid, lds, st);
  if (R4max <= 12) return fine_go<kFP32, 12, false>(mode, a, b, over, grid, lds, st);
  return fine_go<kFP32, 16, false>(mode, a, b, over, grid, lds, st);
}

}  // namespace mra
