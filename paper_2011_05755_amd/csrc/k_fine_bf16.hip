// BF16 instantiations of the evaluation kernel.
#include "fine_impl.h"

namespace mra {

void fine_dispatch_bf16(FineMode mode, int R4max, const FineArgs* a, const FineBatch* b, const FineOver& over, int grid,
                        size_t lds, hipStream_t st) {
  fine_dispatch_16<kBF16, false>(mode, R4max, a, b, over, grid, lds, st);
}

}  // namespace mra
