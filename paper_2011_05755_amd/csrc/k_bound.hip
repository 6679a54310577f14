// Instantiations and launch of the bound kernel.
#include "bound_impl.h"

namespace mra {

// Work items of a piece: row blocks x reference parts.  A workgroup takes all
// reference tiles (its particle operand is read once) unless the launch
// would leave CUs idle; then the references are split, kBoundTiles at least
// to a part, until every CU has a workgroup.
int bound_items(CorrArgs& a, int n_cu) {
  const int nt = bound_row_tiles(a.R4);
  const int blocks = (a.n_row_tiles + nt - 1) / nt;
  int parts = blocks > 0 ? n_cu / blocks : 1;
  const int most = (a.n_ref_tiles + kBoundTiles - 1) / kBoundTiles;
  parts = parts < 1 ? 1 : (parts > most ? most : parts);
  a.kt_per_wg = (a.n_ref_tiles + parts - 1) / parts;
  parts = (a.n_ref_tiles + a.kt_per_wg - 1) / a.kt_per_wg;
  return blocks * parts;
}

static void dispatch(int prec, int R4, const CorrArgs* a, const CorrBatch* b, int grid, hipStream_t st) {
  if (prec == kFP32) bound_dispatch<kFP16, true>(R4, a, b, grid, st);
  else if (prec == kBF16) bound_dispatch<kBF16, false>(R4, a, b, grid, st);
  else bound_dispatch<kFP16, false>(R4, a, b, grid, st);
}

hipError_t launch_bound(int prec, const CorrArgs& a, int n_items, hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
  if (a.R4 < 1 || a.R4 > 16 || !a.ub || (prec == kFP32 && (!a.bnorm || !a.maxabs))) return hipErrorInvalidValue;
  dispatch(prec, a.R4, &a, nullptr, n_items, st);
  return hipGetLastError();
}

hipError_t launch_bound_batch(int prec, const CorrBatch& b, hipStream_t st) {
  if (b.n <= 0 || b.start[b.n] <= 0) return hipSuccess;
  const int bucket = ring_bucket(b.piece[0].R4);
  for (int i = 0; i < b.n; ++i)  // every piece in one ring bucket
    if (b.piece[i].R4 < 1 || ring_bucket(b.piece[i].R4) != bucket || !b.piece[i].ub) return hipErrorInvalidValue;
  dispatch(prec, b.piece[0].R4, nullptr, &b, b.start[b.n], st);
  return hipGetLastError();
}

}  // namespace mra
