// Launch of the evaluation kernel.
#include "fine_impl.h"

namespace mra {

// As many workgroups as the CUs take at once (16 waves each, by registers),
// each taking every grid-th particle.
int fine_grid(int prec, int64_t n, int n_cu) {
  const int64_t most = (int64_t)n_cu * 16 / fine_waves(prec);
  return (int)(n < most ? n : most);
}

static size_t lds_bytes(int prec, int S, int Lp) {
  const size_t state = (size_t)kSlots * 2 * kFinePairs * sizeof(float2);
  const size_t polar = prec == kFP32 ? polar_lds_bytes(Lp) : 0;
  return FineSmem::fixed_bytes(S, fine_waves(prec)) + (state > polar ? state : polar);
}

static void dispatch(int prec, FineMode mode, int R4max, const FineArgs* a, const FineBatch* b, int grid, size_t lds,
                     hipStream_t st) {
  if (mode == kFineTighten) fine_dispatch_tighten(R4max, a, b, grid, lds, st);
  else if (prec == kFP32) fine_dispatch_fp32(mode, R4max, a, b, grid, lds, st);
  else if (prec == kBF16) fine_dispatch_bf16(mode, R4max, a, b, grid, lds, st);
  else fine_dispatch_fp16(mode, R4max, a, b, grid, lds, st);
}

static bool accepts(int prec, FineMode mode, const FineArgs& a) {
  const bool f32 = prec == kFP32 && mode != kFineTighten;
  return a.c.R4 >= 1 && a.c.R4 <= 16 && a.c.S >= 1 && a.c.S <= kMaxShifts && a.c.ub && a.c.rowkey && a.c.A &&
         (!f32 || a.scratch_floats >= (int)(kSlots * a.c.R4 * 64)) &&
         (mode != kFineTighten || (a.c.rownorm && a.c.bnorm && a.c.maxabs)) && (mode != kFineRunnerUp || a.c.excl);
}

hipError_t launch_fine(int prec, FineMode mode, const FineArgs& a, int grid, hipStream_t st) {
  if (a.m.n_part <= 0) return hipSuccess;
  if (grid < 1 || !accepts(prec, mode, a)) return hipErrorInvalidValue;
  dispatch(prec, mode, a.c.R4, &a, nullptr, grid, lds_bytes(mode == kFineTighten ? kFP16 : prec, a.c.S, a.Lp), st);
  return hipGetLastError();
}

hipError_t launch_fine_batch(int prec, FineMode mode, const FineBatch& b, int grid, hipStream_t st) {
  if (b.n <= 0 || b.start[b.n] <= 0) return hipSuccess;
  if (grid < 1) return hipErrorInvalidValue;
  size_t lds = 0;
  int r4 = 0;
  for (int i = 0; i < b.n; ++i) {
    // (the 16-bit instantiations fix the operand's step count: one ring bucket)
    if (!accepts(prec, mode, b.piece[i]) || ring_bucket(b.piece[i].c.R4) != ring_bucket(b.piece[0].c.R4))
      return hipErrorInvalidValue;
    r4 = b.piece[i].c.R4 > r4 ? b.piece[i].c.R4 : r4;
    const size_t need = lds_bytes(mode == kFineTighten ? kFP16 : prec, b.piece[i].c.S, b.piece[i].Lp);
    lds = need > lds ? need : lds;
  }
  dispatch(prec, mode, r4, nullptr, &b, grid, lds, st);
  return hipGetLastError();
}

}  // namespace mra
