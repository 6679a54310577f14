// Launch of the evaluation kernel.
#include <algorithm>

#include "fine_impl.h"

namespace mra {

// As many workgroups as the CUs' registers take at once (16 waves each), each taking
// every grid-th particle (where the LDS takes fewer, the others start as those end).
int fine_grid(int prec, int64_t n, int n_cu) {
  const int64_t most = (int64_t)n_cu * 16 / fine_waves(prec);
  return (int)(n < most ? n : most);
}

static size_t lds_bytes(int prec, int S, int Lp) {
  const size_t state = (size_t)kSlots * 2 * kFinePairs * sizeof(float2);
  const size_t polar = prec == kFP32 ? polar_lds_bytes(Lp) : 0;
  return FineSmem::fixed_bytes(S, fine_waves(prec)) + (state > polar ? state : polar);
}

static void dispatch(int prec, const FineLaunch& f) {
  if (f.mode == kFineTighten) fine_dispatch_tighten(f);
  else if (prec == kFP32) fine_dispatch_fp32(f);
  else if (prec == kBF16) fine_dispatch_bf16(f);
  else fine_dispatch_fp16(f);
}

static bool accepts(int prec, FineMode mode, const FineArgs& a) {
  const bool f32 = prec == kFP32 && mode != kFineTighten;
  return a.c.R4 >= 1 && a.c.R4 <= 16 && a.c.S >= 1 && a.c.S <= kMaxShifts && a.c.ub && a.c.rowkey && a.c.A &&
         (!f32 || a.scratch_floats >= (int)(kSlots * a.c.R4 * 64)) &&
         (mode != kFineTighten || (a.c.rownorm && a.c.bnorm && a.c.maxabs)) && (mode != kFineRunnerUp || a.c.excl);
}

int fine_units(int S, int K) { return (S / kRowTile + 2) * ((K + kOverRefs - 1) / kOverRefs); }

// Steps after which a launch over n particles leaves one of them to the whole
// chip.  One particle in 64 or so (76 px, 100 references, SNR 0.05) has hundreds
// of live pairs, and alone takes 0.4 to 1 ms after the others are done; left
// over, its rows go round once more, spread over all workgroups.  In a launch of
// few rounds of workgroups an early end matters most: BF16 (us, evaluation)
// 300 particles 434 -> 196, 1000: 964 -> 455, 4000: 1581 -> 1030, 8000: 2627 ->
// 1850; FP32 (tightening) 64: 190 -> 179, 256: 1092 -> 358, 4000: 1885 -> 1193.
// In one of more rounds the list holds the fewer, longest ones: after 24 steps
// 20 000 particles BF16 4.70 -> 4.31 ms (after 8: 4.63), 10 000 FP32 3.31 -> 2.69
// (after 8: 4.10).  In a launch that leaves half the workgroups without a
// particle, a particle of few units (5 at 20 references, +-2) is spread out at
// once, after 2 steps: FP32, 64 px, SNR 0.05 (whole call) 50 particles 231 -> 202
// us, 300 of 10 references 367 -> 330; of 20 units (100 references) it is not: 64
// particles 204 against 218.
int fine_over_steps(int64_t n, int units, int n_cu) {
  const int64_t grid = fine_grid(kFP16, INT32_MAX, n_cu);
  return 2 * n <= grid && units <= 16 ? 2 : (n <= 8 * grid ? 8 : 24);
}

static bool sound(int prec, FineMode mode, const FineOver& o, const FineDense& d) {
  const bool spills = prec != kFP32 || mode == kFineTighten;
  const int list = prec == kFP32 ? 1 : 0;
  return d.count && d.tile[list] && d.item[list] && d.grid >= 1 && (mode != kFineTighten || (d.tile[0] && d.item[0])) &&
         (!spills || (o.cap > 0 && o.count && o.item && o.best && o.row && o.pitch >= 1 && o.units >= 1 && o.grid >= 1));
}

hipError_t launch_fine(int prec, FineMode mode, const FineArgs& a, const FineOver& over, const FineDense& dense, int grid,
                       hipStream_t st) {
  if (a.m.n_part <= 0) return hipSuccess;
  if (grid < 1 || !accepts(prec, mode, a) || !sound(prec, mode, over, dense)) return hipErrorInvalidValue;
  dispatch(prec, FineLaunch{mode, a.c.R4, &a, nullptr, over, dense, grid,
                            lds_bytes(mode == kFineTighten ? kFP16 : prec, a.c.S, a.Lp),
                            prec == kFP32 ? polar_lds_bytes(a.Lp) : 0, st});
  return hipGetLastError();
}

hipError_t launch_fine_batch(int prec, FineMode mode, const FineBatch& b, const FineOver& over, const FineDense& dense,
                             int grid, hipStream_t st) {
  if (b.n <= 0 || b.start[b.n] <= 0) return hipSuccess;
  if (grid < 1 || !sound(prec, mode, over, dense)) return hipErrorInvalidValue;
  FineLaunch f{mode, 0, nullptr, &b, over, dense, grid, 0, 0, st};
  for (int i = 0; i < b.n; ++i) {
    const FineArgs& a = b.piece[i];
    // (the 16-bit instantiations fix the operand's step count: one ring bucket)
    if (!accepts(prec, mode, a) || ring_bucket(a.c.R4) != ring_bucket(b.piece[0].c.R4)) return hipErrorInvalidValue;
    f.R4max = std::max(f.R4max, a.c.R4);
    f.lds = std::max(f.lds, lds_bytes(mode == kFineTighten ? kFP16 : prec, a.c.S, a.Lp));
    if (prec == kFP32) f.work = std::max(f.work, polar_lds_bytes(a.Lp));
  }
  dispatch(prec, f);
  return hipGetLastError();
}

}  // namespace mra
