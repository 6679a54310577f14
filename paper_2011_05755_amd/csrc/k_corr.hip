// Host side of the correlation kernel (variant selection and launch) and
// the per-particle merge of row results.  The kernel itself is in
// corr_impl.h, instantiated per precision in k_corr_{fp32,bf16,fp16}.hip.
#include "corr_impl.h"

namespace mra {

// Variant ids (chosen by the caller; see corr_variant_ok):
//   FP32:   0 = 8 waves, A resident, R4 <= 9; 1 = 4 waves, A resident, R4 <= 12;
//           2 = 8 waves, A streamed, R4 <= 16
//   16-bit: 0 = A converted once per row tile and resident, 1 = A re-read
//           and converted per reference tile (8 waves, R4 <= 16)
bool corr_variant_ok(int prec, int variant, int R4) {
  if (R4 < 1 || R4 > 16) return false;
  if (prec == kFP32) return (variant == 0 && R4 <= 9) || (variant == 1 && R4 <= 12) || variant == 2;
  return variant == 0 || variant == 1;
}

int corr_default_variant(int prec, int R4) {
  if (prec == kFP32) return R4 <= 9 ? 0 : 2;
  return 0;
}

static hipError_t launch(int prec, int variant, int mode, const CorrArgs& a, hipStream_t st) {
  if (a.n_row_tiles <= 0) return hipSuccess;
  if (!corr_variant_ok(prec, variant, a.R4) || a.a_layout != a_layout_for(prec, variant) || a.kt_per_wg < 1 ||
      (mode != kTable && !a.rowkey))
    return hipErrorInvalidValue;
  if (prec == kFP32) corr_dispatch_fp32(variant, a, mode, st);
  else if (prec == kBF16) corr_dispatch_bf16(variant, a, mode, st);
  else corr_dispatch_fp16(variant, a, mode, st);
  return hipGetLastError();
}

hipError_t launch_corr(int prec, int variant, bool table, const CorrArgs& a, hipStream_t st) {
  if (table) variant = prec == kFP32 ? 2 : 0;  // any R4 (the host writes the operand for this form)
  return launch(prec, variant, table ? kTable : kArgmax, a, st);
}

hipError_t launch_corr_runner_up(int prec, int variant, const CorrArgs& a, hipStream_t st) {
  if (!a.excl) return hipErrorInvalidValue;
  return launch(prec, variant, kRunnerUp, a, st);
}

// One launch of the arg-max over the pieces of a batch, which take the same instance:
// variant and ring bucket (FP32 variant 0: ring count).
hipError_t launch_corr_batch(int prec, int variant, const CorrBatch& b, hipStream_t st) {
  if (b.n <= 0 || b.start[b.n] <= 0) return hipSuccess;
  const int R4 = b.piece[0].R4;
  for (int i = 0; i < b.n; ++i) {
    const CorrArgs& a = b.piece[i];
    if (!corr_variant_ok(prec, variant, a.R4) || a.a_layout != a_layout_for(prec, variant) || a.kt_per_wg < 1 || !a.rowkey ||
        corr_group(prec, variant, a.R4) != corr_group(prec, variant, R4) || b.start[i + 1] - b.start[i] != corr_items(a))
      return hipErrorInvalidValue;
  }
  if (prec == kFP32) corr_dispatch_fp32(variant, b, st);
  else if (prec == kBF16) corr_dispatch_bf16(variant, b, st);
  else corr_dispatch_fp16(variant, b, st);
  return hipGetLastError();
}

// Per-particle merge of its S row bests (the keys order them as the tie rule
// does) and decoding of the flat index into alignment parameters; one wave
// per particle.
__device__ __forceinline__ void merge_particle(const MergeArgs& m, int n, int ln) {
  const ResultArgs& a = m.r;
  auto value = [&](float v) { return m.maxabs ? fp16_value(v, m.maxabs[n], m.b_scale) : v; };
  unsigned long long best = 0ull;
  for (int s = ln; s < a.S; s += 64) {
    const unsigned long long k = m.rowkey[(size_t)n * a.S + s];
    if (m.row_cc) {
      m.row_cc[(size_t)n * a.S + s] = value(key_value(k));
      m.row_idx[(size_t)n * a.S + s] = key_index(k);
    }
    best = k > best ? k : best;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long other = __shfl_xor(best, o);
    best = other > best ? other : best;
  }
  if (ln == 0) write_result(a, n, value(key_value(best)), key_index(best));
}

__global__ __launch_bounds__(256) void k_merge(MergeArgs m) {
  const int n = (blockIdx.x * 256 + threadIdx.x) >> 6;
  if (n < m.r.n_part) merge_particle(m, n, threadIdx.x & 63);
}

__global__ __launch_bounds__(256) void k_merge_batch(MergeBatch b) {
  const int item = __builtin_amdgcn_readfirstlane((blockIdx.x * 256 + threadIdx.x) >> 6);
  if (item >= b.start[b.n]) return;
  int p = 0;
  while (p + 1 < b.n && b.start[p + 1] <= item) ++p;
  merge_particle(b.piece[p], item - b.start[p], threadIdx.x & 63);
}

hipError_t launch_merge(const MergeArgs& a, hipStream_t st) {
  if (a.r.n_part <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_merge, dim3((a.r.n_part + 3) / 4), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_merge_batch(const MergeBatch& b, hipStream_t st) {
  if (b.n <= 0 || b.start[b.n] <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_merge_batch, dim3((b.start[b.n] + 3) / 4), dim3(256), 0, st, b);
  return hipGetLastError();
}

}  // namespace mra
