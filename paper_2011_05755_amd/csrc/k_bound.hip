// Instantiations and launch of the bound kernel.
#include "bound_impl.h"

namespace mra {

// Work items of a piece: row blocks x halves x reference parts.  A workgroup
// takes all reference tiles (its particle operand is read once) unless the launch
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
  return 2 * ((blocks + 7) & ~7) * parts;
}

// The bounds of kSumRows rows per workgroup: the halves added, raised by the
// margins above, and each row's largest.  16 lanes per row, 16 bytes each:
// bound by its reads and writes (12 bytes per pair).
constexpr int kSumRows = 16;
template <bool ERR>
__device__ __forceinline__ void bound_sum(const CorrArgs& a, int blk) {
  const int row = blk * kSumRows + (threadIdx.x >> 4), c = threadIdx.x & 15;
  if (row >= a.rows) return;  // (16 lanes together)
  float err_s = 0.f, mx = 0.f;
  if constexpr (ERR) {
    err_s = sqrtf(a.rownorm[row] + a.rownorm[a.rows + row]);
    mx = a.maxabs[row / a.S];
  }
  const bool inf = ERR && !(mx * 512.f < INFINITY);
  float* ub = a.ub + (size_t)row * a.ldu;
  const float* hi = a.ub_hi + (size_t)row * a.ldu;
  unsigned long long best = 0ull;
  for (int k0 = 4 * c; k0 < a.ldu; k0 += 64) {
    const float4 x = *reinterpret_cast<const float4*>(ub + k0), y = *reinterpret_cast<const float4*>(hi + k0);
    float v[4] = {x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k = k0 + e;
      // (1e-16: sums of squares below 1e-38 are lost)
      float bound = v[e] * (1.f + 1.f / 4096.f) + 1e-16f;
      if constexpr (ERR) {
        bound += fp16_error(err_s, k < a.K ? a.bnorm[k] * a.b_scale : 0.f, a.R);
        bound = fp16_value(bound, mx, a.b_scale) + 1e-37f;  // (1e-37: what subnormals lose)
        if (inf) bound = INFINITY;
      }
      v[e] = k < a.K ? bound : -INFINITY;
      // (NaN counts as infinite)
      const unsigned long long key = k < a.K ? cand_key(bound == bound ? bound : INFINITY, k) : 0ull;
      best = key > best ? key : best;
    }
    *reinterpret_cast<float4*>(ub + k0) = make_float4(v[0], v[1], v[2], v[3]);
  }
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) {
    const unsigned long long other = __shfl_xor(best, o);
    best = other > best ? other : best;
  }
  if (c == 0) {
    a.rowkey[row] = best;
    if (!(row & (kRowTile - 1))) dense_mask(a)[row / kRowTile] = 0u;
    if constexpr (ERR) a.rownorm[row] = err_s;
  }
}
template <bool ERR>
__global__ __launch_bounds__(16 * kSumRows) void k_bound_sum(CorrArgs a, int* counts) {
  if (blockIdx.x == 0 && threadIdx.x < kFineCounts) counts[threadIdx.x] = 0;
  bound_sum<ERR>(a, blockIdx.x);
}
template <bool ERR>
__global__ __launch_bounds__(16 * kSumRows) void k_bound_sum_batch(CorrBatch b, int* counts) {
  if (blockIdx.x == 0 && threadIdx.x < kFineCounts) counts[threadIdx.x] = 0;
  const int item = blockIdx.x;
  if (item >= b.start[b.n]) return;
  int p = 0;
  while (p + 1 < b.n && b.start[p + 1] <= item) ++p;
  bound_sum<ERR>(b.piece[p], item - b.start[p]);
}

static void dispatch(int prec, int R4, const CorrArgs* a, const CorrBatch* b, int grid, hipStream_t st) {
  if (prec == kFP32) bound_dispatch<kFP16, true>(R4, a, b, grid, st);
  else if (prec == kBF16) bound_dispatch<kBF16, false>(R4, a, b, grid, st);
  else bound_dispatch<kFP16, false>(R4, a, b, grid, st);
}

hipError_t launch_bound(int prec, const CorrArgs& a, int n_items, int* counts, hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
  if (a.R4 < 1 || a.R4 > 16 || !a.ub || !a.ub_hi || !a.rowkey || !counts || a.rows <= 0 || (prec == kFP32 && (!a.bnorm || !a.maxabs))) return hipErrorInvalidValue;
  dispatch(prec, a.R4, &a, nullptr, n_items, st);
  const dim3 grid((a.rows + kSumRows - 1) / kSumRows), block(16 * kSumRows);
  if (prec == kFP32) hipLaunchKernelGGL(k_bound_sum<true>, grid, block, 0, st, a, counts);
  else hipLaunchKernelGGL(k_bound_sum<false>, grid, block, 0, st, a, counts);
  return hipGetLastError();
}

hipError_t launch_bound_batch(int prec, const CorrBatch& b, int* counts, hipStream_t st) {
  if (b.n <= 0 || b.start[b.n] <= 0) return hipSuccess;
  if (!counts) return hipErrorInvalidValue;
  const int bucket = ring_bucket(b.piece[0].R4);
  for (int i = 0; i < b.n; ++i)  // every piece in one ring bucket
    if (b.piece[i].R4 < 1 || ring_bucket(b.piece[i].R4) != bucket || !b.piece[i].ub || !b.piece[i].ub_hi ||
        !b.piece[i].rowkey || b.piece[i].rows <= 0)
      return hipErrorInvalidValue;
  dispatch(prec, b.piece[0].R4, nullptr, &b, b.start[b.n], st);
  CorrBatch sum = b;
  for (int i = 0; i < b.n; ++i) sum.start[i + 1] = sum.start[i] + (b.piece[i].rows + kSumRows - 1) / kSumRows;
  const dim3 grid(sum.start[b.n]), block(16 * kSumRows);
  if (prec == kFP32) hipLaunchKernelGGL(k_bound_sum_batch<true>, grid, block, 0, st, sum, counts);
  else hipLaunchKernelGGL(k_bound_sum_batch<false>, grid, block, 0, st, sum, counts);
  return hipGetLastError();
}

}  // namespace mra
