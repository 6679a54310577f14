// Shared constants, launch-argument structs and launcher declarations of
// the MRA kernels (gfx950).  Host code includes this to launch; kernels
// include it for the argument layouts.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mra {

constexpr int kNphi = 256;          // angles per ring (the paper's workloads)
constexpr int kSlots = 128;         // frequency slots: f = 1..127, slot 0 = (f 0, f 128)

constexpr int kRowTile = 8;         // particle rows (shift, particle) per correlation tile
constexpr int kMaxShifts = 289;     // shifts per particle at the largest search range (+-8)
constexpr int kRefTile = 8;         // references per correlation tile
constexpr int kPolarWaves = 8;      // resampling workgroup: 8 waves, 8 shifts x 8 FFT lanes each
constexpr int kMaxBatchPieces = 12; // stack pieces per batched launch (kernel-argument table)
constexpr int kAvgChunk = 32;       // particles per partial class sum
constexpr int kAvgThreads = 256;

enum Prec { kFP32 = 0, kBF16 = 1, kFP16 = 2 };

// Re-ranked 16-bit forms: the rows whose 16-bit best lies within this
// fraction of the particle's best are the re-ranking candidates (and keep
// their exact best under pruning): one unit roundoff of the contraction's
// operand type, 2^-8 for BF16 and 2^-11 for FP16.
__host__ __device__ constexpr float rerank_margin(int prec) {
  return prec == kBF16 ? 1.f / 256.f : (prec == kFP16 ? 1.f / 2048.f : 0.f);
}

// Layouts of the particle operand A (per row tile of 8 rows, 16 floats per
// (ring, slot): p*8 + row%8):
//   kRingPerm   [ring < 4*R4][position][16], slot s at position slot_pos(s): one
//               (ring, row group) item of the resampler writes one contiguous
//               8 KB run, the slots s = w + 8 i of correlation wave w are contiguous, and
//               positions 2m, 2m+1 interleaved element by element in one
//               128-byte block (float 2k + (pos & 1) holds element k), so
//               that one 8-byte load per lane reads both (FP32, 8 waves,
//               operand resident)
//   kSlotMajor  [slot][ring < 4*R4][16]: each slot's rings contiguous (FP32
//               4-wave and streamed contractions, which re-read the operand)
//   kRingPerm16  the 16-bit forms: elements rounded once by the resampler in
//               the contraction's type (BF16, or FP16 scaled by a power of two
//               per particle), [ring < 4*R4][128 positions][16] per row tile
//               with slot s at position slot_pos(s) (wave w's slots w + 8 i at
//               16 w + i) and each run of 8 positions interleaved by element:
//               element k of position 8 G + j at a16_index(8 G + j, k), so that
//               one 16-byte load gives a lane element k of 8 of its wave's slots
enum ALayout { kRingPerm = 1, kSlotMajor = 2, kRingPerm16 = 3 };
__host__ __device__ constexpr int slot_pos(int s) { return (s & 7) * 16 + (s >> 3); }
// 16-bit index of element k of position pos within one (row tile, ring) block
__host__ __device__ constexpr int a16_index(int pos, int k) { return (pos >> 3) * 128 + k * 8 + (pos & 7); }
// The layout a correlation launch reads (and the resampler must write).
__host__ __device__ constexpr int a_layout_for(int prec, int variant) {
  return prec != kFP32 ? kRingPerm16 : (variant == 0 ? kRingPerm : kSlotMajor);
}
// bytes per operand element of a layout
__host__ __device__ constexpr int a_elem_bytes(int layout) { return layout == kRingPerm16 ? 2 : 4; }

// 16-bit reference operand of one (reference tile, slot): NS = ceil(R4 / 8)
// steps of 8 rings per lane group; with NS >= 2 the last step is stored only
// as wide as the rings it holds (2, 4 or 8 elements per lane): the
// contraction reads that many, and the elements it pads with meet zeros of
// the particle operand.
__host__ __device__ constexpr int b16_tail_width(int R4) {
  return R4 <= 8 ? 8 : (R4 - 8 * ((R4 - 1) / 8) <= 2 ? 2 : (R4 - 8 * ((R4 - 1) / 8) <= 4 ? 4 : 8));
}
// 16-bit elements per (reference tile, slot) block
__host__ __device__ constexpr int b16_slot_elems(int R4) { return (((R4 + 7) / 8 - 1) * 8 + b16_tail_width(R4)) * 64; }

// FP32 reference operand: [reference (padded to whole tiles)][slot][ring group
// * 2 + q][b32_pitch]: a lane's R4 elements contiguous, padded to 16 bytes
__host__ __device__ constexpr int b32_pitch(int R4) { return (R4 + 3) & ~3; }

// Power-of-two FP16 scale of a particle's operand: |a +- b| <= 2 * 256 *
// max|pixel| is mapped below 2^14.
__device__ __forceinline__ int fp16_operand_exponent(float maxabs) {
  const float m = fmaxf(maxabs * 512.f, 1e-30f);
  return 14 - (int)ceilf(log2f(m));
}
__device__ __forceinline__ float fp16_operand_scale(float maxabs) { return ldexpf(1.f, fp16_operand_exponent(maxabs)); }

// A value in the scaled units of a particle with max |pixel| mx against a
// refset of scale b_scale, in its own: by the sum of the exponents (either
// power, or their product, may take a value out of the float range that is within it
// at the end).  NaN where either does not scale into FP16: then v means nothing.
__device__ __forceinline__ float fp16_value(float v, float mx, float b_scale) {
  if (!(mx * 512.f < INFINITY && b_scale < INFINITY)) return NAN;
  return ldexpf(v, -(fp16_operand_exponent(mx) + ilogbf(b_scale)));
}

// Entry of the particle sampling stencil for ring r and angle j (FP64
// positions, used by the FP32 re-score and the single-reference kernel): the floor (dx, dy) of
// r*(cos, sin)(theta_j), stored as bx = 4 dx (the byte offset of the column
// in a float row) and dy, and the bilinear fractions.
struct __attribute__((aligned(16))) Stencil {
  int bx, dy;
  float fx, fy;
};

// Resample + ring-FFT kernel.  out layout depends on the mode:
//  mode 0: correlation operand A in layout a_layout (ALayout),
//          inner index p*8 + row%8 (p = 0: a-b, p = 1: a+b); rings >= R are
//          never written (the correlation kernel masks them)
//  mode 1: polar samples [n][S][R][256]
//  mode 2: ring spectra  [n][S][R][129][2]
struct PolarArgs {
  const float* parts;  // first particle of the chunk, [n][L][L]
  int n_part;
  int L, R, R4, T, S1, S;
  // LDS image: rows x rows pixels of row pitch Lp; image pixel (y, x) at
  // (y + pad, x + pad) (pad < 0: pixels outside are not staged), zeros outside
  // the image; cx: the centre pixel
  int Lp, rows, pad, cx;
  int r_min;           // radius of ring 0
  int a_layout;        // mode 0: ALayout of the operand
  int split;           // mode 0: workgroups per particle
  int prec;            // kRingPerm16: kBF16 or kFP16
  float* maxabs;       // kFP16: out, max |pixel| of each particle of the chunk (operand scale)
  const double2* cs64; // (cos, sin)(2 pi j / 256)
  unsigned long long* rowkey;  // zeroed for the particle's rows, or null
  float* out;          // (mode 0, kRingPerm16: 16-bit elements)
};

// Contraction, bounds and evaluation of a chunk's rows against a refset.
struct CorrArgs {
  const float* A;        // [row tiles][...] in layout a_layout (ALayout; 16-bit elements for kRingPerm16)
  int a_layout;
  int n_row_tiles;
  int rows;              // valid rows in the chunk (n * S)
  const float* B32;      // [n_ref_tiles * 8][128][8][b32_pitch(R4)]
  const uint16_t* B16;   // [ref tiles][128][b16_slot_elems(R4)]: NS - 1 steps [64][8], then [64][BT],
                         // the 64 ordered ring group, reference, q
  int R, R4, n_ref_tiles, K, S, M;
  const float* maxabs;   // FP16 operand: max |pixel| of each particle of the chunk (A scale), else null
  float b_scale;         // FP16 operand: power-of-two scale folded into B16
  const float* bnorm;    // FP32 alignment: norm of each reference's operand (bound error)
  const float2* cs32;
  float* row_cc;         // evaluation: [rows] best CC of the row and its flat index, or null
  int* row_idx;
  float* table;          // debug: [n][K][M][S][256], else null
  const int* excl;       // per particle of the chunk: flat index left out of the arg-max, or null
  float* ub;             // [rows][ldu] upper bound of each pair's CC (-inf past K)
  float* ub_hi;          // [rows][ldu] scratch: the bounds' part of slots 64 .. 127
  int ldu;               // 8 * n_ref_tiles
  unsigned long long* rowkey;  // [rows] each row's largest bound and its reference, or (every pair evaluated) its
                               // best CC and flat index, in cand_key order; every pair evaluated: zeroed by
                               // the resampler.  With bounds, dense_rows and dense_mask follow
  float* rownorm;        // FP32 alignment: [2][rows], first the norm of the row's operand (FP16, scaled; bound
                         // error); scratch of the bounds: the halves' squares
  int kt_per_wg;         // reference tiles per workgroup (bounds, and the correlation of every pair)
};

// Batched form: work item i of the launch is item i - start[p] of piece p
// with start[p] <= i < start[p + 1].
struct CorrBatch {
  int n;
  int start[kMaxBatchPieces + 1];
  CorrArgs piece[kMaxBatchPieces];
};

constexpr int kFineOverCap = 1024;  // (8 (1 + S) bytes each)
// Particles with many pairs to evaluate, left to the whole chip: how many, and
// for each its item number in the launch, its best candidate so far and its
// rows'.
struct FineOver {
  int* count;                // zeroed by the bounds' sum
  int* item;                 // [cap]
  unsigned long long* best;  // [cap]
  unsigned long long* row;   // [cap][pitch]
  int cap, pitch;            // cap 0: none is left over
  int steps;                 // steps after which a particle is left over
  int units;                 // units of work per particle
  int grid;                  // workgroups of that launch
};

// Particles of which so many pairs are live that every pair is evaluated: their
// row tiles and, for the results, their item numbers in the launch.  List 0: with
// the 16-bit operand (FP32: the tightening), list 1: with the FP32 one.  The rows of
// such particles have a bit in the mask of their row tile (dense_mask, zeroed by the
// bounds' sum; list 1 eight bits up) and their best candidate in dense_rows.
struct FineDense {
  int* count;                // [4] row tiles and particles of either list; zeroed by the bounds' sum
  int2* tile[2];             // (piece, row tile)
  int* item[2];
  int grid;                  // workgroups of a launch that evaluates them
};
constexpr int kFineCounts = 6;  // those of FineOver (arg-max, runner-up) and FineDense, end to end
__host__ __device__ constexpr size_t rowkey_bytes(size_t rows, bool bounds) {
  return bounds ? 16 * rows + 4 * ((rows + kRowTile - 1) / kRowTile + 1) : 8 * (rows + 1);
}
__device__ __forceinline__ unsigned long long* dense_rows(const CorrArgs& c) { return c.rowkey + c.rows; }
__device__ __forceinline__ uint32_t* dense_mask(const CorrArgs& c) {
  return reinterpret_cast<uint32_t*>(c.rowkey + 2 * (size_t)c.rows);
}

// Where a chunk's particles' results go.
struct ResultArgs {
  int n_part, S, S1, T, M;
  int runner_up;         // 1: the values are bests without the winner; write only cc2
  int64_t out_off;
  int32_t *ref, *shift_x, *shift_y, *psi, *mirror, *flat;
  float *cc, *cc2;
  int32_t* win;          // chunk-local copy of each winner's flat index, or null
};

// Merge of the rows' bests, every pair having been evaluated.
struct MergeArgs {
  ResultArgs r;
  const unsigned long long* rowkey;  // [n_part * S]
  const float* maxabs;   // FP16: with b_scale, the scale of the rows' values, else null
  float b_scale;
  float* row_cc;         // out, for the re-ranking, or null
  int* row_idx;
};

struct MergeBatch {
  int n;
  int start[kMaxBatchPieces + 1];
  MergeArgs piece[kMaxBatchPieces];
};
static_assert(sizeof(CorrBatch) <= 4096 && sizeof(MergeBatch) <= 4096, "kernel arguments");

// Evaluation of the pairs that can win, one workgroup per particle at a time.
struct FineArgs {
  CorrArgs c;            // A: the rows' operand (16-bit forms) or the scratch tiles (FP32)
  ResultArgs m;          // the particle's outputs
  float margin;          // rows within this fraction of the particle's best keep their exact best
  // FP32: the operand of the rows evaluated is made here, in one scratch tile
  // per workgroup (blockIdx.x * scratch_floats)
  int scratch_floats;
  const float* parts;    // first particle of the chunk
  int L, Lp, pad, cx, r_min;
  const double2* cs64;
};
struct FineBatch {
  int n;
  int start[kMaxBatchPieces + 1];
  FineArgs piece[kMaxBatchPieces];
};
static_assert(sizeof(FineBatch) <= 4096, "kernel arguments");

struct RescoreArgs {
  const float* parts;
  int n_part;
  int64_t out_off;
  int L, R, r_min, Lp, pad, cx, K, T;
  const Stencil* stencil;
  const float* qhat;     // [K][R][256]
  const int32_t *ref, *shift_x, *shift_y, *psi, *mirror;
  float* cc;
  // Re-ranking (rows >= 2): the winners of the particle's `rows` best rows of
  // the 16-bit pass and their neighbours within +-1 angle are re-scored in
  // FP32 and the best of them becomes the result.  rows <= 1: the winner only.
  int rows, S1, S, M;
  float margin;          // rows within this fraction of the particle's 16-bit best are candidates
  const float* row_cc;   // [n_part][S] of the 16-bit pass
  const int* row_idx;
  int32_t *ref_w, *shift_x_w, *shift_y_w, *psi_w, *mirror_w, *flat_w;  // re-ranked outputs
  int32_t* win;          // chunk-local winner copy for the runner-up pass, or null
  float* psi_frac;       // refinement launch: sub-step angle of the final winner
};

// Batched forms of the per-particle kernels: item i of the launch is
// particle i - start[p] of piece p with start[p] <= i < start[p + 1].
struct PolarBatch {
  int n;
  int start[kMaxBatchPieces + 1];
  PolarArgs piece[kMaxBatchPieces];
};
struct RescoreBatch {
  int n;
  int start[kMaxBatchPieces + 1];
  RescoreArgs piece[kMaxBatchPieces];
};

// Alignment against one reference (K = 1): resampling, ring FFTs,
// correlation, inverse FFT and arg-max fused per particle.
struct RfaArgs {
  const float* parts;    // first particle of the call, [n][L][L]
  int n_part;
  int64_t out_off;
  int L, R, T, S1, S, M, Lp, pad, cx, r_min;
  const Stencil* stencil;  // [R][256]
  const double2* cs64;
  const float2* G;       // [R][128]: (c - d, c + d) of the reference's weighted spectrum per slot
  int32_t *ref, *shift_x, *shift_y, *psi, *mirror, *flat;
  float *cc, *cc2;
};

// ---- launchers (one .hip file each) ----
hipError_t launch_polar(int mode, const PolarArgs& a, hipStream_t st);
size_t polar_lds_bytes(int Lp);  // a resampler of 8 waves beside an Lp x Lp image
void polar_window(PolarArgs& a, int lo, int hi);
int polar_waves(const PolarArgs& a);
hipError_t launch_corr(int prec, int variant, bool table, const CorrArgs& a, hipStream_t st);
hipError_t launch_corr_batch(int prec, int variant, const CorrBatch& b, hipStream_t st);
hipError_t launch_corr_runner_up(int prec, int variant, const CorrArgs& a, hipStream_t st);
// 16-bit ring buckets (R4 <= 8, 9..10, 11..12, 13..16): the pieces of a batched launch share one
constexpr int ring_bucket(int R4) { return R4 <= 8 ? 0 : (R4 <= 10 ? 1 : (R4 <= 12 ? 2 : 3)); }
// work items of a bound launch over a's rows; sets a.kt_per_wg.  The launch also
// zeroes counts[0 .. kFineCounts - 1].
int bound_items(CorrArgs& a, int n_cu);
hipError_t launch_bound(int prec, const CorrArgs& a, int n_items, int* counts, hipStream_t st);
hipError_t launch_bound_batch(int prec, const CorrBatch& b, int* counts, hipStream_t st);
// workgroups of an evaluation launch over n particles (FP32: also its scratch tiles)
int fine_grid(int prec, int64_t n, int n_cu);
enum FineMode { kFineArgmax = 0, kFineRunnerUp = 2, kFineTighten = 3 };
hipError_t launch_fine(int prec, FineMode mode, const FineArgs& a, const FineOver& over, const FineDense& dense, int grid,
                       hipStream_t st);
hipError_t launch_fine_batch(int prec, FineMode mode, const FineBatch& b, const FineOver& over, const FineDense& dense,
                             int grid, hipStream_t st);
int fine_units(int S, int K);                         // FineOver::units of a piece
int fine_over_steps(int64_t n, int units, int n_cu);  // FineOver::steps of a launch over n particles
// launches of few particles: workgroups of `waves` waves per particle (of
// n_items 8-row ring items) that fill n_cu CUs with 16 waves each
inline int polar_split(int n_part, int n_items, int n_cu, int waves) {
  const int want = n_part > 0 ? 2 * kPolarWaves * n_cu / waves / n_part : 1, most = (n_items + waves - 1) / waves;
  return want < 1 ? 1 : (want > most ? most : want);
}
// reference tiles per workgroup of a launch of `tiles` row tiles, one workgroup per CU
// at a time: those that end the launch first, rounds of workgroups times their length
// (a workgroup's prologue, which reads the operand of its rows, takes about a third of a
// reference tile's time)
inline int corr_tiles_per_wg(int tiles, int n_ref_tiles, int n_cu) {
  int best = n_ref_tiles;
  double least = 0;
  for (int parts = 1; parts <= n_ref_tiles && (parts == 1 || (int64_t)tiles * parts <= 16 * (int64_t)n_cu); ++parts) {
    const int per = (n_ref_tiles + parts - 1) / parts;
    const int64_t wgs = (int64_t)tiles * ((n_ref_tiles + per - 1) / per);
    const double time = (double)((wgs + n_cu - 1) / n_cu) * (per + 0.35);
    if (parts == 1 || time < least) {
      least = time;
      best = per;
    }
  }
  return best;
}
inline int corr_items(const CorrArgs& a) {
  return a.n_row_tiles * ((a.n_ref_tiles + a.kt_per_wg - 1) / a.kt_per_wg);
}
bool corr_variant_ok(int prec, int variant, int R4);
// stacks with the same value take the same instance of the correlation kernel (of one
// precision and variant)
constexpr int corr_group(int prec, int variant, int R4) { return prec == kFP32 && variant == 0 ? R4 : 16 + ring_bucket(R4); }
int corr_default_variant(int prec, int R4);
hipError_t launch_merge(const MergeArgs& a, hipStream_t st);
hipError_t launch_merge_batch(const MergeBatch& b, hipStream_t st);
hipError_t launch_rescore(const RescoreArgs& a, hipStream_t st);
hipError_t launch_polar_batch(const PolarBatch& b, hipStream_t st);
hipError_t launch_rescore_batch(const RescoreBatch& b, hipStream_t st);
hipError_t launch_refine(const RescoreArgs& a, hipStream_t st);  // psi_frac from the final parameters
hipError_t launch_rfa(const RfaArgs& a, hipStream_t st);
// zero `bytes` (a multiple of 16) at p (16-byte aligned) with a kernel
hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t st);
// count[0] += #{i : cls[i] != prev[i]}; then prev = cls
hipError_t launch_count_changed(const int32_t* cls, int32_t* prev, int n, int* count, hipStream_t st);

// reference preparation
struct RefInfo {     // read back by the host
  float bmax;        // largest |packed value|
  int bad;           // first reference without a positive norm, or 2^31 - 1
};
struct RefArgs {
  const float* refs;
  int K, L, r_min, R, R4, NS, n_ref_tiles, normalize, prec;
  const double2* cs64;
  double* q64;       // [K][R][256]
  double* inv;       // [K]  1/norm (or 1)
  double* norm;      // [K]
  double2* Qs;       // [K][129][R]  w_r Q / (norm 256)
  float* qhat32;     // [K][R][256]
  float* B32;
  uint16_t* B16;
  float2* G1;        // K = 1: [R][128] (c - d, c + d) per slot, else null
  RefInfo* info;
  Stencil* stencil;  // out: [R][256]
  float b_scale;
  float* bnorm;      // FP32: [K] norm of each reference's operand (rounded up), else null
};
hipError_t launch_ref_stage1(const RefArgs& a, hipStream_t st);  // polar, norm, spectra, qhat, bmax
hipError_t launch_ref_stage2(const RefArgs& a, hipStream_t st);  // pack B32 / B16

// class averages
struct AvgArgs {
  const float* parts;
  int64_t N;
  int K, L, cx;
  const int32_t *ref, *shift_x, *shift_y, *psi, *mirror;
  const double2* cs64;
  int n_blk;            // ceil(N / 1024)
  int* blk_cnt;         // [n_blk][K]
  int* blk_off;         // [n_blk][K]
  int* cls_start;       // [K + 1]
  int* chunk_start;     // [K + 1]
  int* order;           // [N]
  int max_chunks;
  float* partial;       // [max_chunks][L*L]
  float* averages;      // [K][L][L] in/out
  int32_t* counts;      // [K]
};
hipError_t launch_averages(const AvgArgs& a, hipStream_t st);

}  // namespace mra
