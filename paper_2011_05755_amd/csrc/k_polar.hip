// Shift + polar resampling and per-ring FFT of particle images (Algorithm 1:
// each shifted particle resampled to polar coordinates and transformed per
// ring) and the FP32 re-score of a winning candidate.
//
// One workgroup per particle (a part of one where there are few), 8 waves
// and two to a CU where the LDS holds two images (16 waves, against 12 with
// three 4-wave groups, which ran 10 % slower), else up to 16 waves.  The
// window of the image that the samples read is staged once in LDS with a zero
// border (coalesced HBM read), beside a float-float cos/sin table; the
// (ring, 8-row group) items of the particle are split between the waves.
// In an item, lane (l, row) needs the 32 samples p[16 n1 + 2l + e] of shift
// `row`; integer shifts move the bilinear taps by whole pixels, so each of
// the 8 lanes of group l computes the positions and weights of 4 of those
// angles (from the table: the item loop issues no memory loads) and samples
// them at all 8 shifts, and a transpose through LDS regroups the samples by
// shift.
// What bounds it (20 000 particles of 76 px, 7 x 7 shifts, 35 rings, BF16):
// LDS, busy 92 % of the time and two fifths of that bank conflicts (a half before
// taps were shared), and the vector units, busy 84 %.  The 16-bit forms read
// each column of taps once for all rows that share it, write their samples
// to the transpose from the branch that takes them, stage each spectrum value
// already rounded, and spread a wave's taps over the circle and over a row
// pitch that collides little: 10.67 -> 9.3 ms (and 128 px, 9 x 9 shifts, 62
// rings, 1200 particles: 2.25 -> 1.79 ms).  The FP32 form serves only the
// unpruned path.
// The 256-point real FFT runs as a 16 x 8 complex FFT across the eight
// lanes l of a shift, with a transpose through a per-wave LDS scratch, and
// the spectra are staged there again so that an item's 128 slots of one
// ring are written as one contiguous 8 KB run of the operand (18 GB in 9.3 ms;
// runs of 64-byte pieces scattered over the tile write far slower).
#include <algorithm>

#include "mra_common.h"
#include "mra_fft.h"
#include "polar_impl.h"

namespace mra {

constexpr int kPolarMaxWaves = 16;

// Workgroup -> item: consecutive items on the same XCD (workgroups are dealt
// to the 8 XCDs round-robin), so row tiles shared by neighbouring particles
// are completed in one L2.  The grid is a multiple of 8.
__device__ __forceinline__ int xcd_item() {
  const int per_xcd = gridDim.x / 8;
  return (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
}

template <int MODE, int OUT>
__device__ __forceinline__ void polar_particle(const PolarArgs& a, int n, int part, float* smem) {
  const int NT = blockDim.x, NW = NT >> 6;
  float* img = smem;  // (first: its tap addresses take no base)
  CosSin* cs = reinterpret_cast<CosSin*>(smem + ((a.rows * a.Lp + 3) & ~3));
  float2* scr = reinterpret_cast<float2*>(cs + kNphi);
  float* red = reinterpret_cast<float*>(scr + NW * 64 * 9);
  const float peak = stage_window(img, a.parts + (size_t)n * a.L * a.L, a.L, a.Lp, a.rows, a.pad, OUT == kOutFP16);
  stage_cs(cs, a.cs64);
  if constexpr (OUT == kOutFP16) {
    float m = peak;
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  }
  __syncthreads();

  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), ln = threadIdx.x & 63;
  const int l = ln >> 3, rl = ln & 7;
  if (a.rowkey && part == 0)
    for (int i = threadIdx.x; i < a.S; i += NT) a.rowkey[(size_t)n * a.S + i] = 0ull;
  float hscale = 1.f;
  if constexpr (OUT == kOutFP16) {
    float m = 0.f;  // max |pixel| of the particle
    for (int i = 0; i < NW; ++i) m = fmaxf(m, red[i]);
    if (threadIdx.x == 0) a.maxabs[n] = m;
    hscale = fp16_operand_scale(m);
  }
  float2* my = scr + w * 64 * 9;                // per-wave scratch: 64 lanes x 9 float2
  float* stage = reinterpret_cast<float*>(my);  // [64 slots][16] in each staging round
  const int base = (a.cx + a.pad) * a.Lp + (a.cx + a.pad);
  const int Lp4 = 4 * a.Lp, s1m = (65536 + a.S1 - 1) / a.S1;
  // lane rl handles row (q0 + grp) * 8 + rl: groups are aligned to the
  // correlation kernel's 8-row tiles
  const int row0 = n * a.S;
  const int q0 = row0 >> 3;
  const int ngrp = ((row0 + a.S - 1) >> 3) - q0 + 1;

  if constexpr (MODE == 0 && OUT != kOutF32) {
    // padding rings of the 16-bit operand are read with the others: zeros
    // (16-byte chunks of one row each)
    const int pad_rings = 4 * a.R4 - a.R, chunks = pad_rings * 256;
    for (int i = part * NT + threadIdx.x; i < ngrp * chunks; i += NT * a.split) {
      const int grp = i / chunks, c = i - grp * chunks;
      const int tile = q0 + grp, row = tile * 8 + (c & 7) - row0;
      if (row >= 0 && row < a.S)
        reinterpret_cast<uint4*>(a.out)[((size_t)(tile * 4 * a.R4 + a.R) * 256) + c] = make_uint4(0u, 0u, 0u, 0u);
    }
  }

  // (ring, row group) items in contiguous blocks per wave (balanced)
  const int n_items = a.R * ngrp;
  const int per_wave = (n_items + NW * a.split - 1) / (NW * a.split);
  const int it0 = (part * NW + w) * per_wave, it1 = min(n_items, it0 + per_wave);
  for (int item = it0; item < it1; ++item) {
    const int ring = item / ngrp, grp = item - ring * ngrp;
    // FP32 operand: the shift and lane indices are made opaque here, so that
    // the addresses derived from them are recomputed in every item instead
    // of being hoisted out of the loop and kept in registers (kept, with
    // those of the lane group's index lx, they take the kernel past 128
    // registers and two workgroups per CU); the 16-bit instances keep them
    // all (about 20 % fewer vector instructions).
    const int lx = l;
    int rx = rl, lnx = ln;
    if constexpr (OUT == kOutF32) {
      asm volatile("" : "+v"(rx), "+v"(lnx));
      // (their ranges restated, so that products with them take the 24-bit multiplier)
      rx &= 7;
      lnx &= 63;
    }
    int k1a, k1b;
    fwd_cols(lx, k1a, k1b);
    const int s = (q0 + grp) * 8 + rx - row0;
    const bool valid = s >= 0 && s < a.S;

    float2 z[16];
    if constexpr (OUT != kOutF32) {
      sample_runs(img, cs, my, (float)(a.r_min + ring), lx, rx, (q0 + grp) * 8 - row0, a.S1, s1m, a.T, 4 * base, Lp4, z);
    } else {
      const int sc = s < 0 ? 0 : (s < a.S ? s : a.S - 1);
      const int o4 = 4 * (base + shift_offset(sc, a.S1, s1m, a.T, a.Lp));
      float v[32];
      sample_ring(img, cs, my, (float)(a.r_min + ring), lx, rx, o4, Lp4, v);
#pragma unroll
      for (int n1 = 0; n1 < 16; ++n1) z[n1] = make_float2(v[2 * n1], v[2 * n1 + 1]);
    }

    if (MODE == 1) {
      if (valid) {
        float* o = a.out + (((size_t)n * a.S + s) * a.R + ring) * kNphi;
#pragma unroll
        for (int n1 = 0; n1 < 16; ++n1) {
          o[16 * n1 + 2 * lx] = z[n1].x;
          o[16 * n1 + 2 * lx + 1] = z[n1].y;
        }
      }
      continue;
    }

    float2 Za[8], Zb[8];
    fft_ring(cs, my, lx, rx, k1a, k1b, z, Za, Zb);

    if (MODE == 0) {
      // The slots are staged, the 64 low ones and then the 64 high ones, and
      // written so that each store instruction covers whole 128-byte lines of
      // the tile.
      const int tile = q0 + grp;
      const int first = row0 - tile * 8;            // rows of this tile before the particle
      const int last = row0 + a.S - tile * 8;       // first row after the particle
      if constexpr (OUT != kOutF32) {
        RingHalves rs;
        ring_halves<OUT>(cs, lx, Za, Zb, hscale, rs);
        uint16_t* blk = reinterpret_cast<uint16_t*>(a.out) + (size_t)(tile * 4 * a.R4 + ring) * kSlots * 16;
        const bool row_in = rx >= first && rx < last;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          write_half(reinterpret_cast<uint32_t*>(my), blk, h, lx, rx, row_in, rs);
          wave_sync();
        }
      } else {
        RingSlots rs;
        ring_slots(cs, lx, Za, Zb, rs);
        const bool slot_major = a.a_layout == kSlotMajor, perm = a.a_layout == kRingPerm;
        const int ss = slot_major ? a.R4 * 64 : 16;
        float* dst = a.out + (slot_major ? (size_t)tile * kSlots * a.R4 * 64 + ring * 16
                                         : ((size_t)tile * 4 * a.R4 + ring) * kSlots * 16);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          stage_slots(stage, h, rx, rs);
          wave_sync();
          write_f32_half(stage, dst, h, lnx, perm, ss, first, last);
          wave_sync();
        }
      }
    } else {  // MODE 2: plain spectra
      float* o = a.out + (((size_t)n * a.S + (valid ? s : 0)) * a.R + ring) * 129 * 2;
      fwd_emit(lx, Za, Zb, [&](int f) { return twid(cs, f & 255); },
               [&](int slot, float re, float im) {
                 if (!valid) return;
                 if (slot == 0) {
                   o[0] = re; o[1] = 0.f;
                   o[256] = im; o[257] = 0.f;
                 } else {
                   o[2 * slot] = re;
                   o[2 * slot + 1] = im;
                 }
               });
    }
  }
}

template <int MODE, int OUT>
__global__ __launch_bounds__(64 * kPolarMaxWaves, 4) void k_polar_fft(PolarArgs a) {
  extern __shared__ float smem[];
  const int i = xcd_item(), n = i / a.split;
  if (n >= a.n_part) return;
  polar_particle<MODE, OUT>(a, n, i - n * a.split, smem);
}

// every piece of a batch writes the same operand type
template <int OUT>
__global__ __launch_bounds__(64 * kPolarMaxWaves, 4) void k_polar_batch(PolarBatch b) {
  extern __shared__ float smem[];
  const int item = xcd_item();
  if (item >= b.start[b.n]) return;
  int p = 0;
  while (p + 1 < b.n && b.start[p + 1] <= item) ++p;
  const int i = item - b.start[p], n = i / b.piece[p].split;
  polar_particle<0, OUT>(b.piece[p], n, i - n * b.piece[p].split, smem);
}

static int polar_out(const PolarArgs& a) {
  return a.a_layout != kRingPerm16 ? kOutF32 : (a.prec == kBF16 ? kOutBF16 : kOutFP16);
}

size_t polar_lds_bytes(int Lp) {
  return (size_t)((Lp * Lp + 3) & ~3) * sizeof(float) + (size_t)kPolarWaves * 64 * 9 * sizeof(float2) +
         (size_t)kNphi * sizeof(CosSin) + kPolarWaves * sizeof(float);
}

constexpr size_t kLdsCu = 160 * 1024;
static size_t polar_lds(int rows, int Lp, int waves) {
  return (size_t)((rows * Lp + 3) & ~3) * sizeof(float) + (size_t)waves * 64 * 9 * sizeof(float2) + (size_t)kNphi * sizeof(CosSin) +
         kPolarMaxWaves * sizeof(float);
}

// The LDS image of the pixels lo .. hi (either axis) that a particle's samples
// read.  Row pitch: the taps of a wave lie on half a circle, and how they fall
// on the 32 banks depends on the pitch modulo 32; over radii up to 15, 30, 35,
// 46 and 62 the pitches 6, 10, 22 and 26 (mod 32) take 3.9, 4.6, 4.9, 5.0 and
// 5.4 LDS cycles per read of 64 taps (2 without conflicts), within 3 % of the
// best of any pitch; a multiple of 32 takes 7, an 80-pixel window's own side 5.4
// (kernel, 76 px BF16: 9.41 ms at pitch 86, 9.60 at 80).  The window's own side where the wider rows would cost
// the CU a workgroup.
void polar_window(PolarArgs& a, int lo, int hi) {
  a.pad = -lo;
  a.rows = hi - lo + 1;
  int P = a.rows;
  while (P % 32 != 6 && P % 32 != 10 && P % 32 != 22 && P % 32 != 26) ++P;
  const size_t wide = polar_lds(a.rows, P, kPolarWaves), own = polar_lds(a.rows, a.rows, kPolarWaves);
  a.Lp = wide > kLdsCu || (wide > kLdsCu / 2 && own <= kLdsCu / 2) ? a.rows : P;
}

// Waves per workgroup: 8, two workgroups to a CU; where the image leaves room
// for only one, as many as its LDS holds, up to 16 (128 px, 9 x 9 shifts, BF16,
// 1200 particles: 1.79 ms with 16 waves, 1.99 with 8).
int polar_waves(const PolarArgs& a) {
  if (polar_lds(a.rows, a.Lp, kPolarWaves) <= kLdsCu / 2) return kPolarWaves;
  int w = kPolarMaxWaves;
  while (w > 1 && polar_lds(a.rows, a.Lp, w) > kLdsCu) --w;
  return w;
}

hipError_t launch_polar_batch(const PolarBatch& b, hipStream_t st) {
  if (b.n <= 0 || b.start[b.n] <= 0) return hipSuccess;
  const int out = polar_out(b.piece[0]);
  int waves = kPolarMaxWaves;
  for (int i = 0; i < b.n; ++i) {
    waves = std::min(waves, polar_waves(b.piece[i]));
    if (polar_out(b.piece[i]) != out) return hipErrorInvalidValue;
  }
  size_t lds = 0;
  for (int i = 0; i < b.n; ++i) lds = std::max(lds, polar_lds(b.piece[i].rows, b.piece[i].Lp, waves));
  const dim3 grid((b.start[b.n] + 7) / 8 * 8), block(64 * waves);
  switch (out) {
    case kOutF32: hipLaunchKernelGGL(k_polar_batch<kOutF32>, grid, block, lds, st, b); break;
    case kOutBF16: hipLaunchKernelGGL(k_polar_batch<kOutBF16>, grid, block, lds, st, b); break;
    default: hipLaunchKernelGGL(k_polar_batch<kOutFP16>, grid, block, lds, st, b); break;
  }
  return hipGetLastError();
}

hipError_t launch_polar(int mode, const PolarArgs& a, hipStream_t st) {
  if (a.n_part <= 0) return hipSuccess;
  if (a.split < 1) return hipErrorInvalidValue;
  const int waves = polar_waves(a);
  const size_t lds = polar_lds(a.rows, a.Lp, waves);
  if (lds > kLdsCu) return hipErrorInvalidValue;
  dim3 grid(((unsigned)a.n_part * a.split + 7) / 8 * 8), block(64 * waves);
  switch (mode) {
    case 0:
      switch (polar_out(a)) {
        case kOutF32: hipLaunchKernelGGL((k_polar_fft<0, kOutF32>), grid, block, lds, st, a); break;
        case kOutBF16: hipLaunchKernelGGL((k_polar_fft<0, kOutBF16>), grid, block, lds, st, a); break;
        default: hipLaunchKernelGGL((k_polar_fft<0, kOutFP16>), grid, block, lds, st, a); break;
      }
      break;
    case 1: hipLaunchKernelGGL((k_polar_fft<1, kOutF32>), grid, block, lds, st, a); break;
    default: hipLaunchKernelGGL((k_polar_fft<2, kOutF32>), grid, block, lds, st, a); break;
  }
  return hipGetLastError();
}

// FP32 re-score of each particle's winner: the direct double sum
// sum_r w_r sum_j p_{s,m}[r][j] * qhat_k[r][(j + a) mod 256] with a = -psi.
// The mirrored samples are the unmirrored stencil read at angle -j (the
// stencil table is built symmetric in j <-> 256 - j).  With a.rows >= 2 the
// candidates are the winners of the particle's a.rows best rows of the 16-bit
// pass and their neighbours one angle step either side; the best FP32 value
// wins (ties: the smallest flat index) and replaces the parameters.  Rows
// whose 16-bit best lies more than a.margin of the particle's 16-bit
// best below it are left out (they cannot win at 16-bit accuracy).
constexpr int kMaxRescoreRows = 8;

constexpr int kRescoreRed = 24;  // reduction slots: 4 waves x 3 lags x up to 2 candidates

// FP32 CC of (ref k, shift soff, mirror m) at the lags lag0 + d, d < ND, for
// the image staged in img; red holds 4 ND doubles.  Reduction in a fixed
// order (per-thread FP32 ring sum, then FP64 across the block), the same for
// every d.
template <int ND>
__device__ __forceinline__ void rescore_lags(const RescoreArgs& a, const float* img, double* red, int k, int m,
                                             int soff, int lag0, double (&out)[ND]) {
  const int base = (a.cx + a.pad) * a.Lp + (a.cx + a.pad);
  const int j = threadIdx.x;
  const int jj = m ? ((kNphi - j) & 255) : j;
  const float* q = a.qhat + (size_t)k * a.R * kNphi;
  float acc[ND];
#pragma unroll
  for (int d = 0; d < ND; ++d) acc[d] = 0.f;
  // unrolled so that the stencil and spectrum loads of several rings are in
  // flight at once (the loop is bound by their latency, not by arithmetic)
#pragma unroll 8
  for (int r = 0; r < a.R; ++r) {
    const Stencil st = a.stencil[r * kNphi + jj];
    const float p = bilin(img, base + st.dy * a.Lp + (st.bx >> 2) + soff, a.Lp, st.fx, st.fy);
    const float w = (float)(a.r_min + r);
#pragma unroll
    for (int d = 0; d < ND; ++d) acc[d] += w * (p * q[r * kNphi + ((j + lag0 + d) & 255)]);
  }
  // FP64 sum over the 256 threads in a fixed order: a butterfly within each
  // wave (every lane ends with the wave's sum), then the four waves' sums in
  // wave order
  double v[ND];
#pragma unroll
  for (int d = 0; d < ND; ++d) {
    v[d] = (double)acc[d];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v[d] += __shfl_xor(v[d], o);
  }
  if ((j & 63) == 0) {
#pragma unroll
    for (int d = 0; d < ND; ++d) red[d * 4 + (j >> 6)] = v[d];
  }
  __syncthreads();
#pragma unroll
  for (int d = 0; d < ND; ++d) out[d] = ((red[d * 4] + red[d * 4 + 1]) + red[d * 4 + 2]) + red[d * 4 + 3];
  __syncthreads();
}

// The same FP32 CC for NC candidates (ref k[c], mirror m[c], shift soff[c])
// at the lags lag0[c] + d, d < 3, evaluated together: each ring's stencil is
// loaded once per mirror that occurs (MIXED: both occur) and serves every
// candidate of that mirror, and the NC * 3 sums share one reduction (red
// holds 12 NC doubles).  Every sum takes the arithmetic of rescore_lags<3> in
// the same order, so the values are bit-identical to evaluating the
// candidates one at a time.  The unroll keeps either form within 80
// registers, six workgroups per CU (the four-candidate form needs 117, and
// its occupancy costs more than the shared loads save).
template <int NC, bool MIXED>
__device__ __forceinline__ void rescore_group(const RescoreArgs& a, const float* img, double* red, const int* k,
                                              const int* m, const int* soff, const int* lag0, double (&out)[NC][3]) {
  const int base = (a.cx + a.pad) * a.Lp + (a.cx + a.pad);
  const int j = threadIdx.x;
  const int jm = (kNphi - j) & 255;
  // unmixed: every candidate's mirror is m[0]
  const Stencil* st0 = a.stencil + (MIXED ? j : (m[0] ? jm : j));
  const Stencil* st1 = a.stencil + jm;
  float acc[NC][3];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int d = 0; d < 3; ++d) acc[c][d] = 0.f;
  static_assert(NC * 12 <= kRescoreRed, "reduction slots");
  constexpr int kUnroll = NC == 1 ? 8 : 2;
#pragma unroll kUnroll
  for (int r = 0; r < a.R; ++r) {
    const Stencil s0 = st0[r * kNphi];
    Stencil s1 = s0;
    if constexpr (MIXED) s1 = st1[r * kNphi];
    const float w = (float)(a.r_min + r);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const Stencil st = (MIXED && m[c]) ? s1 : s0;
      const float p = bilin(img, base + st.dy * a.Lp + (st.bx >> 2) + soff[c], a.Lp, st.fx, st.fy);
      const float* q = a.qhat + ((size_t)k[c] * a.R + r) * kNphi;
#pragma unroll
      for (int d = 0; d < 3; ++d) acc[c][d] += w * (p * q[(j + lag0[c] + d) & 255]);
    }
  }
  // the reduction of rescore_lags, for every sum
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      double v = (double)acc[c][d];
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
      if ((j & 63) == 0) red[(c * 3 + d) * 4 + (j >> 6)] = v;
    }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double* r4 = red + (c * 3 + d) * 4;
      out[c][d] = ((r4[0] + r4[1]) + r4[2]) + r4[3];
    }
  __syncthreads();
}

// Candidates cand[0 .. NC - 1] (flat indices, NC <= 2):
// their FP32 values at the three lags around each one's angle, folded into
// (best, best_i) in list order (ties: the smallest flat index).
template <int NC>
__device__ __forceinline__ void rescore_fold(const RescoreArgs& a, const float* img, double* red, const int* cand,
                                             float& best, int& best_i) {
  int k[NC], m[NC], soff[NC], lag0[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int idx = __builtin_amdgcn_readfirstlane(cand[c]);  // the same in every lane
    const int ang = idx & 255;
    int rest = idx >> 8;
    const int s = rest % a.S;
    rest /= a.S;
    m[c] = rest % a.M;
    k[c] = rest / a.M;
    soff[c] = (s / a.S1 - a.T) * a.Lp + (s % a.S1 - a.T);
    lag0[c] = (ang + 255) & 255;
  }
  bool mixed = false;  // workgroup-uniform
#pragma unroll
  for (int c = 1; c < NC; ++c) mixed |= m[c] != m[0];
  double v[NC][3];
  if (mixed)
    rescore_group<NC, true>(a, img, red, k, m, soff, lag0, v);
  else
    rescore_group<NC, false>(a, img, red, k, m, soff, lag0, v);
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const int i2 = (__builtin_amdgcn_readfirstlane(cand[c]) & ~255) | ((lag0[c] + d) & 255);
      const float f = (float)v[c][d];
      if (f > best || (f == best && i2 < best_i)) {
        best = f;
        best_i = i2;
      }
    }
}

__device__ __forceinline__ void rescore_particle(const RescoreArgs& a, int n, float* smem) {
  float* img = smem;
  double* red = reinterpret_cast<double*>(smem + ((a.Lp * a.Lp + 1) & ~1));
  int* cand = reinterpret_cast<int*>(red + kRescoreRed);  // candidate rows' flat indices
  const int64_t gi = a.out_off + n;
  stage_image(img, a.parts + (size_t)n * a.L * a.L, a.L, a.Lp, a.pad);
  if (a.rows <= 1) {
    __syncthreads();
    const int k = a.ref[gi], m = a.mirror[gi] ? 1 : 0;
    const int sx = a.shift_x[gi], sy = a.shift_y[gi];
    if (k < 0 || k >= a.K || sx < -a.T || sx > a.T || sy < -a.T || sy > a.T) {
      if (threadIdx.x == 0) a.cc[gi] = NAN;
      return;  // uniform over the block
    }
    double v[1];
    rescore_lags<1>(a, img, red, k, m, sy * a.Lp + sx, (kNphi - a.psi[gi]) & 255, v);
    if (threadIdx.x == 0) a.cc[gi] = (float)v[0];
    return;
  }
  // the a.rows best rows of the 16-bit pass, by wave 0: lane l holds rows
  // l + 64 i, and each round takes the largest (value, then smallest flat
  // index) of the rows not yet taken across the wave.  Rows without a
  // candidate (index 2^31 - 1) and NaN values never count.
  if (threadIdx.x < 64) {
    constexpr int kPer = (kMaxShifts + 63) / 64;
    const int l = threadIdx.x;
    float lv[kPer];
    int li[kPer];
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      const int s = l + 64 * e;
      lv[e] = s < a.S ? a.row_cc[(size_t)n * a.S + s] : -INFINITY;
      li[e] = s < a.S ? a.row_idx[(size_t)n * a.S + s] : 0x7fffffff;
      if (lv[e] != lv[e]) li[e] = 0x7fffffff;
    }
    const int nr = a.rows < kMaxRescoreRows ? a.rows : kMaxRescoreRows;
    float top = -INFINITY;
    for (int t = 0; t < kMaxRescoreRows; ++t) {
      float bv = -INFINITY;
      int bi = 0x7fffffff;
      if (t < nr) {  // uniform
#pragma unroll
        for (int e = 0; e < kPer; ++e)
          if (li[e] != 0x7fffffff && (lv[e] > bv || (lv[e] == bv && li[e] < bi))) {
            bv = lv[e];
            bi = li[e];
          }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
          const float ov = __shfl_xor(bv, o);
          const int oi = __shfl_xor(bi, o);
          if (ov > bv || (ov == bv && oi < bi)) {
            bv = ov;
            bi = oi;
          }
        }
#pragma unroll
        for (int e = 0; e < kPer; ++e)
          if (li[e] == bi) li[e] = 0x7fffffff;  // taken (flat indices are distinct)
      }
      if (t == 0) top = bv;
      // only rows within the re-ranking margin of the particle's best are
      // candidates; pruning keeps their bests exact
      const float lim = top > -INFINITY ? top - a.margin * fabsf(top) : top;
      if (l == 0) cand[t] = (t < nr && bv >= lim) ? bi : 0x7fffffff;
    }
  }
  __syncthreads();
  int nc = 0;  // the candidates form a prefix of the list (values descend)
  while (nc < kMaxRescoreRows && __builtin_amdgcn_readfirstlane(cand[nc]) != 0x7fffffff) ++nc;
  float best = -INFINITY;
  int best_i = 0x7fffffff;
  for (int t0 = 0; t0 < nc; t0 += 2) {  // workgroup-uniform
    if (nc - t0 == 1)
      rescore_fold<1>(a, img, red, cand + t0, best, best_i);
    else
      rescore_fold<2>(a, img, red, cand + t0, best, best_i);
  }
  if (threadIdx.x != 0) return;
  if (best_i == 0x7fffffff) {  // the 16-bit pass found no candidate: keep its (invalid) result
    a.cc[gi] = NAN;
    return;
  }
  const int ang = best_i & 255;
  int rest = best_i >> 8;
  const int s = rest % a.S;
  rest /= a.S;
  const int m = rest % a.M, k = rest / a.M;
  a.ref_w[gi] = k;
  a.mirror_w[gi] = m;
  a.shift_x_w[gi] = s % a.S1 - a.T;
  a.shift_y_w[gi] = s / a.S1 - a.T;
  a.psi_w[gi] = (kNphi - ang) & 255;
  a.cc[gi] = best;
  if (a.flat_w) a.flat_w[gi] = best_i;
  if (a.win) a.win[n] = best_i;
}

static size_t rescore_lds_bytes(int Lp) {
  return (size_t)((Lp * Lp + 1) & ~1) * sizeof(float) + kRescoreRed * sizeof(double) +
         kMaxRescoreRows * sizeof(int);
}

__global__ __launch_bounds__(256) void k_rescore(RescoreArgs a) {
  extern __shared__ float smem[];
  rescore_particle(a, blockIdx.x, smem);
}

__global__ __launch_bounds__(256) void k_rescore_batch(RescoreBatch b) {
  extern __shared__ float smem[];
  const int item = blockIdx.x;
  int p = 0;
  while (p + 1 < b.n && b.start[p + 1] <= item) ++p;
  rescore_particle(b.piece[p], item - b.start[p], smem);
}

hipError_t launch_rescore(const RescoreArgs& a, hipStream_t st) {
  if (a.n_part <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_rescore, dim3(a.n_part), dim3(256), rescore_lds_bytes(a.Lp), st, a);
  return hipGetLastError();
}

hipError_t launch_rescore_batch(const RescoreBatch& b, hipStream_t st) {
  if (b.n <= 0 || b.start[b.n] <= 0) return hipSuccess;
  int lp = 0;
  for (int i = 0; i < b.n; ++i) lp = b.piece[i].Lp > lp ? b.piece[i].Lp : lp;
  hipLaunchKernelGGL(k_rescore_batch, dim3(b.start[b.n]), dim3(256), rescore_lds_bytes(lp), st, b);
  return hipGetLastError();
}

// Sub-step angle of each particle's final winner: the FP32 CC at lags
// a - 1, a, a + 1 (a = -psi) and the vertex of the parabola through them.
__global__ __launch_bounds__(256) void k_refine(RescoreArgs a) {
  extern __shared__ float smem[];
  float* img = smem;
  double* red = reinterpret_cast<double*>(smem + ((a.Lp * a.Lp + 1) & ~1));
  const int n = blockIdx.x;
  const int64_t gi = a.out_off + n;
  stage_image(img, a.parts + (size_t)n * a.L * a.L, a.L, a.Lp, a.pad);
  __syncthreads();
  const int k = a.ref[gi], m = a.mirror[gi] ? 1 : 0;
  const int sx = a.shift_x[gi], sy = a.shift_y[gi], psi = a.psi[gi];
  if (k < 0 || k >= a.K || sx < -a.T || sx > a.T || sy < -a.T || sy > a.T) {
    if (threadIdx.x == 0) a.psi_frac[gi] = NAN;
    return;  // uniform over the block
  }
  const int ang = (kNphi - psi) & 255;
  double v[3];
  rescore_lags<3>(a, img, red, k, m, sy * a.Lp + sx, (ang + 255) & 255, v);
  if (threadIdx.x == 0) {
    const double den = v[0] - 2.0 * v[1] + v[2];
    double d = den < 0.0 ? 0.5 * (v[0] - v[2]) / den : 0.0;
    d = d < -0.5 ? -0.5 : (d > 0.5 ? 0.5 : d);
    double f = (double)psi - d;
    if (f < 0.0) f += kNphi;
    if (f >= kNphi) f -= kNphi;
    a.psi_frac[gi] = (float)f;
  }
}

hipError_t launch_refine(const RescoreArgs& a, hipStream_t st) {
  if (a.n_part <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_refine, dim3(a.n_part), dim3(256), rescore_lds_bytes(a.Lp), st, a);
  return hipGetLastError();
}

}  // namespace mra
