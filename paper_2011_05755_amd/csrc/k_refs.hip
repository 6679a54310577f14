// Reference preparation (Algorithm 1: each reference resampled to polar
// coordinates and transformed per ring), done once per reference set in FP64:
//   q_k[r][j]  bilinear polar samples at zero shift,
//   nu_k       weighted ring norm sqrt(sum_r w_r sum_j q^2),
//   Q_k[r][f]  per-ring DFT (direct sum), times w_r / (nu_k * 256),
// then packed into the operand layouts of the correlation kernel:
//   FP32  [ref, padded to whole tiles][slot][2 g + q][t, padded to 16 bytes], ring = g*R4 + t, t < R4
//   16-bit [ref tile][slot][s < NS - 1][64][8], lane = 16 g + 2 (ref%8) + q, ring = g*R4 + 8 s + e,
//          then the last step [64][BT] (BT = 2, 4 or 8: as wide as its rings need);
//          an FP32 refset holds an FP16 one too, for the bounds
// with q = 0 -> c - d and q = 1 -> c + d for c + id = Q_f (slot f = 1..127)
// and c = Q_0, d = Q_128 in slot 0; with one reference also
//   single [ring][slot] (c - d, c + d) for the fused single-reference kernel.
#include "mra_common.h"

namespace mra {

__global__ void k_ref_polar(RefArgs a) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i == 0) *a.info = RefInfo{0.f, INT32_MAX};
  if (i >= (int64_t)a.K * a.R * kNphi) return;
  const int j = i % kNphi;
  const int ring = (i / kNphi) % a.R;
  const int k = i / ((int64_t)kNphi * a.R);
  const int c = a.L / 2;
  const double r = a.r_min + ring;
  const double x = c + r * a.cs64[j].x, y = c + r * a.cs64[j].y;
  const double x0 = floor(x), y0 = floor(y);
  const double fx = x - x0, fy = y - y0;
  const int ix = (int)x0, iy = (int)y0;
  const float* img = a.refs + (size_t)k * a.L * a.L;
  auto pix = [&](int xx, int yy) -> double {
    return (xx >= 0 && xx < a.L && yy >= 0 && yy < a.L) ? (double)img[yy * a.L + xx] : 0.0;
  };
  a.q64[i] = (1 - fx) * (1 - fy) * pix(ix, iy) + fx * (1 - fy) * pix(ix + 1, iy) +
             (1 - fx) * fy * pix(ix, iy + 1) + fx * fy * pix(ix + 1, iy + 1);
}

// Blocks 0 .. K - 1: the norm of reference k.  The next R blocks: the particle
// sampling stencil of one ring each (FP64 positions; exactly symmetric in
// j <-> 256 - j, as the table is).
__global__ __launch_bounds__(256) void k_ref_norm(RefArgs a) {
  __shared__ double red[256];
  const int k = blockIdx.x, j = threadIdx.x;
  if (k >= a.K) {
    const int ring = k - a.K;
    const double r = a.r_min + ring;
    const double x = __dmul_rn(r, a.cs64[j].x), y = __dmul_rn(r, a.cs64[j].y);
    const double fx = floor(x), fy = floor(y);
    Stencil s;
    s.bx = 4 * (int)fx;
    s.dy = (int)fy;
    s.fx = (float)(x - fx);
    s.fy = (float)(y - fy);
    a.stencil[ring * kNphi + j] = s;
    return;
  }
  double acc = 0.0;
#pragma unroll 8
  for (int ring = 0; ring < a.R; ++ring) {
    const double q = a.q64[((size_t)k * a.R + ring) * kNphi + j];
    acc += (double)(a.r_min + ring) * q * q;
  }
  red[j] = acc;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (j < h) red[j] += red[j + h];
    __syncthreads();
  }
  if (j == 0) {
    const double nu = sqrt(red[0]);
    a.norm[k] = nu;
    a.inv[k] = a.normalize ? (nu > 0.0 ? 1.0 / nu : 0.0) : 1.0;
    if (!(nu > 0.0)) atomicMin(&a.info->bad, k);
  }
}

// Per-ring DFTs of one reference (blockIdx.x), by the direct sum in FP64 (its
// order, ascending angles, is part of the result); also qhat and the
// largest packed value.  Lane = ring, so that the reads of Q's rows are
// conflict-free, the twiddles uniform (scalar) loads and Qs is written
// coalesced; a wave sums 4 frequencies per read (wave 0 of part 0 also f =
// 128, the partner of f = 0 in slot 0).  FP64 FMA bound: one thread per
// (frequency, ring) reading its own row from memory took 0.2 ms for 100
// references of 36 rings, this 0.03 ms.
constexpr int kDftParts = 4, kDftPitch = kNphi + 1;
__global__ __launch_bounds__(512) void k_ref_spectra(RefArgs a) {
  extern __shared__ double rows[];  // [R][kDftPitch]
  const int k = blockIdx.x, part = blockIdx.y;
  const double inv = a.inv[k];
  for (int i = threadIdx.x; i < a.R * kNphi; i += 512) {
    const double q = a.q64[(size_t)k * a.R * kNphi + i];
    rows[(i / kNphi) * kDftPitch + i % kNphi] = q;
    if (part == 0) a.qhat32[(size_t)k * a.R * kNphi + i] = (float)(q * inv);
  }
  __syncthreads();
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), ln = threadIdx.x & 63;
  const int ring = ln < a.R ? ln : a.R - 1;
  const double* q = rows + ring * kDftPitch;
  const int f0 = (part * 8 + w) * 4;
  const bool first = f0 == 0;  // wave-uniform
  double re[5] = {0, 0, 0, 0, 0}, im[4] = {0, 0, 0, 0};
#pragma unroll 4
  for (int j = 0; j < kNphi; ++j) {
    const double v = q[j];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double2 t = a.cs64[((f0 + e) * j) & 255];
      re[e] += v * t.x;
      im[e] -= v * t.y;
    }
    if (first) re[4] += v * a.cs64[(128 * j) & 255].x;
  }
  const double s = (double)(a.r_min + ring) * inv / kNphi;
  float m = 0.f;
  auto seen = [&](double c, double d) { m = fmaxf(m, fmaxf((float)fabs(c - d), (float)fabs(c + d))); };
  double2* out = a.Qs + (size_t)k * 129 * a.R + ring;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const double2 v = make_double2(re[e] * s, im[e] * s);
    if (ln < a.R) out[(size_t)(f0 + e) * a.R] = v;
    if (!(first && e == 0)) seen(v.x, v.y);
  }
  if (first) {  // (its imaginary part, zero up to rounding, is not used)
    const double2 v = make_double2(re[4] * s, 0.0);
    if (ln < a.R) out[(size_t)128 * a.R] = v;
    seen(re[0] * s, v.x);
  }
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
  if (ln == 0) atomicMax(reinterpret_cast<unsigned int*>(&a.info->bmax), __float_as_uint(m));
}

// element of reference ref (q, slot) at ring `ring`
__device__ __forceinline__ double packed_value(const RefArgs& a, int ref, int slot, int q, int ring) {
  if (ring >= a.R || ref >= a.K) return 0.0;
  const double2* Q = a.Qs + (size_t)ref * 129 * a.R;
  double c, d;
  if (slot == 0) {
    c = Q[0 * a.R + ring].x;
    d = Q[128 * a.R + ring].x;
  } else {
    c = Q[slot * a.R + ring].x;
    d = Q[slot * a.R + ring].y;
  }
  return q ? c + d : c - d;
}

__device__ __forceinline__ void pack32(const RefArgs& a, int64_t i) {
  const int pitch = b32_pitch(a.R4);
  if (i >= (int64_t)a.n_ref_tiles * kRefTile * kSlots * 8 * pitch) return;
  const int t = i % pitch, gq = (i / pitch) & 7, slot = (i / (8 * pitch)) % kSlots;
  const int ref = i / ((int64_t)8 * pitch * kSlots);
  a.B32[i] = t < a.R4 ? (float)packed_value(a, ref, slot, gq & 1, (gq >> 1) * a.R4 + t) : 0.f;
}

__device__ __forceinline__ void pack16(const RefArgs& a, int64_t i) {
  const int se = b16_slot_elems(a.R4), bt = b16_tail_width(a.R4);
  if (i >= (int64_t)a.n_ref_tiles * kSlots * se) return;
  const int off = i % se;
  const int slot = (i / se) % kSlots, kt = i / ((int64_t)se * kSlots);
  const int full = (a.NS - 1) * 512;  // elements of the steps stored 8 wide
  int lane, t;
  if (off < full) {
    lane = (off / 8) % 64;
    t = 8 * (off / 512) + off % 8;
  } else {
    lane = (off - full) / bt;
    t = 8 * (a.NS - 1) + (off - full) % bt;
  }
  // lane = 16 ring group + 2 reference + q
  const int g = lane >> 4;
  const double v = t < a.R4 ? packed_value(a, kt * kRefTile + ((lane >> 1) & 7), slot, lane & 1, g * a.R4 + t) * a.b_scale : 0.0;
  if (a.prec == kBF16) {
    __bf16 h = (__bf16)(float)v;
    a.B16[i] = __builtin_bit_cast(uint16_t, h);
  } else {
    _Float16 h = (_Float16)(float)v;
    a.B16[i] = __builtin_bit_cast(uint16_t, h);
  }
}

// K = 1: the single reference's weighted spectrum per (ring, slot) as
// (c - d, c + d), read by the fused single-reference kernel.
__device__ __forceinline__ void pack_single(const RefArgs& a, int64_t i) {
  if (i >= a.R * kSlots) return;
  const int ring = i / kSlots, slot = i % kSlots;
  double c, d;
  if (slot == 0) {
    c = a.Qs[0 * a.R + ring].x;
    d = a.Qs[128 * a.R + ring].x;
  } else {
    c = a.Qs[slot * a.R + ring].x;
    d = a.Qs[slot * a.R + ring].y;
  }
  a.G1[i] = make_float2((float)(c - d), (float)(c + d));
}

// Norm of reference k's packed operand, 2 sum |Q|^2 over its slots and
// rings, rounded up.
__device__ __forceinline__ void operand_norm(const RefArgs& a, int k) {
  __shared__ double red[4];
  double s = 0.0;
  for (int i = threadIdx.x; i < 129 * a.R; i += 256) {
    const double2 q = a.Qs[(size_t)k * 129 * a.R + i];
    s += 2.0 * (q.x * q.x + q.y * q.y);
  }
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) a.bnorm[k] = (float)(sqrt(((red[0] + red[1]) + red[2]) + red[3]) * (1.0 + 1e-6));
}

// Every operand the refset keeps, in one launch (from block `first` on): block
// ranges of n.
struct PackBlocks {
  unsigned single, f32, half, norm;
};
__global__ __launch_bounds__(256) void k_ref_pack(RefArgs a, PackBlocks n, unsigned first) {
  unsigned b = first + blockIdx.x;
  auto at = [&] { return b * (int64_t)256 + threadIdx.x; };
  if (b < n.single) return pack_single(a, at());
  b -= n.single;
  if (b < n.f32) return pack32(a, at());
  b -= n.f32;
  if (b < n.half) return pack16(a, at());
  operand_norm(a, b - n.half);
}

static inline unsigned blocks_for(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

hipError_t launch_ref_stage1(const RefArgs& a, hipStream_t st) {
  const int64_t nq = (int64_t)a.K * a.R * kNphi;
  hipLaunchKernelGGL(k_ref_polar, dim3(blocks_for(nq, 256)), dim3(256), 0, st, a);
  hipLaunchKernelGGL(k_ref_norm, dim3(a.K + a.R), dim3(256), 0, st, a);
  hipLaunchKernelGGL(k_ref_spectra, dim3(a.K, kDftParts), dim3(512), (size_t)a.R * kDftPitch * sizeof(double), st, a);
  return hipGetLastError();
}

hipError_t launch_ref_stage2(const RefArgs& a, hipStream_t st) {
  PackBlocks n{};
  if (a.G1) n.single = blocks_for((int64_t)a.R * kSlots, 256);
  if (a.B32) n.f32 = blocks_for((int64_t)a.n_ref_tiles * kRefTile * kSlots * 8 * b32_pitch(a.R4), 256);
  if (a.B16) n.half = blocks_for((int64_t)a.n_ref_tiles * kSlots * b16_slot_elems(a.R4), 256);
  if (a.bnorm) n.norm = a.K;
  // (a launch holds fewer than 2^32 work-items; FP32 sets pass that at 131 072 to 340 000 references)
  const unsigned total = n.single + n.f32 + n.half + n.norm, most = 0xffffff;
  for (unsigned first = 0; first < total; first += most)
    hipLaunchKernelGGL(k_ref_pack, dim3(total - first < most ? total - first : most), dim3(256), 0, st, a, n, first);
  return hipGetLastError();
}

}  // namespace mra
