// Device helpers shared by the kernels that resample particles onto the
// polar grid: the image staged in LDS with a zero border, bilinear taps,
// twiddles and a wave-level barrier.
#pragma once

#include <type_traits>

#include "mra_common.h"
#include "mra_fft.h"

namespace mra {

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// (cos, sin)(2 pi j / 256) as float-float pairs, cos = ch + cl and
// sin = sh + sl, staged in LDS: the resampling positions and, through
// (ch, sh), the ring FFT twiddles.
struct __attribute__((aligned(16))) CosSin {
  float ch, sh, cl, sl;
};

__device__ __forceinline__ void stage_cs(CosSin* t, const double2* cs64) {
  for (int j = threadIdx.x; j < kNphi; j += blockDim.x) {
    const double2 v = cs64[j];
    CosSin c;
    c.ch = (float)v.x;
    c.sh = (float)v.y;
    c.cl = (float)(v.x - (double)c.ch);
    c.sl = (float)(v.y - (double)c.sh);
    t[j] = c;
  }
}

// exp(-2 pi i e / 256) from the staged table
__device__ __forceinline__ float2 twid(const CosSin* t, int e) {
  const float2 v = *reinterpret_cast<const float2*>(t + e);
  return make_float2(v.x, -v.y);
}

// Batches of eight loads per thread are issued before any is stored, so the
// HBM latency is paid once per batch rather than once per element.
__device__ __forceinline__ void stage_image(float* img, const float* src, int L, int Lp, int pad) {
  constexpr int kB = 8;
  const int n = Lp * Lp;
  for (int i0 = threadIdx.x; i0 < n; i0 += kB * blockDim.x) {
    float v[kB];
#pragma unroll
    for (int b = 0; b < kB; ++b) {
      const int i = i0 + b * blockDim.x;
      const int yy = i / Lp - pad, xx = i % Lp - pad;
      v[b] = (i < n && yy >= 0 && yy < L && xx >= 0 && xx < L) ? src[yy * L + xx] : 0.f;
    }
#pragma unroll
    for (int b = 0; b < kB; ++b) {
      const int i = i0 + b * blockDim.x;
      if (i < n) img[i] = v[b];
    }
  }
}

// The window of PolarArgs (rows x rows pixels at pitch Lp).  peak: the whole
// image is read, also where the window is smaller, and the thread's largest
// |pixel| returned.
__device__ __forceinline__ float stage_window(float* img, const float* src, int L, int Lp, int rows, int pad, bool peak) {
  constexpr int kB = 8;
  const int lo = peak ? min(0, -pad) : -pad, side = (peak ? max(L, rows - pad) : rows - pad) - lo;
  const int n = side * side;
  float m = 0.f;
  for (int i0 = threadIdx.x; i0 < n; i0 += kB * blockDim.x) {
    float v[kB];
    int at[kB];
#pragma unroll
    for (int b = 0; b < kB; ++b) {
      const int i = i0 + b * blockDim.x;
      const int q = i / side, yy = q + lo, xx = i - q * side + lo;
      v[b] = (i < n && yy >= 0 && yy < L && xx >= 0 && xx < L) ? src[yy * L + xx] : 0.f;
      const int wy = yy + pad, wx = xx + pad;
      at[b] = i < n && wy >= 0 && wy < rows && wx >= 0 && wx < rows ? wy * Lp + wx : -1;
    }
#pragma unroll
    for (int b = 0; b < kB; ++b) {
      if (at[b] >= 0) img[at[b]] = v[b];
      m = fmaxf(m, fabsf(v[b]));
    }
  }
  return m;
}

// The same taps for a byte offset o4 of the top-left pixel and the row pitch
// Lp4 in bytes.
__device__ __forceinline__ float bilin4(const float* img, int o4, int Lp4, float fx, float fy) {
  const char* p = reinterpret_cast<const char*>(img) + o4;
  const float i00 = *reinterpret_cast<const float*>(p), i10 = *reinterpret_cast<const float*>(p + 4);
  const float i01 = *reinterpret_cast<const float*>(p + Lp4), i11 = *reinterpret_cast<const float*>(p + Lp4 + 4);
  const float top = i00 + fx * (i10 - i00);
  const float bot = i01 + fx * (i11 - i01);
  return top + fy * (bot - top);
}

// Offset (in pixels) of integer shift s = sy_index * S1 + sx_index, both
// indices counted from -T, for an image of pitch Lp: (sy - T) Lp + (sx - T).
// s / S1 is taken as (s * m) >> 16 with m = ceil(65536 / S1), which is exact
// for 0 <= s < 65536 / S1 (here s < 289 and S1 <= 17).
__device__ __forceinline__ int shift_offset(int s, int S1, int m, int T, int Lp) {
  const int q = __mul24(s, m) >> 16;
  return __mul24(q, Lp - S1) + s - T * (Lp + 1);
}

// Bilinear taps of the staged image at offset rr (cos, sin) of angle entry
// c from a shift's centre pixel.  Floor and fractions come from the
// float-float cos/sin: each fraction is within a few FP32 ulps of the one
// the FP64 position gives.  Where the position lies within rounding of a
// pixel boundary, floor(rr * ch) can be one off the exact floor; the
// fraction is then just outside [0, 1), the sample is the same up to
// rounding, and the taps reach one pixel further, which the zero border of
// the staged image allows for.  Integer shifts move the taps by whole
// pixels, so one position split serves every shift: the byte offset of the
// top-left tap from the shift's centre pixel, and the four weights.
__device__ __forceinline__ int polar_offset(float rr, const CosSin& c, int Lp4) {
  const float xf = floorf(rr * c.ch), yf = floorf(rr * c.sh);
  return __mul24((int)yf, Lp4) + 4 * (int)xf;
}
__device__ __forceinline__ void polar_weights(float rr, const CosSin& c, float& w00, float& w10, float& w01,
                                              float& w11) {
  const float xf = floorf(rr * c.ch), yf = floorf(rr * c.sh);
  const float fx = fmaf(rr, c.cl, fmaf(rr, c.ch, -xf));
  const float fy = fmaf(rr, c.sl, fmaf(rr, c.sh, -yf));
  const float gx = 1.f - fx, gy = 1.f - fy;
  w00 = gx * gy;
  w10 = fx * gy;
  w01 = gx * fy;
  w11 = fx * fy;
}
__device__ __forceinline__ float bilin4w(const float* img, int o4, int Lp4, float w00, float w10, float w01,
                                         float w11) {
  const char* p = reinterpret_cast<const char*>(img) + o4;
  const float i00 = *reinterpret_cast<const float*>(p), i10 = *reinterpret_cast<const float*>(p + 4);
  const float i01 = *reinterpret_cast<const float*>(p + Lp4), i11 = *reinterpret_cast<const float*>(p + Lp4 + 4);
  return fmaf(w11, i11, fmaf(w01, i01, fmaf(w10, i10, w00 * i00)));
}

__device__ __forceinline__ float bilin(const float* img, int o, int Lp, float fx, float fy) {
  const float i00 = img[o], i10 = img[o + 1], i01 = img[o + Lp], i11 = img[o + Lp + 1];
  const float top = i00 + fx * (i10 - i00);
  const float bot = i01 + fx * (i11 - i01);
  return top + fy * (bot - top);
}

// lane J's value of each group of 8 consecutive lanes, to all 8
// (ds_swizzle bit-mask mode: source lane = (lane & 0x18) | J within 32)
template <int J>
__device__ __forceinline__ int group_bcast(int v) {
  return __builtin_amdgcn_ds_swizzle(v, 0x18 | (J << 5));
}

// One ring at 8 shifts: the 32 bilinear samples v[i] = p[16 n1 + 2 l + e]
// (i = 2 n1 + e) of the lane's shift.  Lane (l, r) of the wave: group l of
// the FFT, shift r; o4 is the byte offset of that shift's centre pixel.
// Positions and weights do not depend on the shift: lane r of group l takes
// them for the angles i = r (mod 8), from the staged cos/sin (no memory
// loads), and samples those at all 8 shifts; a transpose through the wave's
// scratch `my` (64 x 9 float2), in two halves of 16 angles, hands each lane
// its own shift's samples.
__device__ __forceinline__ void sample_ring(const float* img, const CosSin* cs, float2* my, float rr, int l, int r,
                                            int o4, int Lp4, float (&v)[32]) {
  const CosSin* cp = cs + 2 * l;
  const int o4s[8] = {group_bcast<0>(o4), group_bcast<1>(o4), group_bcast<2>(o4), group_bcast<3>(o4),
                      group_bcast<4>(o4), group_bcast<5>(o4), group_bcast<6>(o4), group_bcast<7>(o4)};
  float* tr = reinterpret_cast<float*>(my);  // [64 (l, shift)][17]: row pitch 17 spreads the banks
#pragma unroll
  for (int hf = 0; hf < 2; ++hf) {
    float smp[2][8];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int i = 16 * hf + 8 * b + r;
      const CosSin c = cp[16 * (i >> 1) + (i & 1)];
      const int off = polar_offset(rr, c, Lp4);
      float w00, w10, w01, w11;
      polar_weights(rr, c, w00, w10, w01, w11);
#pragma unroll
      for (int j = 0; j < 8; ++j) smp[b][j] = bilin4w(img, o4s[j] + off, Lp4, w00, w10, w01, w11);
    }
    wave_sync();  // the scratch's earlier readers are done
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int j = 0; j < 8; ++j) tr[(l * 8 + j) * 17 + 8 * b + r] = smp[b][j];
    wave_sync();
#pragma unroll
    for (int q = 0; q < 16; ++q) v[16 * hf + q] = tr[(l * 8 + r) * 17 + q];
  }
  wave_sync();  // before the FFT's transposes reuse the scratch
}

// An angle's bilinear sample: the byte offset of its top-left tap from a
// shift's centre pixel, and its weights.
struct Tap {
  int off;
  float w00, w10, w01, w11;
  __device__ __forceinline__ void set(float rr, const CosSin& c, int Lp4) {
    off = polar_offset(rr, c, Lp4);
    polar_weights(rr, c, w00, w10, w01, w11);
  }
  __device__ __forceinline__ float operator()(float i00, float i10, float i01, float i11) const {
    return fmaf(w11, i11, fmaf(w01, i01, fmaf(w10, i10, w00 * i00)));
  }
};

// The taps of an angle at the rows (shifts) J0 .. J1 - 1 of 8, run K of the
// pattern, consecutive in an image row: the taps of one shift are the left
// taps of the next, so the run reads J1 - J0 + 1 columns instead of twice their
// number.  at: byte address of the first shift's top-left tap.
struct TapColumns {
  float t0[12], t1[12];  // run after run: upper and lower pixel row
  template <int J0, int J1, int K>
  __device__ __forceinline__ void read(const char* at, int Lp4) {
    const float* p0 = reinterpret_cast<const float*>(at);
    const float* p1 = reinterpret_cast<const float*>(at + Lp4);
#pragma unroll
    for (int i = 0; i <= J1 - J0; ++i) {
      t0[J0 + K + i] = p0[i];
      t1[J0 + K + i] = p1[i];
    }
  }
  // row j's sample goes to tr[17 j] (written here: handed back, the values
  // are copied where the patterns' branches meet)
  template <int J0, int J1, int K>
  __device__ __forceinline__ void sample(const Tap& tap, float* tr) const {
#pragma unroll
    for (int i = J0 + K; i < J1 + K; ++i) tr[17 * (i - K)] = tap(t0[i], t0[i + 1], t1[i], t1[i + 1]);
  }
};
// Two angles at 8 consecutive rows: they wrap to the next image row of the search
// grid after A rows and every S further ones.  at: byte address of each
// angle's top-left tap at shift offset 0; o[k] the offset of run k's first
// shift.  All taps are read before the first sample is written: the compiler
// does not move a read across a write to the same LDS (one angle's at a
// time: 1 % slower).
template <int A, int S>
__device__ __forceinline__ void sample_pattern(const char* const (&at)[2], const int (&o)[4], int Lp4,
                                               const Tap (&tap)[2], float* tr) {
  constexpr int e0 = A < 8 ? A : 8, e1 = A + S < 8 ? A + S : 8, e2 = A + 2 * S < 8 ? A + 2 * S : 8;
  static_assert(A + 3 * S >= 8, "at most four runs");
  TapColumns t[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    t[e].template read<0, e0, 0>(at[e] + o[0], Lp4);
    if constexpr (e0 < 8) t[e].template read<e0, e1, 1>(at[e] + o[1], Lp4);
    if constexpr (e1 < 8) t[e].template read<e1, e2, 2>(at[e] + o[2], Lp4);
    if constexpr (e2 < 8) t[e].template read<e2, 8, 3>(at[e] + o[3], Lp4);
  }
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    t[e].template sample<0, e0, 0>(tap[e], tr + 8 * e);
    if constexpr (e0 < 8) t[e].template sample<e0, e1, 1>(tap[e], tr + 8 * e);
    if constexpr (e1 < 8) t[e].template sample<e1, e2, 2>(tap[e], tr + 8 * e);
    if constexpr (e2 < 8) t[e].template sample<e2, 8, 3>(tap[e], tr + 8 * e);
  }
}

// As sample_ring for 8 consecutive rows s0 .. s0 + 7 of the search grid (s =
// sy S1 + sx; rows outside it take shifts of its first or last grid row and
// are not used), z[n1] = (p[16 n1 + 2 l], p[16 n1 + 2 l + 1]).  Lane r of group
// l takes the angles of n1 = 2 r + hf, both of the pair, in half hf: a wave's
// taps spread over the whole circle, which collides less in the banks than n1
// = r and 8 + r, half a circle each (76 px BF16: 9.41 against 9.60 ms).  base4: byte
// offset of the image centre.  What the resampler spends most LDS time on is
// the taps: with shared columns they are 40 to 48 two-word reads per ring and
// 8 rows, 64 without.  s0 and all but the lane indices are wave-uniform.
__device__ __forceinline__ void sample_runs(const float* img, const CosSin* cs, float2* my, float rr, int l, int r, int s0,
                                            int S1, int s1m, int T, int base4, int Lp4, float2 (&z)[16]) {
  const int sy0 = (((s0 + 8 * S1) * s1m) >> 16) - 8, sx0 = s0 - sy0 * S1, a = S1 - sx0;
  int o[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    int sy = sy0 + k;
    sy = sy < 0 ? 0 : (sy < S1 ? sy : S1 - 1);
    o[k] = base4 + (sy - T) * Lp4 + 4 * ((k == 0 ? sx0 : 0) - T);
  }
  // 8 S + A of sample_pattern; grids of more than 7 columns wrap as S = 7 does
  const int pattern = S1 == 1 ? 0 : (a >= 8 ? 64 : 8 * (S1 < 7 ? S1 : 7) + a);
  float* tr = reinterpret_cast<float*>(my);  // [64 (l, row)][17]: row pitch 17 spreads the banks
#pragma unroll
  for (int hf = 0; hf < 2; ++hf) {
    wave_sync();  // the scratch's earlier readers are done
    Tap tap[2];
    const char* at[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      tap[e].set(rr, cs[16 * (2 * r + hf) + 2 * l + e], Lp4);
      at[e] = reinterpret_cast<const char*>(img) + tap[e].off;
    }
    float* out = tr + l * 8 * 17 + r;
    auto take = [&](auto a_c, auto s_c) {
      sample_pattern<decltype(a_c)::value, decltype(s_c)::value>(at, o, Lp4, tap, out);
    };
    switch (pattern) {  // wave-uniform
      case 0:  // one shift: the particle's own row is one of the 8, all take its sample
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const float* p0 = reinterpret_cast<const float*>(at[e] + base4);
          const float* p1 = reinterpret_cast<const float*>(at[e] + base4 + Lp4);
          const float v = tap[e](p0[0], p0[1], p1[0], p1[1]);
#pragma unroll
          for (int j = 0; j < 8; ++j) out[17 * j + 8 * e] = v;
        }
        break;
      case 25: take(std::integral_constant<int, 1>{}, std::integral_constant<int, 3>{}); break;
      case 26: take(std::integral_constant<int, 2>{}, std::integral_constant<int, 3>{}); break;
      case 27: take(std::integral_constant<int, 3>{}, std::integral_constant<int, 3>{}); break;
      case 41: take(std::integral_constant<int, 1>{}, std::integral_constant<int, 5>{}); break;
      case 42: take(std::integral_constant<int, 2>{}, std::integral_constant<int, 5>{}); break;
      case 43: take(std::integral_constant<int, 3>{}, std::integral_constant<int, 5>{}); break;
      case 44: take(std::integral_constant<int, 4>{}, std::integral_constant<int, 5>{}); break;
      case 45: take(std::integral_constant<int, 5>{}, std::integral_constant<int, 5>{}); break;
      case 57: take(std::integral_constant<int, 1>{}, std::integral_constant<int, 7>{}); break;
      case 58: take(std::integral_constant<int, 2>{}, std::integral_constant<int, 7>{}); break;
      case 59: take(std::integral_constant<int, 3>{}, std::integral_constant<int, 7>{}); break;
      case 60: take(std::integral_constant<int, 4>{}, std::integral_constant<int, 7>{}); break;
      case 61: take(std::integral_constant<int, 5>{}, std::integral_constant<int, 7>{}); break;
      case 62: take(std::integral_constant<int, 6>{}, std::integral_constant<int, 7>{}); break;
      case 63: take(std::integral_constant<int, 7>{}, std::integral_constant<int, 7>{}); break;
      default: take(std::integral_constant<int, 8>{}, std::integral_constant<int, 8>{});
    }
    wave_sync();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const float* t = tr + (l * 8 + r) * 17 + q;
      z[2 * q + hf] = make_float2(t[0], t[8]);
    }
  }
  wave_sync();  // before the FFT's transposes reuse the scratch
}

// Ring FFT of the lane's samples: the two columns fwd_emit takes
// (k1a, k1b = fwd_cols(l)).
__device__ __forceinline__ void fft_ring(const CosSin* cs, float2* my, int l, int r, int k1a, int k1b, float2 (&z)[16],
                                         float2 (&Za)[8], float2 (&Zb)[8]) {
  dft16<-1>(z);
#pragma unroll
  for (int k1 = 1; k1 < 16; ++k1) z[k1] = cmul(z[k1], twid(cs, 2 * ((l * k1) & 127)));
  // transpose through the scratch in two halves: lane l's first column
  // k1a lies in 0..7, its second k1b in 8..15.  Entries are ordered
  // (l, shift) with the shift fastest, which spreads a wave's accesses
  // over the banks better than (shift, l).
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int k1 = 0; k1 < 8; ++k1) my[(l * 8 + r) * 9 + k1] = z[8 * h + k1];
    wave_sync();
#pragma unroll
    for (int n2 = 0; n2 < 8; ++n2) {
      if (h == 0) Za[n2] = my[(n2 * 8 + r) * 9 + k1a];
      else Zb[n2] = my[(n2 * 8 + r) * 9 + k1b - 8];
    }
    wave_sync();
  }
  dft8<-1>(Za);
  dft8<-1, false>(Zb);
}

// The lane's 16 spectrum values as operand entries (a - b, a + b).  Every
// real split yields one slot below 64 and one above (128 - f, or lane 0's 0
// and 64): both are kept, so that the 64 low and the 64 high slots can be
// staged one after the other.
struct RingSlots {
  int lo_s[8], hi_s[8];
  float lo_a[8], lo_b[8], hi_a[8], hi_b[8];
};
__device__ __forceinline__ void ring_slots(const CosSin* cs, int l, const float2 (&Za)[8], const float2 (&Zb)[8],
                                           RingSlots& o) {
  int e = 0, s0 = 0;
  float a0 = 0.f, b0 = 0.f;
  fwd_emit(l, Za, Zb, [&](int f) { return twid(cs, f & 255); },
           [&](int slot, float re, float im) {
             const int k = e >> 1;
             if ((e++ & 1) == 0) {
               s0 = slot; a0 = re - im; b0 = re + im;
             } else {
               const bool first_low = s0 < slot;
               o.lo_s[k] = first_low ? s0 : slot;
               o.hi_s[k] = first_low ? slot : s0;
               o.lo_a[k] = first_low ? a0 : re - im;
               o.lo_b[k] = first_low ? b0 : re + im;
               o.hi_a[k] = first_low ? re - im : a0;
               o.hi_b[k] = first_low ? re + im : b0;
             }
           });
}

// Operand element type written in mode 0: FP32 (kRingPerm or kSlotMajor,
// chosen at run time), or BF16 / FP16 in kRingPerm16.
enum PolarOut { kOutF32 = 0, kOutBF16 = 1, kOutFP16 = 2 };

// Two values in the contraction's 16-bit type, each rounded to nearest
// (even) once, packed with x in the low half.
template <int OUT>
__device__ __forceinline__ uint32_t pack16(float x, float y) {
  typedef float f32x2v __attribute__((ext_vector_type(2)));
  const f32x2v v = {x, y};
  if constexpr (OUT == kOutBF16) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
  } else {
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2));
  }
}

// The lane's spectrum values in the contraction's 16-bit type, (a - b) in the
// low half and (a + b) in the high half of a dword per slot; each value
// rounded once (FP16 scaled by the particle's power of two).
struct RingHalves {
  int lo_s[8], hi_s[8];
  uint32_t lo[8], hi[8];
};
template <int OUT>
__device__ __forceinline__ void ring_halves(const CosSin* cs, int l, const float2 (&Za)[8], const float2 (&Zb)[8],
                                            float scale, RingHalves& o) {
  int e = 0, s0 = 0;
  uint32_t v0 = 0;
  fwd_emit(l, Za, Zb, [&](int f) { return twid(cs, f & 255); },
           [&](int slot, float re, float im) {
             const int k = e >> 1;
             float a = re - im, b = re + im;
             if constexpr (OUT == kOutFP16) {
               a *= scale;
               b *= scale;
             }
             const uint32_t v = pack16<OUT>(a, b);
             if ((e++ & 1) == 0) {
               s0 = slot; v0 = v;
             } else {
               const bool first_low = s0 < slot;
               o.lo_s[k] = first_low ? s0 : slot;
               o.hi_s[k] = first_low ? slot : s0;
               o.lo[k] = first_low ? v0 : v;
               o.hi[k] = first_low ? v : v0;
             }
           });
}

// 16-bit operand (kRingPerm16): the low (h = 0) or high slots of one ring and 8
// rows, staged as [64 slots][8 rows] dwords (lanes write and read consecutive
// dwords).  The slots 64 h + w + 8 i are the run G = 2 w + h; lane (w, row)
// writes the two elements k = row and 8 + row of its 8 positions as one
// 16-byte store each, the 8 rows of a run together whole 128-byte lines.
__device__ __forceinline__ void write_half(uint32_t* stage, uint16_t* blk, int h, int w, int row, bool row_in,
                                           const RingHalves& o) {
#pragma unroll
  for (int k = 0; k < 8; ++k) stage[(h ? o.hi_s[k] - 64 : o.lo_s[k]) * 8 + row] = h ? o.hi[k] : o.lo[k];
  wave_sync();
  uint32_t x[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) x[i] = stage[(w + 8 * i) * 8 + row];
  uint32_t u[2][4];
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    u[0][d] = __builtin_amdgcn_perm(x[2 * d + 1], x[2 * d], 0x05040100u);
    u[1][d] = __builtin_amdgcn_perm(x[2 * d + 1], x[2 * d], 0x07060302u);
  }
  if (row_in) {
#pragma unroll
    for (int p = 0; p < 2; ++p)
      *reinterpret_cast<uint4*>(blk + a16_index(16 * w + 8 * h, 8 * p + row)) =
          make_uint4(u[p][0], u[p][1], u[p][2], u[p][3]);
  }
}

// Stages the low (h = 0) or high (h = 1) slots as [64 slots][16] floats
// (entry p * 8 + shift), the four 16-byte chunks of a slot XOR-swizzled by
// slot & 3, so the eight lanes l that write at once hit distinct banks.
__device__ __forceinline__ void stage_slots(float* stage, int h, int r, const RingSlots& o) {
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int sl = h ? o.hi_s[k] - 64 : o.lo_s[k];
    const int sw = (sl & 3) << 2;
    stage[sl * 16 + (r ^ sw)] = h ? o.hi_a[k] : o.lo_a[k];
    stage[sl * 16 + ((8 + r) ^ sw)] = h ? o.hi_b[k] : o.lo_b[k];
  }
}

// FP32 operand: writes one ring's staged slots of half h to the row tile
// block.  kRingPerm (perm): dst = the ring's [position][16] block; lane
// (pp = lane / 8, c = lane % 8) writes elements 2c, 2c+1 (rows rp, rp + 1) of
// the position pair 16 it + 4 h + lp, whose slots are 64 h + sp and
// 64 h + sp + 8, interleaved by element.  Otherwise slot s goes to dst + s ss,
// in 16-byte pieces: the lane's piece of slot 64 h + 16 it + lane / 4.  Only
// rows first <= row < last of the tile are written.
__device__ __forceinline__ void write_f32_half(const float* stage, float* dst, int h, int ln, bool perm, int ss,
                                               int first, int last) {
  const int part = ln & 3;                       // rows (part & 1) * 4 .. +3 of p = part >> 1
  const int r0 = (part & 1) * 4;
  const bool full = r0 >= first && r0 + 4 <= last;
  const int j = ln >> 2;
  float* const lane_dst = dst + (size_t)__mul24(j, ss) + part * 4;
  const int pp = ln >> 3, c = ln & 7;
  const int lp = 8 * (pp >> 2) + (pp & 3), sp = (pp >> 2) + 16 * (pp & 3);
  const int rp = 2 * (c & 3);
  const bool full_p = rp >= first && rp + 2 <= last;
  float* const pair_dst = dst + 32 * lp + 4 * c;
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    if (perm) {
      const int s0 = 2 * it + sp, s1 = s0 + 8, sw = (s0 & 3) << 2;  // s1 & 3 == s0 & 3
      const float2 v0 = *reinterpret_cast<const float2*>(stage + s0 * 16 + ((2 * c) ^ sw));
      const float2 v1 = *reinterpret_cast<const float2*>(stage + s1 * 16 + ((2 * c) ^ sw));
      float* o = pair_dst + 32 * (16 * it + 4 * h);
      if (full_p) {
        *reinterpret_cast<float4*>(o) = make_float4(v0.x, v1.x, v0.y, v1.y);
      } else {
        if (rp >= first && rp < last) { o[0] = v0.x; o[1] = v1.x; }
        if (rp + 1 >= first && rp + 1 < last) { o[2] = v0.y; o[3] = v1.y; }
      }
      continue;
    }
    const int sl = it * 16 + (ln >> 2);
    const float4 val = *reinterpret_cast<const float4*>(stage + sl * 16 + ((part ^ (sl & 3)) << 2));
    float* o = lane_dst + (size_t)(64 * h + 16 * it) * ss;
    if (full) {
      *reinterpret_cast<float4*>(o) = val;
    } else {
      if (r0 + 0 >= first && r0 + 0 < last) o[0] = val.x;
      if (r0 + 1 >= first && r0 + 1 < last) o[1] = val.y;
      if (r0 + 2 >= first && r0 + 2 < last) o[2] = val.z;
      if (r0 + 3 >= first && r0 + 3 < last) o[3] = val.w;
    }
  }
}

}  // namespace mra
