// Ring-weighted correlation of particle rows with references (Sec. 3:
// FFT(x)' x FFT(y) per ring, references on a second grid axis, inverse FFT of
// the CC table, arg-max by reduction as in Fig. 2): the matrix-core
// contraction of one 8-row x 8-reference tile, the inverse FFT over angle of
// its pairs, and the kernel k_corr that evaluates every pair of a launch (CC
// table, and alignment with pruning off).  The kernels that evaluate only the
// pairs that can win are in bound_impl.h and fine_impl.h.
//
// A row is particle * S + shift.  For each frequency slot f the matrix cores
// compute the 16 x 16 block
//     U[(p,row), (q,ref)] = sum_r A_f[(p,row), r] * B_f[r, (q,ref)],
//     A rows: p = 0 -> a - b, p = 1 -> a + b  (particle spectrum a + ib)
//     B cols: q = 0 -> c - d, q = 1 -> c + d  (reference spectrum c + id,
//             weighted by w_r, divided by the ring norm and by 256)
// whose four entries per (row, ref) are the spectrum H of the complex signal
// c0 + i c1 (unmirrored CC + i * mirrored CC) at f and 256 - f (see
// mra_fft.h).  The 128 slots of all 64 (row, ref) pairs sit in LDS (128 KiB);
// then a 16 x 16 inverse FFT over angle (two passes through LDS) yields the
// CC at all 256 angles for both mirrors.
//
// NW waves (8, or 4 in one FP32 variant): wave w owns slots w, w+NW, ... in
// the contraction.  In the resident variants the particle operand A of
// those slots is read once per row tile and kept in registers (FP32:
// R4 <= 9 with 8 waves, R4 <= 12 with 4 waves; packed 16-bit for the BF16 /
// FP16 forms) for all reference tiles; the streamed variants re-read it per
// reference tile.  The reference operand B is streamed from L2 with a slot
// prefetch.  Variants are tile configurations; they do not change any result.
#pragma once
#include <type_traits>

#include "mra_common.h"
#include "mra_fft.h"

namespace mra {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float2 w256c(const float2* cs, int e) {
  float2 c = cs[e & 255];
  return make_float2(c.x, -c.y);
}

__device__ __forceinline__ bool better(float v, int i, float bv, int bi) {
  return v > bv || (v == bv && i < bi);
}

template <int PREC>
struct Op16;
template <>
struct Op16<kBF16> {
  typedef bf16x8 T;
  static __device__ __forceinline__ uint16_t bits(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }
  static __device__ __forceinline__ f32x4 mfma(T a, T b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};
template <>
struct Op16<kFP16> {
  typedef f16x8 T;
  static __device__ __forceinline__ uint16_t bits(float x) { return __builtin_bit_cast(uint16_t, (_Float16)x); }
  static __device__ __forceinline__ f32x4 mfma(T a, T b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
};

// Order of the 16 x 16 matrix-core block.  Its rows are (row, p) and its
// columns (ref, q), interleaved: block row 2 row + p, block column 2 ref + q.
// The reference operand is packed in that column order; the particle
// operand is stored with position p * 8 + row, which block row j reads
// through a_block_pos(j).  Lane ln then holds column 2 ref + q = ln & 15 for the
// rows 2 (ln / 16) and 2 (ln / 16) + 1, both p: the four entries U_pq of a
// (row, ref) pair sit in two neighbouring lanes (q = 0, 1).
__device__ __forceinline__ int a_block_pos(int j) { return (j & 1) * 8 + (j >> 1); }
// The (row, ref) pair that lane ln gathers, as row * 8 + ref: row
// 2 (ln / 16) + q, ref (ln / 2) & 7, q = ln & 1.
__device__ __forceinline__ int lane_pair(int ln) { return (2 * (ln >> 4) + (ln & 1)) * 8 + ((ln >> 1) & 7); }

// Particle operand of lane ln for slot `slot` in the slot-major layout: ring
// g*R4 + t of lane group g = ln/16 at element 16 t (kRingPerm is read two slots at a
// time with a_pair).  Rings >= R are padding that the polar kernel never writes:
// callers mask them.
__device__ __forceinline__ const float* a_lane(const CorrArgs& a, int tile, int slot, int ln) {
  return a.A + (size_t)(tile * kSlots + slot) * 64 * a.R4 + ((ln >> 4) * a.R4) * 16 + a_block_pos(ln & 15);
}
// Element t of the lane's operand: ring (ln/16)*R4 + t.  The load is never
// conditional (a conditional load waits for its data before the next one is
// issued): its element index is clamped into the slot's block, and elements
// t >= R4 and padding rings >= R (which hold no data) are cleared by an AND
// with a mask that is opaque to the optimiser, which would otherwise turn
// the select back into a branch around the load.
__device__ __forceinline__ float a_elem(const CorrArgs& a, const float* ap, int ln, int t, bool nt) {
  const int tt = t < a.R4 ? t : a.R4 - 1;
  const float x = nt ? __builtin_nontemporal_load(ap + 16 * tt) : ap[16 * tt];
  uint32_t keep = (t < a.R4 && (ln >> 4) * a.R4 + t < a.R) ? 0xffffffffu : 0u;
  asm("" : "+v"(keep));
  return __uint_as_float(__float_as_uint(x) & keep);
}

// Elements t of two slots at once in the permuted layout (kRingPerm): ap
// points at element 0 of the lane's pair block; masks as in a_elem.
typedef float f32x2 __attribute__((ext_vector_type(2)));
template <int RX = 0>
__device__ __forceinline__ f32x2 a_pair(const CorrArgs& a, const float* ap, int ln, int t) {
  const int R4 = RX > 0 ? RX : a.R4;
  const int tt = t < R4 ? t : R4 - 1;
  const f32x2 x = __builtin_nontemporal_load(reinterpret_cast<const f32x2*>(ap + tt * kSlots * 16));
  uint32_t keep = (t < R4 && (ln >> 4) * R4 + t < a.R) ? 0xffffffffu : 0u;
  asm("" : "+v"(keep));
  f32x2 r;
  r.x = __uint_as_float(__float_as_uint(x.x) & keep);
  r.y = __uint_as_float(__float_as_uint(x.y) & keep);
  return r;
}

// FP32 reference operand of reference k and slot `slot`: the lane's R4
// elements (ring group ln / 16, q = ln & 1) are contiguous.
template <int RX = 0>
__device__ __forceinline__ const float* b32_lane(const CorrArgs& a, int k, int slot, int ln) {
  return a.B32 + ((size_t)(k * kSlots + slot) * 8 + (ln >> 4) * 2 + (ln & 1)) * b32_pitch(RX > 0 ? RX : a.R4);
}
// 16-bit reference operand: place of the lane's elements (reference r of
// the tile, ring group ln / 16, q = ln & 1) in each step of a slot's block.
__device__ __forceinline__ int b16_lane(int r, int ln) { return (ln & 0x30) + 2 * r + (ln & 1); }

// swap the values of neighbouring lanes (DPP quad_perm [1, 0, 3, 2]; every
// lane is enabled, so no old value is needed)
__device__ __forceinline__ float swap_adjacent(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xb1, 0xf, 0xf, false));
}

// Block of one slot -> the lane's pair (lane_pair(ln)): the four entries U_pq
// gathered with one exchange between the two lanes of the pair, as the state
// halves (U00, U01) and (U11, U10).
__device__ __forceinline__ void pair_gather(int ln, const f32x4& acc, float2& h0, float2& h1) {
  const bool q = ln & 1;
  // lane q = 0 holds (row 2g: U00, U10; row 2g + 1: U00, U10), lane q = 1
  // the same rows' U01, U11; each sends the entries of the other's row
  const float r0 = swap_adjacent(q ? acc[0] : acc[2]), r1 = swap_adjacent(q ? acc[1] : acc[3]);
  h0 = make_float2(q ? r0 : acc[0], q ? acc[2] : r0);
  h1 = make_float2(q ? acc[3] : r1, q ? r1 : acc[1]);
}
__device__ __forceinline__ void pair_block(float2* stc, int slot, int ln, int P, f32x4 acc) {
  float2 h0, h1;
  pair_gather(ln, acc, h0, h1);
  stc[(slot * 2) * 64 + P] = h0;
  stc[(slot * 2 + 1) * 64 + P] = h1;
}

// Contraction of one reference tile with FP32 operands for the wave's
// 128/NW slots (slot = w + NW*i).  EXACT: R4 == MAXR, else R4 <= MAXR at
// run time (mixed ring counts in one batched launch).  RES: the
// particle operand of all the wave's slots is loaded once per row tile and
// kept in registers for every reference tile; otherwise it is streamed with
// the reference operand.  Operands of the next two slots are prefetched.
template <int NW, int MAXR, bool RES, bool EXACT>
struct Fp32Contract {
  static constexpr int SPW = kSlots / NW;
  static constexpr int RX = EXACT ? MAXR : 0;
  static constexpr int LAYOUT = (NW == 8 && RES) ? kRingPerm : kSlotMajor;
  float areg[RES ? SPW : 1][RES ? MAXR : 1];

  // the lane's reference operand of slot `slot` in reference tile kt, in
  // 16-byte loads (with one load per element and none before the particle
  // operand's, a launch of one tile pair per CU took 50 us instead of 29)
  __device__ __forceinline__ void load_b(const CorrArgs& a, int kt, int slot, int ln, float (&dst)[MAXR]) const {
    const float* bp = b32_lane<RX>(a, kt * kRefTile + ((ln >> 1) & 7), slot, ln);
    const int last = b32_pitch(RX > 0 ? RX : a.R4) / 4 - 1;
#pragma unroll
    for (int q = 0; q < (MAXR + 3) / 4; ++q) {  // unconditional, whole quads (elements t >= R4 are not used)
      const f32x4 v = *reinterpret_cast<const f32x4*>(bp + 4 * (q < last ? q : last));
#pragma unroll
      for (int t = 4 * q; t < 4 * q + 4; ++t)
        if (t < MAXR) dst[t] = v[t & 3];
    }
  }
  // PRE (8 waves, resident operand): the reference
  // operand of the wave's first slot of reference tile kt is loaded before
  // the inverse FFT of the previous tile, so its latency passes under it
  // (one slot: the registers of two would spill in these forms)
  static constexpr bool PRE = RES && NW == 8;
  float bpre[PRE ? MAXR : 1];
  __device__ __forceinline__ void prefetch(const CorrArgs& a, int kt, int w, int ln) {
    if constexpr (PRE) load_b(a, kt, w, ln, bpre);
  }

  __device__ __forceinline__ void load_a(const CorrArgs& a, int tile, int /*k*/, int w, int ln) {
    if constexpr (RES) {
      if constexpr (LAYOUT == kRingPerm) {
        // the wave's slots w + 8 i sit at positions 16 w + i, in pairs
        // (i even, i + 1) interleaved by element: one base address, constant
        // offsets, one 8-byte load for two slots
        const int R4 = RX > 0 ? RX : a.R4;
        const float* a0 = a.A + ((size_t)(tile * 4 + (ln >> 4)) * R4 * kSlots + 16 * w) * 16 + 2 * a_block_pos(ln & 15);
#pragma unroll
        for (int i2 = 0; i2 < SPW / 2; ++i2) {
#pragma unroll
          for (int t = 0; t < MAXR; ++t) {
            const f32x2 v = a_pair<RX>(a, a0 + 32 * i2, ln, t);
            areg[2 * i2][t] = v.x;
            areg[2 * i2 + 1][t] = v.y;
          }
        }
      } else {
#pragma unroll
        for (int i = 0; i < SPW; ++i) {
          const float* ap = a_lane(a, tile, w + NW * i, ln);
#pragma unroll
          for (int t = 0; t < MAXR; ++t) areg[i][t] = a_elem(a, ap, ln, t, true);
        }
      }
    }
  }

  __device__ __forceinline__ void run(const CorrArgs& a, float2* stc, int tile, int kt, int w, int ln) {
    const int R4 = EXACT ? MAXR : a.R4;
    const int P = lane_pair(ln);
    auto loadb = [&](int i, float (&dst)[MAXR]) { load_b(a, kt, w + NW * i, ln, dst); };
    if constexpr (RES) {
      // slots in pairs: two independent accumulation chains keep the matrix
      // pipe busy; the reference operand of the next pair is in flight
      float b[4][MAXR];
      if constexpr (PRE) {
#pragma unroll
        for (int t = 0; t < MAXR; ++t) b[0][t] = bpre[t];
      } else {
        loadb(0, b[0]);
      }
      loadb(1, b[1]);
#pragma unroll
      for (int i = 0; i < SPW; i += 2) {
        f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < MAXR; ++t) {
          if (t < R4) {
            acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(areg[i][t], b[i % 4][t], acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(areg[i + 1][t], b[(i + 1) % 4][t], acc1, 0, 0, 0);
          }
        }
        if (i + 2 < SPW) loadb(i + 2, b[(i + 2) % 4]);
        if (i + 3 < SPW) loadb(i + 3, b[(i + 3) % 4]);
        pair_block(stc, w + NW * i, ln, P, acc0);
        pair_block(stc, w + NW * (i + 1), ln, P, acc1);
      }
    } else {
      // both operands streamed, one slot ahead (explicit double buffer so
      // that the slot loop need not be unrolled)
      float b0[MAXR], a0[MAXR], b1[MAXR], a1[MAXR];
      auto loada = [&](int i, float (&dst)[MAXR]) {
        const float* ap = a_lane(a, tile, w + NW * i, ln);
#pragma unroll
        for (int t = 0; t < MAXR; ++t) dst[t] = a_elem(a, ap, ln, t, false);
      };
      auto chain = [&](const float (&x)[MAXR], const float (&y)[MAXR], int slot) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < MAXR; ++t)
          if (t < R4) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[t], y[t], acc, 0, 0, 0);
        pair_block(stc, slot, ln, P, acc);
      };
      loadb(0, b0);
      loada(0, a0);
#pragma unroll 1
      for (int i = 0; i < SPW; i += 2) {
        loadb(i + 1, b1);
        loada(i + 1, a1);
        chain(a0, b0, w + NW * i);
        if (i + 2 < SPW) {
          loadb(i + 2, b0);
          loada(i + 2, a0);
        }
        chain(a1, b1, w + NW * (i + 1));
      }
    }
  }
};

// Contraction with 16-bit operands; NS = ceil(MAXR / 8) <= 2 steps of 8
// rings per lane group.  MAXR is the ring bucket of R4 (8: 1..8, 10: 9..10, 12:
// 11..12, 16: 13..16), which fixes the step count and the width of the last
// step: with MAXR = 10 or 12 it holds at most 2 or 4 rings per lane group
// (NARROW), and the particle operand keeps 1 or 2 dwords of it per slot (TD)
// instead of 4.  The particle operand arrives rounded to the contraction's type
// (FP16 already scaled per particle) in the 16-bit ring-major layout.  RES: it
// is read once per row tile and kept packed in registers, two values per
// dword; otherwise it is re-read per reference tile, one slot ahead.  The
// reference operand's last step is stored as wide as its rings need
// (b16_tail_width: 2 TD elements, 8 where it is not narrow).
template <int PREC, int NW, int MAXR, bool RES>
struct Half16Contract {
  static constexpr int SPW = kSlots / NW;
  static constexpr int NS = (MAXR + 7) / 8;
  static_assert(NS <= 2, "at most two steps of 8 rings per lane group");
  static constexpr bool NARROW = NS == 2 && MAXR - 8 <= 4;
  static constexpr int NF = NARROW ? 1 : NS;  // steps held 8 wide
  static constexpr int TD = NARROW ? (MAXR - 8 + 1) / 2 : 0;  // dwords of the narrow step
  typedef typename Op16<PREC>::T V;
  // one slot's operand of the lane: the steps held 8 wide, then (NARROW) the
  // last step's elements (t[1] only with TD = 2)
  struct Frag {
    u32x4 f[NF];
    u32x2 t;
  };
  Frag areg[RES ? SPW : 1];
  Frag bpre;                     // RES: reference operand of the wave's first slot, loaded ahead

  // Element t (ring (ln/16) R4 + t) of the lane's row for each t < MAXR is
  // read unconditionally, its index clamped into the row tile's rings: an
  // element t >= R4 repeats the last one, and padding rings >= R hold zeros;
  // the reference operand is zero at both.
  __device__ __forceinline__ const uint16_t* ring_block(const CorrArgs& a, int tile, int t, int ln) const {
    const int tt = t < a.R4 ? t : a.R4 - 1;
    return reinterpret_cast<const uint16_t*>(a.A) + ((size_t)(tile * 4 + (ln >> 4)) * a.R4 + tt) * kSlots * 16;
  }
  // Two 16-bit values as the contraction's dword: x's and y's element j of
  // their 8 (v_perm byte selection)
  static __device__ __forceinline__ uint32_t pick2(uint32_t x, uint32_t y, int odd) {
    return __builtin_amdgcn_perm(y, x, odd ? 0x07060302u : 0x05040100u);
  }

  // The lane's operand of slot `slot` (streamed variant): one 2-byte load
  // per element.
  __device__ __forceinline__ void fetch(const CorrArgs& a, int tile, int slot, int ln, Frag& dst, bool nt) {
    const int idx = a16_index(slot_pos(slot), a_block_pos(ln & 15));
    uint32_t v[8 * NS];
#pragma unroll
    for (int t = 0; t < 8 * NS; ++t) {
      if (t < MAXR) {
        const uint16_t* bp = ring_block(a, tile, t, ln) + idx;
        v[t] = nt ? (uint32_t)__builtin_nontemporal_load(bp) : (uint32_t)*bp;
      } else {
        v[t] = 0u;
      }
    }
#pragma unroll
    for (int d = 0; d < 4 * NF; ++d) dst.f[d / 4][d % 4] = v[2 * d] | (v[2 * d + 1] << 16);
    if constexpr (NARROW) {
#pragma unroll
      for (int d = 0; d < TD; ++d) dst.t[d] = v[8 + 2 * d] | (v[9 + 2 * d] << 16);
    }
  }

  // The operand of all the wave's slots w + 8 i, of the lane's block row:
  // element k (p * 8 + row % 8) of row tile `tile` (either may differ by lane).
  // Per element t, one 16-byte load of the interleaved run 2 w + hh gives
  // slots i = 8 hh .. 8 hh + 7; dword regroups them per slot: dword d (elements
  // t = 2 d, 2 d + 1) of slot 8 hh + j.
  __device__ __forceinline__ void load_run(const CorrArgs& a, int tile, int k, int w, int ln, int hh,
                                           u32x4 (&u)[8 * NS]) const {
    static_assert(NW == 8, "the interleaved runs hold 8 slots of each of 8 waves");
#pragma unroll
    for (int t = 0; t < 8 * NS; ++t) {
      if (t < MAXR) {
        const u32x4* bp = reinterpret_cast<const u32x4*>(ring_block(a, tile, t, ln) + a16_index(16 * w + 8 * hh, k));
        u[t] = __builtin_nontemporal_load(bp);
      } else {
        u[t] = u32x4{0u, 0u, 0u, 0u};
      }
    }
  }
  static __device__ __forceinline__ uint32_t dword(const u32x4 (&u)[8 * NS], int j, int d) {
    return pick2(u[2 * d][j >> 1], u[2 * d + 1][j >> 1], j & 1);
  }
  // put(i, d, x) takes dword d of slot i
  template <class Put>
  __device__ __forceinline__ void read_a(const CorrArgs& a, int tile, int k, int w, int ln, Put put) const {
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      u32x4 u[8 * NS];
      load_run(a, tile, k, w, ln, hh, u);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
#pragma unroll
        for (int d = 0; d < 4 * NF + TD; ++d) put(8 * hh + j, d, dword(u, j, d));
      }
    }
  }
  __device__ __forceinline__ void load_a(const CorrArgs& a, int tile, int k, int w, int ln) {
    if constexpr (RES)
      read_a(a, tile, k, w, ln, [&](int i, int d, uint32_t x) {
        if (d < 4 * NF) areg[i].f[d / 4][d % 4] = x;
        else areg[i].t[d - 4 * NF] = x;
      });
  }

  // the lane's reference operand of slot `slot` in reference tile kt (elements
  // t >= R4 are stored as zeros)
  static constexpr int BT = NARROW ? 2 * TD : 8;         // last step: elements per lane
  static constexpr int SE = (NS - 1) * 512 + 64 * BT;    // elements per slot block
  __device__ __forceinline__ void load_b(const CorrArgs& a, int kt, int slot, int ln, Frag& dst) const {
    load_b_at(a, kt, slot, ln, 0, dst);
  }
  // the same from the place pl (b16_lane) of a tile kt, `tile_off` elements
  // further (per lane: any reference)
  __device__ __forceinline__ void load_b_at(const CorrArgs& a, int kt, int slot, int pl, size_t tile_off,
                                            Frag& dst) const {
    const uint16_t* bp = a.B16 + (size_t)(kt * kSlots + slot) * SE;
    dst.f[0] = *reinterpret_cast<const u32x4*>(bp + (tile_off + pl * 8));
    if constexpr (NS == 2) {
      const uint16_t* tp = bp + 512 + (tile_off + pl * BT);
      if constexpr (!NARROW) dst.f[1] = *reinterpret_cast<const u32x4*>(tp);
      else if constexpr (TD == 2) dst.t = *reinterpret_cast<const u32x2*>(tp);
      else dst.t[0] = *reinterpret_cast<const uint32_t*>(tp);
    }
  }
  // RES: start loading the first slot of reference tile kt, which the next
  // run() uses (its latency then passes during the inverse FFT)
  __device__ __forceinline__ void prefetch(const CorrArgs& a, int kt, int w, int ln) {
    if constexpr (RES) load_b(a, kt, w, ln, bpre);
  }

  // one slot's block: operand x of the particle rows, y of the references
  __device__ __forceinline__ f32x4 product(const Frag& x, const Frag& y) const {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NF; ++s)
      acc = Op16<PREC>::mfma(__builtin_bit_cast(V, x.f[s]), __builtin_bit_cast(V, y.f[s]), acc);
    if constexpr (NARROW) {
      // the last step is a K = 32 product with the other elements zero: a K = 16
      // product accumulated straight onto the K = 32 one's result gave
      // wrong sums on gfx950 when the two issued back to back
      const u32x4 xa = {x.t[0], TD > 1 ? x.t[1] : 0u, 0u, 0u}, yb = {y.t[0], TD > 1 ? y.t[1] : 0u, 0u, 0u};
      acc = Op16<PREC>::mfma(__builtin_bit_cast(V, xa), __builtin_bit_cast(V, yb), acc);
    }
    return acc;
  }

  __device__ __forceinline__ void run(const CorrArgs& a, float2* stc, int tile, int kt, int w, int ln) {
    const int P = lane_pair(ln);
    auto loadb = [&](int i, Frag& dst) { load_b(a, kt, w + NW * i, ln, dst); };
    auto chain = [&](const Frag& x, const Frag& y, int slot) { pair_block(stc, slot, ln, P, product(x, y)); };
    if constexpr (RES) {
      Frag b[2];
      b[0] = bpre;
#pragma unroll
      for (int i = 0; i < SPW; ++i) {
        if (i + 1 < SPW) loadb(i + 1, b[(i + 1) % 2]);
        chain(areg[RES ? i : 0], b[i % 2], w + NW * i);
        // keep each slot's store next to its products (a schedule that
        // defers them all holds 16 blocks of results and runs slower)
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      // explicit double buffer so that the slot loop need not be unrolled
      Frag b0, b1, x0, x1;
      loadb(0, b0);
      fetch(a, tile, w, ln, x0, false);
#pragma unroll 1
      for (int i = 0; i < SPW; i += 2) {
        loadb(i + 1, b1);
        fetch(a, tile, w + NW * (i + 1), ln, x1, false);
        chain(x0, b0, w + NW * i);
        if (i + 2 < SPW) {
          loadb(i + 2, b0);
          fetch(a, tile, w + NW * (i + 2), ln, x0, false);
        }
        chain(x1, b1, w + NW * (i + 1));
      }
    }
  }
};

__device__ __forceinline__ void lds_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A candidate (CC value v, flat index iota < 2^31 - 1) as one 64-bit key whose
// unsigned order is the arg-max order: larger v first, then smaller iota.  0
// is below every candidate.
__device__ __forceinline__ unsigned long long cand_key(float v, int iota) {
  const uint32_t u = __float_as_uint(v == 0.f ? 0.f : v);  // -0 ties with +0, as in the float order
  const uint32_t o = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ((unsigned long long)o << 32) | (unsigned long long)(0x7fffffffu - (uint32_t)iota);
}
__device__ __forceinline__ float key_value(unsigned long long k) {
  if (k == 0ull) return -INFINITY;
  const uint32_t o = (uint32_t)(k >> 32);
  return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}
__device__ __forceinline__ int key_index(unsigned long long k) {
  return k == 0ull ? 0x7fffffff : (int)(0x7fffffffu - (uint32_t)k);
}

// What rounding both operands to FP16 can add to a pair's CC (see
// bound_impl.h), in their scaled units: sa = norm of the row's rounded operand,
// nb = norm of the reference's (scaled) operand, R rings.
__device__ __forceinline__ float fp16_error(float sa, float nb, int R) {
  const float u = 1.f / 2048.f, eta = sqrtf(2.f * kSlots * R) / 16384.f;
  const float Na = (sa + eta) * (1.f + 1.f / 1024.f), Da = u * Na + eta, Db = u * nb + eta;
  return 1.41421363f * (1.f + 1.f / 64.f) * (Da * nb + Na * Db + Da * Db);
}

// Tightens the bound of a pair of particle n (FP32 alignment) by the best CC of its
// FP16 operands, which is within fp16_error of the FP32 one's, and within its own
// rounding (2^-12 of the bound).  Returns a value that the FP32 one reaches,
// or -inf.
__device__ __forceinline__ float tighten_pair(const CorrArgs& c, int n, int row, int k, float cc) {
  float* u = c.ub + (size_t)row * c.ldu + k;
  const float err = fp16_error(c.rownorm[row], c.bnorm[k] * c.b_scale, c.R) + 1e-16f;
  const float own = *u * (1.f / 4096.f), mx = c.maxabs[n];
  const float hi = fp16_value(cc + err, mx, c.b_scale) + own + 1e-37f;
  const float lo = fp16_value(cc - err, mx, c.b_scale) - own - 1e-37f;
  if (hi < *u) *u = hi;
  return lo > -INFINITY && lo < INFINITY ? lo : -INFINITY;
}
// The largest CC of a lane's 16 angles and both mirrors as ordered bits, any NaN as
// infinite.
__device__ __forceinline__ uint32_t largest_cc(const float2 (&x)[16], int M) {
  float mx = -INFINITY;
  bool nan = false;
#pragma unroll
  for (int n2 = 0; n2 < 16; ++n2) {
    mx = fmaxf(mx, M == 2 ? fmaxf(x[n2].x, x[n2].y) : x[n2].x);
    nan |= !(x[n2].x == x[n2].x) || !(x[n2].y == x[n2].y);
  }
  return (uint32_t)(cand_key(nan ? INFINITY : mx, 0) >> 32);
}

// What a tile computes: the per-row arg-max, the full CC table (debug),
// the arg-max with one candidate per particle left out (the runner-up pass), or
// the tightening of its pairs' bounds, with a value that each row's FP32 best reaches.
constexpr int kArgmax = 0, kTable = 1, kRunnerUp = 2, kTighten = 3;

constexpr size_t kStateFloats = (size_t)kSlots * 2 * 64 * 2;  // spectra of the 64 (row, ref) pairs

// The inverse FFT over angle of n_live pairs whose spectra the contraction
// left in the state stc ([128 slots][2 halves][PS]; n_live the same in every
// wave): done(i, n1, x) is called by one lane per (pair i, n1 < 16) with the
// complex CC x[n2] (unmirrored + i mirrored) at the angles n1 + 16 n2.  With
// PS = 64 pair i's entries are at list[i], otherwise at i.  Contains a workgroup
// barrier; the caller has one between the contraction and this, and one
// before the state is written again.
//
// With CPWX columns (pass 1) and rows (pass 2) per wave, the working waves'
// columns / rows are CPWX * w + c, c = 0 .. CPWX-1: lane group c (LPCX lanes)
// takes column / row c for the live pairs list[n0 + ln % LPCX].  The first
// waves hold rows below 8 and the others rows from 8 on, so that every wave's
// pass-2 addresses share one shape (a lane base plus constant offsets).  At
// most 16 live pairs fit 4 columns of 16 lanes per wave: then waves 0..3 (one
// per SIMD) do the passes and the others wait at the barrier, so each SIMD
// issues one wave's instructions instead of two.
template <int NW, bool SPLIT, int PS, class Done>
__device__ __forceinline__ void inverse_pairs(float2* stc, const float2* tw, const int* list, int n_live, int w, int ln,
                                              Done done) {
  auto passes = [&](auto cpw_c) {
    constexpr int CPWX = decltype(cpw_c)::value, LPCX = 64 / CPWX;
    const bool work = CPWX * w < 16;  // wave-uniform

    // ---------------- inverse FFT over angle, pass 1 ----------------
    // H_j (j = 16 k1 + k2) of pair P: half 0 of slot j (j < 128) or half 1
    // of slot 256 - j (j >= 128; slot 0 for j = 128)
    if (work) {
#pragma unroll 1
      for (int n0 = 0; n0 < n_live; n0 += LPCX) {
        // lane-derived values are recomputed here rather than kept live
        // across the caller's loop, where the registers hold the operand
        int lnx = ln;
        asm volatile("" : "+v"(lnx));
        const int lane_n = lnx % LPCX, k2 = CPWX * w + lnx / LPCX;
        const bool act = n0 + lane_n < n_live;
        const int A = PS == 64 ? list[act ? n0 + lane_n : 0] : (act ? n0 + lane_n : 0);
        const int lo = k2 * 2 * PS + A, hi = A - k2 * 2 * PS;
        const int mid = k2 == 0 ? PS + A : hi + 257 * PS;
        auto at = [&](int k1) { return k1 < 8 ? lo + k1 * 32 * PS : (k1 == 8 ? mid : hi + (513 - 32 * k1) * PS); };
        float2 x[16];
#pragma unroll
        for (int k1 = 0; k1 < 16; ++k1) x[k1] = stc[at(k1)];
        inv_pass1(k2, x, [&](int e) { return tw[e & 255]; });
        if (act) {
#pragma unroll
          for (int n1 = 0; n1 < 16; ++n1) stc[at(n1)] = x[n1];
        }
      }
    }
    __syncthreads();

    // ---------------- pass 2 ----------------
    // Rows below 8 read upwards from slot 16 n1, the others downwards from
    // slot 256 - 16 n1.  SPLIT: one loop per direction (each wave runs one),
    // so that either keeps its 16 reads at constant offsets from one address
    // (in one loop the compiler merges the two read sets into 31 per-element
    // addresses); the 4-wave kernels, whose registers are full, keep one loop.
    auto pass2 = [&](auto dir_c) {
      constexpr int dir = decltype(dir_c)::value;  // 1 up, 2 down, 0 either (chosen per wave)
#pragma unroll 1
      for (int n0 = 0; n0 < n_live; n0 += LPCX) {
        int lnx = ln;
        asm volatile("" : "+v"(lnx));
        const int lane_n = lnx % LPCX, c = lnx / LPCX, n1 = CPWX * w + c;
        const bool act = n0 + lane_n < n_live;
        const int i = act ? n0 + lane_n : 0, A = PS == 64 ? list[i] : i;
        float2 x[16];
        const bool low = dir == 1 || (dir == 0 && CPWX * w < 8);
        if (low) {
          const int base = n1 * 32 * PS + A;
#pragma unroll
          for (int k2 = 0; k2 < 16; ++k2) x[k2] = stc[base + k2 * 2 * PS];
        } else if constexpr (dir == 2) {
          const int base = (513 - 32 * n1) * PS + A;  // k2 = 0; k2 steps go down by 2 PS
          int top = base - 15 * 2 * PS;               // k2 = 15, the lowest address
          asm volatile("" : "+v"(top));               // the base of the reads (not re-associated)
          x[0] = stc[n1 == 8 ? PS + A : base];
#pragma unroll
          for (int k2 = 1; k2 < 16; ++k2) x[k2] = stc[top + (15 - k2) * 2 * PS];
        } else {
          const int base = (513 - 32 * n1) * PS + A;
          x[0] = stc[n1 == 8 ? PS + A : base];
#pragma unroll
          for (int k2 = 1; k2 < 16; ++k2) x[k2] = stc[base - k2 * 2 * PS];
        }
        inv_pass2(x);
        if (act) done(i, n1, x);
      }
    };
    if (work) {
      if constexpr (SPLIT) {
        if (CPWX * w < 8) pass2(std::integral_constant<int, 1>{});  // wave-uniform
        else pass2(std::integral_constant<int, 2>{});
      } else {
        pass2(std::integral_constant<int, 0>{});
      }
    }
  };
  if constexpr (NW == 8) {
    if (n_live <= 16) passes(std::integral_constant<int, 4>{});  // workgroup-uniform
    else passes(std::integral_constant<int, 2>{});
  } else {
    passes(std::integral_constant<int, 16 / NW>{});
  }
}

// The best of a lane's 16 angles n1 + 16 n2 and both mirrors (mirror search),
// if it reaches thr: its value in bv and m * 256 + angle in bi (the smallest
// of those equal to it), else bi = 2^31 - 1.  ex: the candidate left out
// (runner-up pass), or -1.  -inf and NaN are never candidates.
template <int MODE>
__device__ __forceinline__ void pick_best(const float2 (&x)[16], int n1, int M, float thr, int ex, float& bv, int& bi) {
  bv = -INFINITY;
  bi = 0x7fffffff;
  float mx = -INFINITY;
#pragma unroll
  for (int n2 = 0; n2 < 16; ++n2) mx = fmaxf(mx, M == 2 ? fmaxf(x[n2].x, x[n2].y) : x[n2].x);
  if (!(mx >= thr) || mx == -INFINITY) return;
  if (MODE == kArgmax) {
    // the lane's best is mx; its key is the smallest among the candidates
    // equal to it (keys grow with n2, mirror 1 after 0)
    bv = mx;
    if (M == 2) {
#pragma unroll
      for (int n2 = 15; n2 >= 0; --n2) bi = x[n2].y == mx ? 256 + n1 + 16 * n2 : bi;
    }
#pragma unroll
    for (int n2 = 15; n2 >= 0; --n2) bi = x[n2].x == mx ? n1 + 16 * n2 : bi;
  } else {
#pragma unroll
    for (int n2 = 0; n2 < 16; ++n2) {
      const int ang = n1 + 16 * n2;
      if (ang != ex && better(x[n2].x, ang, bv, bi)) { bv = x[n2].x; bi = ang; }
      if (M == 2 && 256 + ang != ex && better(x[n2].y, 256 + ang, bv, bi)) {
        bv = x[n2].y;
        bi = 256 + ang;
      }
    }
    if (!(bv >= thr) || bv == -INFINITY) bi = 0x7fffffff;
  }
}

// The candidate m * 256 + angle left out of (reference k, shift s) when the
// flat index e (or -1) lies in that pair, else -1.
__device__ __forceinline__ int excluded_at(int e, int k, int s, int S, int M) {
  if (e < 0) return -1;
  const int rest = e >> 8, se = rest % S, km = rest / S;
  return (se == s && km / M == k) ? (km % M) * 256 + (e & 255) : -1;
}

// Particle n's outputs from its best CC and flat index (2^31 - 1: none).
__device__ __forceinline__ void write_result(const ResultArgs& a, int n, float best, int bi) {
  const int64_t o = a.out_off + n;
  if (!(best == best)) bi = 0x7fffffff;  // (FP16: the particle does not scale into it)
  if (a.runner_up) {  // second pass: the best over every candidate but the winner
    a.cc2[o] = bi == 0x7fffffff ? NAN : best;
    return;
  }
  if (a.win) a.win[n] = bi == 0x7fffffff ? -1 : bi;
  if (bi == 0x7fffffff) {  // no ordered candidate (NaN input): report an invalid winner
    a.ref[o] = -1;
    a.mirror[o] = 0;
    a.shift_x[o] = 0;
    a.shift_y[o] = 0;
    a.psi[o] = 0;
    a.cc[o] = NAN;
    if (a.flat) a.flat[o] = -1;
    if (a.cc2) a.cc2[o] = NAN;
    return;
  }
  const int ang = bi & 255;
  int rest = bi >> 8;
  const int s = rest % a.S;
  rest /= a.S;
  const int m = rest % a.M, k = rest / a.M;
  a.ref[o] = k;
  a.mirror[o] = m;
  a.shift_x[o] = s % a.S1 - a.T;
  a.shift_y[o] = s / a.S1 - a.T;
  a.psi[o] = (kNphi - ang) & 255;
  a.cc[o] = best;
  if (a.flat) a.flat[o] = bi;
  if (a.cc2) a.cc2[o] = NAN;
}

template <int NW>
struct CorrSmem {
  float2* stc;              // [128][2][64] spectra of the 64 (row, ref) pairs
  unsigned long long* key;  // [8] best candidate of each row so far (ordered key, 0 = none)
  int* list;                // [NW][64] each wave's list of the pairs of the inverse FFT
  float2* tw;               // exp(-2 pi i e / 256)
  uint32_t* pmax;           // [64] tightening: largest CC of each pair (ordered bits)
  __device__ __forceinline__ CorrSmem(float* smem) {
    stc = reinterpret_cast<float2*>(smem);
    key = reinterpret_cast<unsigned long long*>(smem + kStateFloats);
    list = reinterpret_cast<int*>(key + 8);
    tw = reinterpret_cast<float2*>(list + NW * 64);
    pmax = reinterpret_cast<uint32_t*>(tw + kNphi);
  }
  static constexpr size_t bytes() {
    return kStateFloats * sizeof(float) + 8 * sizeof(unsigned long long) + NW * 64 * sizeof(int) +
           kNphi * sizeof(float2) + 64 * sizeof(uint32_t);
  }
};

// The rows of row tile `tile` (bit r of `rows`: its row r) against the reference
// tiles kt0 .. kt1 - 1, every pair evaluated; the rows' bests go to a.rowkey.  The
// operand is that of tile a_tile in a.A.
template <int PREC, int NW, class Contract, int MODE, bool SPLIT>
__device__ __forceinline__ void corr_tile(const CorrArgs& a, int tile, int a_tile, uint32_t rows, int kt0, int kt1,
                                          const CorrSmem<NW>& sm, Contract& con) {
  const int tid = threadIdx.x, ln = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (tid < 8) sm.key[tid] = 0ull;
  if (MODE == kTighten && w == 0) sm.pmax[ln] = 0u;
  con.prefetch(a, kt0, w, ln);
  // (FP16: each particle's operand rows come scaled by a power of two of its
  // own, exact, so results do not depend on how particles are grouped)
  con.load_a(a, a_tile, a_block_pos(ln & 15), w, ln);
  for (int kt = kt0; kt < kt1; ++kt) {
    con.run(a, sm.stc, a_tile, kt, w, ln);
    con.prefetch(a, kt + 1 < kt1 ? kt + 1 : kt0, w, ln);
    __syncthreads();
    const uint64_t live = __ballot(((rows >> (ln >> 3)) & 1u) && kt * kRefTile + (ln & 7) < a.K);
    int* list = sm.list + w * 64;
    if ((live >> ln) & 1)
      list[__builtin_amdgcn_mbcnt_hi((uint32_t)(live >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)live, 0))] = ln;
    lds_wave_sync();
    inverse_pairs<NW, SPLIT, 64>(sm.stc, sm.tw, list, __popcll(live), w, ln, [&](int i, int n1, const float2(&x)[16]) {
      const int P = list[i];
      const int row = tile * kRowTile + (P >> 3), k = kt * kRefTile + (P & 7);
      const int n = row / a.S, s = row - n * a.S;
      if constexpr (MODE == kTable) {
        // (FP16: the particle's operand and the refset's are scaled by powers of two)
        auto value = [&](float v) { return PREC == kFP16 ? fp16_value(v, a.maxabs[n], a.b_scale) : v; };
        for (int m = 0; m < a.M; ++m) {
          float* o = a.table + ((((size_t)n * a.K + k) * a.M + m) * a.S + s) * kNphi;
#pragma unroll
          for (int n2 = 0; n2 < 16; ++n2) o[n1 + 16 * n2] = value(m ? x[n2].y : x[n2].x);
        }
      } else if constexpr (MODE == kTighten) {
        atomicMax(&sm.pmax[P], largest_cc(x, a.M));
      } else {
        const int ex = MODE == kRunnerUp ? excluded_at(a.excl[n], k, s, a.S, a.M) : -1;
        float bv;
        int bi;
        pick_best<MODE>(x, n1, a.M, key_value(sm.key[P >> 3]), ex, bv, bi);
        if (bi != 0x7fffffff) {
          const int iota = ((k * a.M + (bi >> 8)) * a.S + s) * kNphi + (bi & 255);
          atomicMax(&sm.key[P >> 3], cand_key(bv, iota));
        }
      }
    });
    __syncthreads();
    if (MODE == kTighten && w == 0) {
      if ((live >> ln) & 1) {
        const int row = tile * kRowTile + (ln >> 3);
        const float cc = key_value((unsigned long long)sm.pmax[ln] << 32);
        const float lo = tighten_pair(a, row / a.S, row, kt * kRefTile + (ln & 7), cc);
        if (lo > -INFINITY) atomicMax(&sm.key[ln >> 3], cand_key(lo, 0));
      }
      sm.pmax[ln] = 0u;
    }
  }
  if (MODE != kTable && tid < 8 && ((rows >> tid) & 1u)) atomicMax(&a.rowkey[tile * kRowTile + tid], sm.key[tid]);
}

template <int PREC, int NW, int MAXR, bool RES, bool EXACT>
struct ContractFor {
  typedef typename std::conditional<PREC == kFP32, Fp32Contract<NW, MAXR, RES, EXACT>,
                                    Half16Contract<PREC == kFP32 ? kBF16 : PREC, NW, MAXR, RES>>::type type;
};

template <int PREC, int NW, int MAXR, bool RES, bool EXACT, int MODE>
__device__ __forceinline__ void corr_item(const CorrArgs& a, int item, float* smem) {
  CorrSmem<NW> sm(smem);
  if (threadIdx.x < kNphi) sm.tw[threadIdx.x] = w256c(a.cs32, threadIdx.x);
  typename ContractFor<PREC, NW, MAXR, RES, EXACT>::type con;
  const int part = item / a.n_row_tiles, tile = item - part * a.n_row_tiles, kt0 = part * a.kt_per_wg;
  const uint32_t rows = (1u << min(kRowTile, a.rows - tile * kRowTile)) - 1u;
  corr_tile<PREC, NW, decltype(con), MODE, NW == 8>(a, tile, tile, rows, kt0, min(kt0 + a.kt_per_wg, a.n_ref_tiles), sm,
                                                    con);
}

template <int PREC, int NW, int MAXR, bool RES, bool EXACT, int MODE>
__global__ __launch_bounds__(NW * 64) void k_corr(CorrArgs a) {
  extern __shared__ float smem[];
  corr_item<PREC, NW, MAXR, RES, EXACT, MODE>(a, blockIdx.x, smem);
}

// Several stacks' tiles in one launch: where each is a few rounds of workgroups, the
// rounds that end half empty are one (12 stacks of 300 particles against 8 references, 5500
// to 15 000 rows each, whole call BF16 3440 us one by one, 2670 here; FP32 4340, 3410).
template <int PREC, int NW, int MAXR, bool RES, bool EXACT>
__global__ __launch_bounds__(NW * 64) void k_corr_batch(CorrBatch b) {
  extern __shared__ float smem[];
  const int item = blockIdx.x;
  int p = 0;
  while (p + 1 < b.n && b.start[p + 1] <= item) ++p;
  corr_item<PREC, NW, MAXR, RES, EXACT, kArgmax>(b.piece[p], item - b.start[p], smem);
}

template <int P_, int NW_, int MR_, bool RES_, bool EXACT_>
struct Cfg {
  static constexpr int P = P_, NW = NW_, MR = MR_;
  static constexpr bool RES = RES_, EXACT = EXACT_;
};

template <class C, int MODE>
inline void launch_mode(const CorrArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((k_corr<C::P, C::NW, C::MR, C::RES, C::EXACT, MODE>), dim3(corr_items(a)), dim3(C::NW * 64),
                     CorrSmem<C::NW>::bytes(), st, a);
}

// What a dispatch launches: mode kArgmax, kTable (write the CC table) or kRunnerUp over one
// chunk's row tiles, or the batched arg-max.
template <class C, int MODE>
inline void launch_mode(const CorrBatch& b, hipStream_t st) {
  static_assert(MODE == kArgmax, "only the arg-max is batched");
  hipLaunchKernelGGL((k_corr_batch<C::P, C::NW, C::MR, C::RES, C::EXACT>), dim3(b.start[b.n]), dim3(C::NW * 64),
                     CorrSmem<C::NW>::bytes(), st, b);
}
inline const CorrArgs& first_piece(const CorrArgs& a) { return a; }
inline const CorrArgs& first_piece(const CorrBatch& b) { return b.piece[0]; }

// Per-precision instantiation sets (one translation unit each).
void corr_dispatch_fp32(int variant, const CorrArgs& a, int mode, hipStream_t st);
void corr_dispatch_bf16(int variant, const CorrArgs& a, int mode, hipStream_t st);
void corr_dispatch_fp16(int variant, const CorrArgs& a, int mode, hipStream_t st);
void corr_dispatch_fp32(int variant, const CorrBatch& b, hipStream_t st);
void corr_dispatch_bf16(int variant, const CorrBatch& b, hipStream_t st);
void corr_dispatch_fp16(int variant, const CorrBatch& b, hipStream_t st);

template <class C>
inline void corr_go(const CorrArgs& a, int mode, hipStream_t st) {
  if (mode == kTable) launch_mode<C, kTable>(a, st);
  else if (mode == kRunnerUp) launch_mode<C, kRunnerUp>(a, st);
  else launch_mode<C, kArgmax>(a, st);
}
template <class C>
inline void corr_go(const CorrBatch& b, int, hipStream_t st) {
  launch_mode<C, kArgmax>(b, st);
}

// 16-bit forms: operand ring bucket MAXR in {8, 10, 12, 16} (R4 <= 8, 9..10,
// 11..12, 13..16).
template <int PREC, bool RES, class Args>
inline void corr_dispatch_16(const Args& a, int mode, hipStream_t st) {
  const int R4 = first_piece(a).R4;
  if (R4 <= 8) return corr_go<Cfg<PREC, 8, 8, RES, true>>(a, mode, st);
  if (R4 <= 10) return corr_go<Cfg<PREC, 8, 10, RES, true>>(a, mode, st);
  if (R4 <= 12) return corr_go<Cfg<PREC, 8, 12, RES, true>>(a, mode, st);
  return corr_go<Cfg<PREC, 8, 16, RES, true>>(a, mode, st);
}

}  // namespace mra
