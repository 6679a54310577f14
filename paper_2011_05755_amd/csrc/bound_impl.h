// Upper bound of the CC of every (row, reference) pair over all 256 angles
// and both mirrors, from a 16-bit contraction whose results never leave the
// registers: the first half of the arg-max, which decides which pairs the
// second half (fine_impl.h) has to evaluate.
//
// With the entries U of a pair's 16-bit products (see corr_impl.h), per mirror m,
//   c_m(a) <= |g_0| + |g_128| + sum_{f=1}^{127} 2 |G_m,f|      (triangle inequality),
//   2|G_0,f| = |(U00 + U11, U01 - U10)|, 2|G_1,f| = |(U01 + U10, U00 - U11)|.
// The 16 lowest slots enter with these magnitudes; the others, in groups of
// 2, 4 and 8 slots, through Cauchy-Schwarz over the group's energy:
// sum 2|G_m,f| <= sqrt(n 2 sum U^2) for n slots (no exchange between lanes
// and one square root per group; on 76 px, 100 references it leaves about a
// quarter more pairs than all 128 magnitudes would).  The bound is raised by
// 2^-12 of itself against its own rounding and that of the inverse FFT
// (both below 10^-5 relative).
//
// FP32 alignment (ERR): the operands here are the FP32 ones rounded to FP16
// (scaled by powers of two), so the bound is also raised by what that rounding
// can change.  With |a - fl(a)| <= u |a| + eta (u = 2^-11; eta = 2^-14, the
// smallest normal number, so that flushed subnormals are covered), per slot
// |dU_pq| <= |da_p||b_q| + |a_p||db_q| + |da_p||db_q| over the rings, and
//   sum_f |d(2 G_f)| <= sqrt(2) (Da Nb + Na Db + Da Db),
// Na, Nb the norms of the row's and the reference's whole operand and Da =
// u Na + eta sqrt(n), Db alike (n elements each).  That is about 0.5 % of a
// particle's best CC at SNR 0.05.  A particle whose pixels do not scale into
// FP16 (not finite, or within 2^9 of overflow) gets infinite bounds.
//
// A 4-wave workgroup holds half the slots (0 .. 63 or 64 .. 127) of the
// operand of NT row tiles (16 rows; 8 where more than 48 rings leave no registers
// for two) in registers and streams the reference operand once for all of
// them: two row tiles per read halve the stream from L2 (160 KiB per reference
// tile at 35 rings).  Two workgroups share a CU and run independently, so one
// multiplies while the other waits for its operand from HBM, meets its waves or
// writes.  20 000 x 49 rows, 100 references, 35 rings, BF16: 8.8 ms with the sum
// of the halves, 9.1 with one 8-wave workgroup over all slots; 3001 x 49 rows,
// 50 references, 36 rings, FP16: 0.86 and 0.97 ms.  What bounds it: matrix and
// vector instructions, 39 and 43 % of the time and hardly at once with two
// waves per SIMD; without the reference loads it runs 16 % shorter, with
// nothing but loads 26 %.  (No faster: 8 slots ahead instead of 4; the products
// of a slot in one run, also at raised priority; 32 rows per workgroup, which
// halves what L2 delivers.)  The waves' partial
// bounds meet in LDS every kBoundTiles reference tiles, in two alternating
// buffers: one barrier per kBoundTiles.  The halves' bounds are added, and
// each row's largest found, by k_bound_sum.
#pragma once

#include "corr_impl.h"

namespace mra {

constexpr int kBoundTiles = 4;

// Bound terms of one pair of lanes and row tile.  Lane q = ln & 1 gathers row
// 2 (ln / 16) + q; with x, y its own entries of that row and u, v the partner
// lane's, (x, y, u, v) = (U00, U10, U01, U11) in lane q = 0 and (U01, U11, U00,
// U10) in lane q = 1: the two magnitudes come out with the mirrors swapped in
// lane q = 1, which is undone once, when the sums are stored.
struct BoundSum {
  float b0, b1;  // exact magnitudes (swapped mirrors in odd lanes)
  float c;       // group terms, the same for both mirrors
  float e0, e1;  // energy of the running group: rows 2 (ln / 16) and 2 (ln / 16) + 1, this lane's column
  __device__ __forceinline__ void clear() { b0 = b1 = c = e0 = e1 = 0.f; }
  __device__ __forceinline__ void exact(const f32x4& acc, bool q, bool slot0) {
    const float x = q ? acc[2] : acc[0], y = q ? acc[3] : acc[1];
    const float u = swap_adjacent(q ? acc[0] : acc[2]), v = swap_adjacent(q ? acc[1] : acc[3]);
    const float s = x + v, d = x - v, s2 = u + y, d2 = u - y;
    float t0 = __builtin_amdgcn_sqrtf(fmaf(s, s, d2 * d2)), t1 = __builtin_amdgcn_sqrtf(fmaf(s2, s2, d * d));
    if (slot0) t0 = t1 = 0.25f * (fabsf(s + s2) + fabsf(s - s2));  // |g_0| + |g_128|, the same for both mirrors
    b0 += t0;
    b1 += t1;
  }
  __device__ __forceinline__ void energy(const f32x4& acc) {
    e0 = fmaf(acc[0], acc[0], fmaf(acc[1], acc[1], e0));
    e1 = fmaf(acc[2], acc[2], fmaf(acc[3], acc[3], e1));
  }
  __device__ __forceinline__ void close_group(bool q, int n) {
    const float own = q ? e1 : e0, other = swap_adjacent(q ? e0 : e1);
    c += __builtin_amdgcn_sqrtf(2.f * n * (own + other));
    e0 = e1 = 0.f;
  }
};

// Squares of the lane's operand elements (FP16), for the row norms.
__device__ __forceinline__ float dword_square(uint32_t d, float s) {
  typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
  const f16x2 v = __builtin_bit_cast(f16x2, d);
  return __builtin_amdgcn_fdot2(v, v, s, false);
}

// A row tile's operand in registers: per slot of the wave the steps held 8
// wide, and the narrow last step (TD dwords per slot, where there is one)
// of 4 / TD slots packed into one matrix-core operand.  The reference
// operand that meets it holds its slot's dwords in the same place and zeros
// elsewhere, so no slot's particle operand is padded (padded, two row tiles
// would not fit the registers).
template <class Con>
struct BoundA {
  static constexpr int NF = Con::NF, TD = Con::TD, SPQ = TD ? 4 / TD : 1;
  u32x4 f[Con::SPW][NF];
  u32x4 q[TD ? Con::SPW / SPQ : 1];
  // the runs of waves w and w + 4 of 8 in half h
  __device__ __forceinline__ void load(const Con& con, const CorrArgs& a, int tile, int w, int h, int ln) {
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      u32x4 u[8 * Con::NS];
      con.load_run(a, tile, a_block_pos(ln & 15), w + 4 * r, ln, h, u);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int i = 8 * r + j;
#pragma unroll
        for (int d = 0; d < 4 * NF + TD; ++d) {
          const uint32_t x = Con::dword(u, j, d);
          if (d < 4 * NF) f[i][d / 4][d % 4] = x;
          else q[i / SPQ][(i % SPQ) * TD + d - 4 * NF] = x;
        }
      }
    }
  }
};
// One slot's reference operand; i is the slot's index in the wave.  An object
// takes slots of one place i % SPQ only, so the zeros beside it are written
// once (they are hidden from the compiler, which would write them again
// with every load).
template <class Con>
struct BoundB {
  u32x4 f[Con::NF];
  u32x4 q;
  __device__ __forceinline__ void clear() {
    uint32_t z = 0;
    asm("" : "+v"(z));
    q = u32x4{z, z, z, z};
  }
  __device__ __forceinline__ void load(const Con& con, const CorrArgs& a, int kt, int slot, int i, int ln) {
    typename Con::Frag b;
    con.load_b(a, kt, slot, ln, b);
#pragma unroll
    for (int s = 0; s < Con::NF; ++s) f[s] = b.f[s];
    if constexpr (Con::TD > 0) {
      constexpr int SPQ = 4 / Con::TD;
#pragma unroll
      for (int d = 0; d < Con::TD; ++d) q[i % SPQ * Con::TD + d] = b.t[d];
    }
  }
};
// The slot's block of NT row tiles, the tiles' products interleaved: a step
// that adds to the last one's result waits for it.
template <int PREC, class Con, int NT>
__device__ __forceinline__ void bound_products(const BoundA<Con> (&x)[NT], const BoundB<Con>& y, int i,
                                               f32x4 (&acc)[NT]) {
  typedef typename Con::V V;
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < Con::NF; ++s)
#pragma unroll
    for (int t = 0; t < NT; ++t)
      acc[t] = Op16<PREC>::mfma(__builtin_bit_cast(V, x[t].f[i][s]), __builtin_bit_cast(V, y.f[s]), acc[t]);
  if constexpr (Con::TD > 0)
#pragma unroll
    for (int t = 0; t < NT; ++t)
      acc[t] = Op16<PREC>::mfma(__builtin_bit_cast(V, x[t].q[i / (4 / Con::TD)]), __builtin_bit_cast(V, y.q), acc[t]);
}

constexpr int kBoundWaves = 4, kBoundThreads = 64 * kBoundWaves;
template <int NT>
struct BoundSmem {
  // partial bounds of both mirrors, [2][kBoundTiles][waves][NT][64]; 16 more
  // per tile spread the banks of the sums
  static constexpr int kTile = kBoundWaves * NT * 64 + 16;
  float2* pp;
  float* norm;  // [waves][NT * 8] partial squared row norms
  __device__ __forceinline__ BoundSmem(float* smem) {
    pp = reinterpret_cast<float2*>(smem);
    norm = smem + 2 * kBoundTiles * kTile * 2;
  }
  static constexpr size_t bytes() { return (2 * kBoundTiles * kTile * 2 + kBoundWaves * NT * 8) * sizeof(float); }
};

// Row blocks of a launch, padded so that every XCD gets both halves.
__device__ __forceinline__ int bound_blocks(const CorrArgs& a, int nt) {
  return ((a.n_row_tiles + nt - 1) / nt + 7) & ~7;
}

// Half H of the slots of row block blk (NT tiles) against the reference tiles
// of part `part` (a.kt_per_wg each); H = 0: with 16 slots of magnitudes.
template <int PREC, int MAXR, int NT, bool ERR, int H>
__device__ __forceinline__ void bound_item(const CorrArgs& a, int blk, int part, float* smem) {
  const BoundSmem<NT> sm(smem);
  const int tid = threadIdx.x, ln = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kt0 = part * a.kt_per_wg, kt1 = min(kt0 + a.kt_per_wg, a.n_ref_tiles);
  typedef Half16Contract<PREC, 8, MAXR, false> Con;
  constexpr int SPW = Con::SPW;
  Con con;
  BoundA<Con> A[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)  // (a tile past the last repeats it; its bounds are not stored)
    A[t].load(con, a, min(blk * NT + t, a.n_row_tiles - 1), w, H, ln);
  if constexpr (ERR) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < SPW; ++i) {
#pragma unroll
        for (int d = 0; d < 4 * Con::NF; ++d) s = dword_square(A[t].f[i][d / 4][d % 4], s);
      }
#pragma unroll
      for (int d = 0; d < SPW * Con::TD; ++d) s = dword_square(A[t].q[d / 4][d % 4], s);
      // lane's block row j = ln & 15 is (row j / 2, p = j % 2), ring group ln / 16
      s += __shfl_xor(s, 1);
      s += __shfl_xor(s, 16);
      s += __shfl_xor(s, 32);
      if (ln < 16 && !(ln & 1)) sm.norm[w * NT * 8 + t * 8 + (ln >> 1)] = s;
    }
  }
  const int P = lane_pair(ln);
  const bool q = ln & 1;
  // slot i of the wave: i = 8 r + j is slot j of the run of wave w + 4 r
  auto slot = [&](int i) { return 64 * H + w + 4 * (i >> 3) + 8 * (i & 7); };
  // the reference operand is kept D slots ahead, across reference tiles
  // (one slot ahead, a slot takes a whole L2 latency); the sums of a slot are
  // taken while the next one's products run
  constexpr int D = Con::TD == 2 ? 2 : 4;
  BoundB<Con> b[D];
#pragma unroll
  for (int i = 0; i < D; ++i) {
    b[i].clear();
    b[i].load(con, a, kt0, slot(i), i, ln);
  }
  auto take = [&](BoundSum& s, const f32x4& acc, int i) {
    const int j = i & 7;
    if (H == 0 && j < 2) s.exact(acc, q, w == 0 && i == 0);
    else s.energy(acc);
    if (H == 0 && j == 3) s.close_group(q, 2);
    if (j == 7) s.close_group(q, H == 0 ? 4 : 8);
  };
  int buf = 0;
  for (int kb = kt0; kb < kt1; kb += kBoundTiles, buf ^= 1) {
    const int nu = min(kBoundTiles, kt1 - kb);
#pragma unroll 1
    for (int u = 0; u < nu; ++u) {
      const int kt = kb + u;
      BoundSum bs[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) bs[t].clear();
      const int ktn = kt + 1 < kt1 ? kt + 1 : kt0;
      f32x4 acc[NT];
#pragma unroll
      for (int i = 0; i < SPW; ++i) {
        f32x4 cur[NT];
        bound_products<PREC>(A, b[i % D], i, cur);
        b[i % D].load(con, a, i + D < SPW ? kt : ktn, slot((i + D) % SPW), i + D, ln);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          if (i > 0) take(bs[t], acc[t], i - 1);
          acc[t] = cur[t];
        }
        // one slot at a time: a schedule that runs further ahead holds more
        // results and reference operands than there are registers
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) take(bs[t], acc[t], SPW - 1);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const float m0 = bs[t].b0 + bs[t].c, m1 = bs[t].b1 + bs[t].c;
        sm.pp[(buf * kBoundTiles + u) * sm.kTile + (w * NT + t) * 64 + P] =
            q ? make_float2(m1, m0) : make_float2(m0, m1);
      }
    }
    __syncthreads();
    // 4 tiles' references side by side: whole lines of a row's bounds
    for (int i = tid; i < NT * 64 * kBoundTiles; i += kBoundThreads) {
      const int u = (i >> 3) % kBoundTiles, lr = i / (8 * kBoundTiles), t = lr >> 3, pr = (lr & 7) * 8 + (i & 7);
      const int row = blk * NT * kRowTile + lr;
      if (u >= nu || row >= a.rows) continue;
      float B0 = 0.f, B1 = 0.f;
#pragma unroll
      for (int w2 = 0; w2 < kBoundWaves; ++w2) {
        const float2 v = sm.pp[(buf * kBoundTiles + u) * sm.kTile + (w2 * NT + t) * 64 + pr];
        B0 += v.x;
        B1 += v.y;
      }
      (H ? a.ub_hi : a.ub)[(size_t)row * a.ldu + (kb + u) * kRefTile + (i & 7)] = a.M == 2 ? fmaxf(B0, B1) : B0;
    }
    if constexpr (ERR) {
      const int row = blk * NT * kRowTile + tid;
      if (kb == 0 && tid < NT * kRowTile && row < a.rows) {
        float s = 0.f;
#pragma unroll
        for (int w2 = 0; w2 < kBoundWaves; ++w2) s += sm.norm[w2 * NT * 8 + tid];
        a.rownorm[H * a.rows + row] = s;
      }
    }
  }
}

// Work item of a piece: half (r / 8) % 2 of row block (r / 16) 8 + r % 8, r the
// item in its reference part.
template <int PREC, int MAXR, int NT, bool ERR>
__device__ __forceinline__ void bound_dispatch_item(const CorrArgs& a, int item, float* smem) {
  const int per_part = 2 * bound_blocks(a, NT);
  const int part = item / per_part, r = item - part * per_part, blk = (r >> 4) * 8 + (r & 7);
  if (blk * NT >= a.n_row_tiles) return;
  if (r & 8) bound_item<PREC, MAXR, NT, ERR, 1>(a, blk, part, smem);
  else bound_item<PREC, MAXR, NT, ERR, 0>(a, blk, part, smem);
}

template <int PREC, int MAXR, int NT, bool ERR>
__global__ __launch_bounds__(kBoundThreads, 2) void k_bound(CorrArgs a) {
  extern __shared__ float smem[];
  bound_dispatch_item<PREC, MAXR, NT, ERR>(a, blockIdx.x, smem);
}

// Batched form over the items of several stacks (start[p]: piece p's first).
template <int PREC, int MAXR, int NT, bool ERR>
__global__ __launch_bounds__(kBoundThreads, 2) void k_bound_batch(CorrBatch b) {
  extern __shared__ float smem[];
  const int item = blockIdx.x;
  if (item >= b.start[b.n]) return;
  int p = 0;
  while (p + 1 < b.n && b.start[p + 1] <= item) ++p;
  bound_dispatch_item<PREC, MAXR, NT, ERR>(b.piece[p], item - b.start[p], smem);
}

template <int PREC, int MAXR, int NT, bool ERR>
inline void bound_go(const CorrArgs* a, const CorrBatch* b, int grid, hipStream_t st) {
  const size_t lds = BoundSmem<NT>::bytes();
  if (b) hipLaunchKernelGGL((k_bound_batch<PREC, MAXR, NT, ERR>), dim3(grid), dim3(kBoundThreads), lds, st, *b);
  else hipLaunchKernelGGL((k_bound<PREC, MAXR, NT, ERR>), dim3(grid), dim3(kBoundThreads), lds, st, *a);
}

// Row tiles per workgroup of the ring count R4.
constexpr int bound_row_tiles(int R4) { return R4 <= 12 ? 2 : 1; }

template <int PREC, bool ERR>
inline void bound_dispatch(int R4, const CorrArgs* a, const CorrBatch* b, int grid, hipStream_t st) {
  if (R4 <= 8) return bound_go<PREC, 8, 2, ERR>(a, b, grid, st);
  if (R4 <= 10) return bound_go<PREC, 10, 2, ERR>(a, b, grid, st);
  if (R4 <= 12) return bound_go<PREC, 12, 2, ERR>(a, b, grid, st);
  return bound_go<PREC, 16, 1, ERR>(a, b, grid, st);
}

}  // namespace mra
