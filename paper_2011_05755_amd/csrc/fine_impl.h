// Second half of the arg-max: with the upper bound of every (row, reference)
// pair known (bound_impl.h), evaluate only the pairs that can still win.
//
// One workgroup takes a particle.  It orders the particle's rows (shifts) by
// their largest bound and takes them in groups of up to eight, best first,
// until the best CC found exceeds every bound that is left.  The first group
// starts with each row's best reference, which settles the threshold for nearly all else;
// after that the pairs of a group whose bound reaches it are collected and
// evaluated 16 at a time, from up to 8 references picked freely.  On 76 px
// particles with 100 references at SNR 0.05 about 12 of the 4900 pairs are
// evaluated, in two to three such steps, so the kernel is bound by the latency
// of a step's phases (operands, contraction, inverse FFT, each between
// barriers), not by their arithmetic: the state holds 16 pairs and both
// operands are streamed through the registers, so that several workgroups
// share a CU: by registers 4 of 4 waves (16-bit forms) or 2 of 8 (FP32); by LDS one less
// of the former from 121 shifts on, and only one of the latter from 90 px or so (its image).
// Lanes of rows or references that a step does not need repeat those it does,
// and load nothing more.
//
// The result is the arg-max over every pair: a pair that is never evaluated
// has a bound below the best CC (part_thr: below it by the re-ranking margin
// in the re-ranked 16-bit forms, so that every row within that margin keeps its
// exact best).  Bounds that are not below it in every case, infinite and NaN
// ones included, are evaluated, and ties are decided by the flat index in
// cand_key, whatever the order of evaluation.
//
// 16-bit forms read the rows' operand as the resampler left it.  FP32
// alignment makes the FP32 operand of the eight rows here (resampling and
// ring FFTs as in the resampling kernel, the same arithmetic), in a scratch
// tile per workgroup that stays in the caches, so the FP32 operand of all rows
// never goes through HBM.  Before that (kFineTighten) the FP16 operand's own CC
// of the live pairs replaces their bounds: it is within fp16_error of the FP32
// one, which leaves 3 to 4 rows per particle instead of 10 to 13, one group of
// eight instead of two (76 px, 100 references, tightening and evaluation against
// evaluation alone: 64 particles 254 against 420 us, 512: 517 against 1325).
//
// A particle that has not come to its end after some steps is left to the
// whole chip (k_fine_over): the pairs of its row tiles and references are
// units of work for every workgroup, the bests meet in memory, and k_fine_done
// writes the result, or after tightening the rows' largest bounds.  The
// arg-max is over the same pairs and more, so the result is the same.
//
// A particle of which the first step leaves more than an eighth of all pairs live
// (references that are noisy images themselves, as in the first passes of a
// classification) is not evaluated here: its row tiles go to k_dense, which
// evaluates (FP32: tightens) every pair of theirs.  FP32 particles with many live
// pairs left after tightening (blank images, whose candidates all tie) have their rows
// evaluated there in FP32 too.
#pragma once

#include <climits>

#include "bound_impl.h"
#include "polar_impl.h"

namespace mra {

constexpr int kFinePairs = 16;     // pairs evaluated at a time
constexpr int kFineList = 512;     // entries of the list of live pairs
static_assert(kFineTighten == kTighten && kFineRunnerUp == kRunnerUp && kFineArgmax == kArgmax, "one set of modes");

// The pruning threshold a particle's best so far imposes on its rows: the
// best itself, or (re-ranked 16-bit forms) margin * |best| below it, so that
// every row within that margin of the particle's best keeps its exact best.
__device__ __forceinline__ float part_thr(float best, float margin) {
  return (margin > 0.f && best > -INFINITY) ? best - margin * fabsf(best) : best;
}

// The rows and references of a step: block row pair (row j, p) takes row
// rows[j], block column pair (reference d, q) reference refs[d]; pair P = j * 8
// + d has the state index rank[P], or -1 if it is not evaluated.  One copy per
// wave.
struct FineStep {
  int rank[64];
  int refs[8];
  int j[kFinePairs], k[kFinePairs];  // row and reference of each evaluated pair
};

__device__ __forceinline__ void store_live(float2* stc, int slot, int ln, const f32x4& acc, int rank) {
  float2 h0, h1;
  pair_gather(ln, acc, h0, h1);
  if (rank >= 0) {
    stc[(slot * 2) * kFinePairs + rank] = h0;
    stc[(slot * 2 + 1) * kFinePairs + rank] = h1;
  }
}

// Contractions of one step for the wave's slots, both operands streamed; the
// products and their order are those of corr_impl.h.
//
// 16-bit forms, NW waves: the lane's block row is element k of row tile `tile`,
// counted from the particle's first (c.A points there); ref is the lane's
// reference.  Wave w takes the operand's runs 2 (w + NW i) + hh of 8 slots.
template <int PREC, int MAXR, int NW>
struct FineContract16 {
  typedef Half16Contract<PREC, 8, MAXR, false> Base;
  typedef typename Base::Frag Frag;
  static constexpr int kSlotsPerWave = kSlots / NW;
  // the wave's q-th slot, 8 of a run at a time: run index q / 8
  static __device__ __forceinline__ int slot_of(int q, int w) {
    const int run = q >> 3;  // (w8, hh) = (w + NW (run / 2), run % 2)
    return w + NW * (run >> 1) + 8 * (8 * (run & 1) + (q & 7));
  }
  static __device__ __forceinline__ void run(const CorrArgs& c, float2* stc, int tile, int k, int ref, int w, int ln,
                                             int rank) {
    // opaque lane values: what is derived from them is computed here, not
    // kept in registers across the caller's loops
    asm volatile("" : "+v"(tile), "+v"(k), "+v"(ln), "+v"(rank), "+v"(ref));
    ln &= 63;
    Base con;
    constexpr int D = 4;  // reference operand kept D slots ahead
    Frag b[D];
    const int pl = b16_lane(ref & 7, ln);
    const size_t tile_off = (size_t)(ref >> 3) * (kSlots * Base::SE);
#pragma unroll
    for (int i = 0; i < D; ++i) con.load_b_at(c, 0, slot_of(i, w), pl, tile_off, b[i]);
    const uint32_t lane_off = (uint32_t)((tile * 4 + (ln >> 4)) * c.R4) * (kSlots * 16 * 2) + k * 16;
#pragma unroll 1
    for (int run = 0; run < kSlotsPerWave / 8; ++run) {
      const int g = 2 * (w + NW * (run >> 1)) + (run & 1);
      u32x4 u[8 * Base::NS];
#pragma unroll
      for (int t = 0; t < 8 * Base::NS; ++t) {
        if (t < MAXR) {
          const char* at = reinterpret_cast<const char*>(c.A) + (size_t)(t < c.R4 ? t : c.R4 - 1) * (kSlots * 16 * 2) +
                           g * 256;  // the same for every lane
          u[t] = *reinterpret_cast<const u32x4*>(at + lane_off);
        } else {
          u[t] = u32x4{0u, 0u, 0u, 0u};
        }
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int q = 8 * run + j;
        Frag x;
#pragma unroll
        for (int d = 0; d < 4 * Base::NF; ++d) x.f[d / 4][d % 4] = Base::dword(u, j, d);
#pragma unroll
        for (int d = 0; d < Base::TD; ++d) x.t[d] = Base::dword(u, j, 4 * Base::NF + d);
        const f32x4 acc = con.product(x, b[j % D]);
        // (past the last slot it reads the last one again)
        con.load_b_at(c, 0, slot_of(q + D < kSlotsPerWave ? q + D : kSlotsPerWave - 1, w), pl, tile_off, b[j % D]);
        store_live(stc, slot_of(q, w), ln, acc, rank);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
};

// FP32, 8 waves: the operand is the scratch tile c.A (kRingPerm: the wave's
// slots w + 8 i in pairs, one 8-byte load for two slots).
template <int MAXR>
struct FineContract32 {
  static constexpr int M4 = (MAXR + 3) / 4;
  struct Ops {
    f32x2 a[MAXR];
    f32x4 b0[M4], b1[M4];
  };
  static __device__ __forceinline__ void load(const CorrArgs& c, const float* ap, const float* bp, int i2, int ln,
                                              Ops& o) {
#pragma unroll
    for (int t = 0; t < MAXR; ++t) o.a[t] = a_pair<0>(c, ap + 32 * i2, ln, t);
    const int last = b32_pitch(c.R4) / 4 - 1;
    const float* b0 = bp + (size_t)i2 * 16 * 8 * b32_pitch(c.R4);
    const float* b1 = b0 + (size_t)8 * 8 * b32_pitch(c.R4);
#pragma unroll
    for (int t = 0; t < M4; ++t) {  // unconditional (see corr_impl.h)
      o.b0[t] = *reinterpret_cast<const f32x4*>(b0 + 4 * (t < last ? t : last));
      o.b1[t] = *reinterpret_cast<const f32x4*>(b1 + 4 * (t < last ? t : last));
    }
  }
  static __device__ __forceinline__ void run(const CorrArgs& c, float2* stc, int, int, int ref, int w, int ln,
                                             int rank) {
    asm volatile("" : "+v"(ln), "+v"(rank), "+v"(ref));
    ln &= 63;
    const float* ap = c.A + ((size_t)(ln >> 4) * c.R4 * kSlots + 16 * w) * 16 + 2 * a_block_pos(ln & 15);
    const float* bp = b32_lane(c, ref, w, ln);
    auto mul = [&](int i2, const Ops& o) {
      f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < MAXR; ++t) {
        if (t < c.R4) {
          acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(o.a[t].x, o.b0[t / 4][t % 4], acc0, 0, 0, 0);
          acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(o.a[t].y, o.b1[t / 4][t % 4], acc1, 0, 0, 0);
        }
      }
      store_live(stc, w + 16 * i2, ln, acc0, rank);
      store_live(stc, w + 16 * i2 + 8, ln, acc1, rank);
    };
    if constexpr (MAXR <= 9) {  // two slots ahead
      Ops o[2];
      load(c, ap, bp, 0, ln, o[0]);
#pragma unroll 1
      for (int i2 = 0; i2 < 8; i2 += 2) {
        load(c, ap, bp, i2 + 1, ln, o[1]);
        mul(i2, o[0]);
        load(c, ap, bp, i2 + 2 < 8 ? i2 + 2 : 7, ln, o[0]);
        mul(i2 + 1, o[1]);
      }
    } else {
#pragma unroll 1
      for (int i2 = 0; i2 < 8; ++i2) {
        Ops o;
        load(c, ap, bp, i2, ln, o);
        mul(i2, o);
      }
    }
  }
};

// LDS of a workgroup: S rows, NW waves.
struct FineSmem {
  unsigned long long* key;    // [S] best candidate of each row (0 = none)
  unsigned long long* pbest;  // best of the particle
  float2* tw;                 // exp(-2 pi i e / 256)
  float* rowmax;              // [S] largest bound of each row
  int* rowarg;                // [S] its reference
  int* order;                 // [S] rows by falling rowmax
  int* taken;                 // [S] 16-bit forms: the row has been in a group
  int* shift;                 // [8] the group's rows
  int* count;                 // entries of the list
  uint32_t* pmax;             // [kFinePairs] tighten: largest CC of each pair (ordered bits)
  uint32_t* live;             // [kFineList] live pairs: reference * 8 + row of the group
  FineStep* step;             // [NW]
  float* work;                // the pairs' state; between steps (FP32) the image, scratch and cos/sin
  static constexpr int pad(int S) { return (S + 3) & ~3; }
  __device__ __forceinline__ FineSmem(float* smem, int S, int NW) {
    const int P = pad(S);
    key = reinterpret_cast<unsigned long long*>(smem);
    pbest = key + P;
    tw = reinterpret_cast<float2*>(pbest + 2);
    live = reinterpret_cast<uint32_t*>(tw + kNphi);
    rowmax = reinterpret_cast<float*>(live + kFineList);
    rowarg = reinterpret_cast<int*>(rowmax + P);
    order = rowarg + P;
    taken = order + P;
    shift = taken + P;
    count = shift + 8;
    pmax = reinterpret_cast<uint32_t*>(count + 4);
    step = reinterpret_cast<FineStep*>(pmax + kFinePairs);
    work = reinterpret_cast<float*>(step + NW);
  }
  static constexpr size_t fixed_bytes(int S, int NW) {
    return (size_t)(pad(S) + 2) * 8 + kNphi * sizeof(float2) + kFineList * sizeof(uint32_t) + 4 * (size_t)pad(S) * 4 +
           (8 + 4 + kFinePairs) * 4 + NW * sizeof(FineStep);
  }
};
static_assert(sizeof(FineStep) % 16 == 0 && FineSmem::fixed_bytes(49, 4) % 16 == 0, "the work area is 16-byte aligned");

// FP32: the operand of rows first .. last - 1 of a row tile, row r being particle n at
// its shift shift_of(r) (any for the other rows), into the scratch tile, one ring per
// wave at a time (8 waves).  PERM: layout kRingPerm, else kSlotMajor.
template <bool PERM, class Shift>
__device__ __forceinline__ void fine_operand(const FineArgs& a, int n, Shift shift_of, int first, int last, float* work,
                                             float* tile) {
  float* img = work;
  float2* scr = reinterpret_cast<float2*>(work + ((a.Lp * a.Lp + 3) & ~3));
  CosSin* cs = reinterpret_cast<CosSin*>(scr + kPolarWaves * 64 * 9);
  stage_image(img, a.parts + (size_t)n * a.L * a.L, a.L, a.Lp, a.pad);
  stage_cs(cs, a.cs64);
  __syncthreads();
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), ln_ = threadIdx.x & 63;
  const int l_ = ln_ >> 3, r_ = ln_ & 7;
  float2* my = scr + w * 64 * 9;
  float* stage = reinterpret_cast<float*>(my);
  const int base = (a.cx + a.pad) * a.Lp + (a.cx + a.pad);
  const int s1m = (65536 + a.m.S1 - 1) / a.m.S1;
  const int o4 = 4 * (base + shift_offset(shift_of(r_), a.m.S1, s1m, a.m.T, a.Lp));
#pragma unroll 1
  for (int ring = w; ring < a.c.R; ring += 8) {
    // opaque lane indices: addresses are recomputed per ring instead of
    // being held in registers across the loop
    int l = l_, r = r_, ln = ln_;
    asm volatile("" : "+v"(l), "+v"(r), "+v"(ln));
    l &= 7;
    r &= 7;
    ln &= 63;
    int k1a, k1b;
    fwd_cols(l, k1a, k1b);
    float v[32];
    float2 z[16], Za[8], Zb[8];
    sample_ring(img, cs, my, (float)(a.r_min + ring), l, r, o4, 4 * a.Lp, v);
#pragma unroll
    for (int n1 = 0; n1 < 16; ++n1) z[n1] = make_float2(v[2 * n1], v[2 * n1 + 1]);
    fft_ring(cs, my, l, r, k1a, k1b, z, Za, Zb);
    RingSlots rs;
    ring_slots(cs, l, Za, Zb, rs);
    float* dst = tile + (size_t)ring * (PERM ? kSlots * 16 : 16);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      stage_slots(stage, h, r, rs);
      wave_sync();
      write_f32_half(stage, dst, h, ln, PERM, PERM ? 16 : a.c.R4 * 64, first, last);
      wave_sync();
    }
  }
}

// Where a particle is, for the functions below.
struct FineAt {
  int n, row0, S;
  int ex0;             // runner-up: the excluded flat index
  const float* ub;     // the particle's bounds
};

// Evaluates the group's pairs from i0 on, up to 16 a step: the cnt entries of
// the list (listed), or rows 0 .. cnt - 1 with their best reference.  At most
// `steps` steps (counted down); false if entries are left.
template <int PREC, int NW, class Contract, int MODE>
__device__ __forceinline__ bool fine_steps(const FineArgs& a, const CorrArgs& c, const FineSmem& sm, const FineAt& at,
                                           int cnt, bool listed, int& i0, int& steps) {
  const int tid = threadIdx.x, ln = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = at.n, row0 = at.row0, S = at.S, ex0 = at.ex0;
  const float* ub = at.ub;
  float2* stc = reinterpret_cast<float2*>(sm.work);
  FineStep& st = sm.step[w];
  auto threshold = [&]() { return part_thr(key_value(*sm.pbest), a.margin); };
#pragma unroll 1
  while (i0 < cnt) {
    if (steps <= 0) return false;
    // the next step: entries i0 .. i0 + 15 that are still live, up to the
    // first whose reference would be the ninth (lane i < 16: entry i0 + i;
    // every wave does the same)
    bool on = ln < kFinePairs && i0 + ln < cnt;
    int j = 0, k = 0;
    if (on) {
      if (listed) {
        const uint32_t e = sm.live[i0 + ln];
        k = (int)(e >> 3);
        j = (int)(e & 7u);
        // (a long list: the threshold may have passed it since)
        if (i0 > 0) on = !(ub[(size_t)sm.shift[j] * c.ldu + k] < threshold());
      } else {
        j = ln;
        k = sm.rowarg[sm.shift[ln]];
      }
    }
    uint32_t m = (uint32_t)__ballot(on);
    int first = ln;  // the first entry with this one's reference
#pragma unroll
    for (int e = kFinePairs - 1; e >= 0; --e)
      if (((m >> e) & 1) && __builtin_amdgcn_readlane(k, e) == k && e < first) first = e;
    const uint32_t fm = (uint32_t)__ballot(on && first == ln);
    const int d = __popc(fm & ((1u << (first & 31)) - 1u));
    const uint32_t over = (uint32_t)__ballot(on && d >= 8);
    const int take = over ? __ffs(over) - 1 : kFinePairs;
    i0 += take;
    m &= (1u << take) - 1u;
    if (m == 0) continue;  // the same in every wave
    --steps;
    const int np = __popc(m), e0 = __ffs(m) - 1;
    const int ka = __builtin_amdgcn_readlane(k, e0), ja = __builtin_amdgcn_readlane(j, e0);
    lds_wave_sync();  // the wave is done with its last step
    st.rank[ln] = -1;
    if (ln < 8) st.refs[ln] = ka;
    lds_wave_sync();
    if (ln < kFinePairs && ((m >> ln) & 1)) {
      const int r = __popc(m & ((1u << ln) - 1u));
      st.rank[j * 8 + d] = r;
      if (first == ln) st.refs[d] = k;
      st.j[r] = j;
      st.k[r] = k;
    }
    lds_wave_sync();
    {
      // rows without a pair repeat the first pair's
      const int jr = (ln & 15) >> 1;
      bool used = false;
#pragma unroll
      for (int r = 0; r < 8; ++r) used |= st.rank[jr * 8 + r] >= 0;
      const int row = row0 + sm.shift[used ? jr : ja];
      Contract::run(c, stc, (row >> 3) - (row0 >> 3), (ln & 1) * 8 + (row & 7), st.refs[(ln >> 1) & 7], w, ln,
                    st.rank[lane_pair(ln)]);
    }
    __syncthreads();
    inverse_pairs<NW, true, kFinePairs>(stc, sm.tw, nullptr, np, w, ln, [&](int i, int n1, const float2(&x)[16]) {
      if constexpr (MODE == kFineTighten) {
        atomicMax(&sm.pmax[i], largest_cc(x, c.M));
      } else {
        const int s = sm.shift[st.j[i]], k = st.k[i];
        const int ex = MODE == kRunnerUp ? excluded_at(ex0, k, s, S, c.M) : -1;
        float bv;
        int bi;
        pick_best<MODE == kRunnerUp ? kRunnerUp : kArgmax>(x, n1, c.M, key_value(sm.key[s]), ex, bv, bi);
        if (bi != 0x7fffffff) {
          const unsigned long long key = cand_key(bv, ((k * c.M + (bi >> 8)) * S + s) * kNphi + (bi & 255));
          atomicMax(&sm.key[s], key);
          atomicMax(sm.pbest, key);
        }
      }
    });
    __syncthreads();
    if constexpr (MODE == kFineTighten) {
      if (tid < np) {
        const float cc = key_value((unsigned long long)sm.pmax[tid] << 32);
        const float lo = tighten_pair(c, n, row0 + sm.shift[st.j[tid]], st.k[tid], cc);
        if (lo > -INFINITY) atomicMax(sm.pbest, cand_key(lo, 0));
        sm.pmax[tid] = 0u;
      }
      __syncthreads();
    }
  }
  return true;
}

// A row's largest bound, after some have been tightened: one wave.  Returns the
// lane's bounds that reach thr.
__device__ __forceinline__ int largest_bound(const CorrArgs& c, int row, float thr, int ln) {
  const float* ub = c.ub + (size_t)row * c.ldu;
  unsigned long long best = 0ull;
  int live = 0;
  for (int k = ln; k < c.K; k += 64) {
    const float v = ub[k];
    const unsigned long long key = cand_key(v == v ? v : INFINITY, k);
    best = key > best ? key : best;
    live += !(v < thr);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long other = __shfl_xor(best, o);
    best = other > best ? other : best;
  }
  if (ln == 0) c.rowkey[row] = best;
  return live;
}

// A particle with many live pairs, left to the whole chip: its bests so far
// and its number go to the list, unless the list is full.
__device__ __forceinline__ bool fine_spill(const FineSmem& sm, const FineOver& over, int item, int S) {
  __syncthreads();  // every wave has read the list's length
  if (threadIdx.x == 0) *sm.count = atomicAdd(over.count, 1);
  __syncthreads();
  const int e = *sm.count;
  __syncthreads();
  if (e >= over.cap) return false;
  if (threadIdx.x == 0) {
    over.item[e] = item;
    over.best[e] = *sm.pbest;
  }
  for (int s = threadIdx.x; s < S; s += blockDim.x) over.row[(size_t)e * over.pitch + s] = sm.key[s];
  __syncthreads();  // before the next particle's keys
  return true;
}

// More live pairs than one in kDenseShare make a particle dense.  A step here takes 13 us
// of a CU for 16 pairs, a row tile x reference tile of k_dense 6.6 us (BF16) for 64: even at
// one in 8 (76 px, 100 references, 3000 particles at SNR 0.02, BF16: 7.55, 7.24 and 6.83 ms
// at one in 6, 8 and 12; 10 000 at SNR 0.05, FP32: 18.3, 18.5 and 19.0; 64 px, 50 references,
// 200 particles, BF16: 309, 251, 248 and 246 us at one in 3, 8, 16 and 32).  After
// tightening: than one in kDenseShare32, as a step takes about 60 us there (FP32 operands
// of which none is kept), and the row tile's operand is made again.
constexpr int kDenseShare = 8, kDenseShare32 = 12;

// Whether a particle is dense at the threshold of its best so far: first by its
// rows, then by its pairs.  Called by the whole workgroup, behind a barrier.
template <int NW>
__device__ __forceinline__ bool fine_dense(const CorrArgs& c, const FineSmem& sm, const float* ub, float thr) {
  const int ln = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int rows = 0;
  for (int s0 = 0; s0 < c.S; s0 += 64)
    rows += __popcll(__ballot(s0 + ln < c.S && !(sm.rowmax[s0 + ln < c.S ? s0 + ln : 0] < thr)));
  if (rows * kDenseShare <= c.S) return false;  // (the same in every wave)
  int pairs = 0;
  for (int s = w; s < c.S; s += NW) {
    if (sm.rowmax[s] < thr) continue;
    const float* u = ub + (size_t)s * c.ldu;
    for (int k0 = 0; k0 < c.K; k0 += 64) {
      const int k = k0 + ln;
      pairs += __popcll(__ballot(k < c.K && !(u[k < c.K ? k : 0] < thr)));
    }
  }
  if (ln == 0) atomicAdd(&sm.count[1], pairs);
  __syncthreads();
  return (int64_t)sm.count[1] * kDenseShare > (int64_t)c.S * c.K;
}

// Puts a dense particle and its row tiles (each once, by the particle that comes
// first) on list LIST, and clears its rows' bests.
template <int LIST>
__device__ __forceinline__ void fine_list_dense(const CorrArgs& c, int row0, const FineDense& dense, int piece, int item) {
  const int t = (row0 >> 3) + threadIdx.x;
  if (8 * t < row0 + c.S) {
    const int lo = max(row0 - 8 * t, 0), hi = min(row0 + c.S - 8 * t, 8);
    const uint32_t bits = ((1u << hi) - 1u) & ~((1u << lo) - 1u);
    const uint32_t before = atomicOr(&dense_mask(c)[t], bits << (8 * LIST)) >> (8 * LIST);
    if ((before & 0xffu) == 0u) dense.tile[LIST][atomicAdd(&dense.count[2 * LIST], 1)] = make_int2(piece, t);
  }
  if (threadIdx.x == 0) dense.item[LIST][atomicAdd(&dense.count[2 * LIST + 1], 1)] = item;
  for (int s = threadIdx.x; s < c.S; s += blockDim.x) dense_rows(c)[row0 + s] = 0ull;
  __syncthreads();  // before the next particle's keys
}

// Particle n's results from its rows' bests: one wave.  clear: the rows' bests are
// zeroed, for the runner-up pass.
template <int PREC>
__device__ __forceinline__ void finish_rows(const FineArgs& a, int n, unsigned long long* rows, bool clear, int ln) {
  const CorrArgs& c = a.c;
  auto value = [&](float v) { return PREC == kFP16 ? fp16_value(v, c.maxabs[n], c.b_scale) : v; };
  unsigned long long best = 0ull;
  for (int s = ln; s < c.S; s += 64) {
    const unsigned long long key = rows[s];
    if (c.row_cc) {
      c.row_cc[(size_t)n * c.S + s] = value(key_value(key));
      c.row_idx[(size_t)n * c.S + s] = key_index(key);
    }
    if (clear) rows[s] = 0ull;
    best = key > best ? key : best;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long other = __shfl_xor(best, o);
    best = other > best ? other : best;
  }
  if (ln == 0) write_result(a.m, n, value(key_value(best)), key_index(best));
}

template <int PREC, int NW, class Contract, int MODE>
__device__ __forceinline__ void fine_particle(const FineArgs& a, CorrArgs c, int n, const FineOver& over,
                                              const FineDense& dense, int piece, int item, float* smem) {
  constexpr int kThreads = 64 * NW;
  const FineSmem sm(smem, c.S, NW);
  const int tid = threadIdx.x, ln = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = c.S, row0 = n * S;
  float* ub = c.ub + (size_t)row0 * c.ldu;
  if (PREC != kFP32)  // the particle's first row tile
    c.A = reinterpret_cast<const float*>(reinterpret_cast<const uint16_t*>(c.A) +
                                         (size_t)(row0 >> 3) * (kSlots * c.R4 * 64));
  const FineAt at{n, row0, S, MODE == kRunnerUp ? c.excl[n] : -1, ub};
  int steps = over.cap > 0 ? over.steps : INT_MAX;
  auto value = [&](float v) { return PREC == kFP16 ? fp16_value(v, c.maxabs[n], c.b_scale) : v; };
  if constexpr (PREC == kFP32 || MODE == kRunnerUp) {
    // a dense particle: k_dense has run (FP32), or will (16-bit runner-up; k_fine_done
    // writes the result)
    if ((dense_mask(c)[row0 >> 3] >> ((row0 & 7) + (PREC == kFP32 ? 8 : 0))) & 1u) {
      if (PREC == kFP32 && w == 0) finish_rows<PREC>(a, n, dense_rows(c) + row0, true, ln);
      return;
    }
  }
  if constexpr (MODE == kFineTighten) {
    // nothing to tighten: the particle does not scale into FP16, or is blank
    const float mx = c.maxabs[n];
    if (!(mx * 512.f < INFINITY) || mx == 0.f) return fine_list_dense<1>(c, row0, dense, piece, item);
  }

  for (int i = tid; i < kNphi; i += kThreads) sm.tw[i] = w256c(c.cs32, i);
  for (int s = tid; s < S; s += kThreads) {
    const unsigned long long kk = c.rowkey[row0 + s];
    const int k = key_index(kk);
    sm.rowmax[s] = key_value(kk);
    sm.rowarg[s] = k < c.K ? k : 0;
    sm.key[s] = 0ull;
    sm.taken[s] = 0;
  }
  if (tid == 0) {
    *sm.pbest = 0ull;
    sm.count[1] = 0;
  }
  if (tid < kFinePairs) sm.pmax[tid] = 0u;
  __syncthreads();
  for (int s = tid; s < S; s += kThreads) {
    const float m = sm.rowmax[s];
    int rank = 0;
#pragma unroll 8
    for (int t = 0; t < S; ++t) {
      const float v = sm.rowmax[t];
      rank += (v > m || (v == m && t < s)) ? 1 : 0;
    }
    sm.order[rank] = s;
  }
  __syncthreads();

  auto threshold = [&]() { return part_thr(key_value(*sm.pbest), a.margin); };
  bool first_group = true;
  for (int g0 = 0; g0 < S; first_group = false) {
    // the next group: up to eight live rows.  FP32, which makes their operand
    // here, takes the next eight in order; the 16-bit forms those in the row
    // tile of the next one, whose operand shares cache lines.  (Every wave
    // reads the same values here: the last update of *pbest and of taken lies
    // before a barrier, so all take the same way.)
    const float thr0 = threshold();
    const int top = sm.order[g0];
    if (sm.rowmax[top] < thr0) break;
    int nrow;
    if constexpr (PREC == kFP32) {
      const int i = g0 + (ln & 7);
      const bool live = i < S && !(sm.rowmax[sm.order[i < S ? i : 0]] < thr0);
      nrow = __popc((uint32_t)__ballot(live) & 0xffu);  // a prefix: rowmax falls
      // rows past the live ones repeat the first
      if (tid < 8) sm.shift[tid] = sm.order[g0 + (tid < nrow ? tid : 0)];
      g0 += 8;
    } else {
      const int s = (((row0 + top) >> 3) << 3) + (ln & 7) - row0;
      const bool live = ln < 8 && s >= 0 && s < S && !sm.taken[s] && !(sm.rowmax[s] < thr0);
      const uint32_t m = (uint32_t)__ballot(live);
      nrow = __popc(m);
      __syncthreads();
      if (tid < 8) {
        if (live) {
          sm.shift[__popc(m & ((1u << ln) - 1u))] = s;
          sm.taken[s] = 1;
        }
        if (ln >= nrow) sm.shift[ln] = top;
      }
    }
    __syncthreads();
    if constexpr (PREC != kFP32)
      while (g0 < S && sm.taken[sm.order[g0]]) ++g0;
    if constexpr (PREC == kFP32) {
      fine_operand<true>(a, n, [&](int r) { return sm.shift[r]; }, 0, 8, sm.work, const_cast<float*>(c.A));
      __syncthreads();  // the tile is written and the work area is free for the state
    }

    // the references in windows, as many as the list holds for these rows (one row,
    // 5000 references: 10 windows instead of the 79 that eight rows take); before the
    // first window of the first group (base < 0) each row's best reference
    const int lw = __builtin_ctz(kFineList) - (nrow > 4 ? 3 : (nrow > 2 ? 2 : nrow - 1)), refs = 1 << lw;
    for (int base = first_group ? -refs : 0; base < c.K; base += refs) {
      int cnt = nrow;
      if (base >= 0) {
        if (tid == 0) *sm.count = 0;
        __syncthreads();
        const float thr = threshold();
        for (int i = tid; i < kFineList; i += kThreads) {
          const int j = i >> lw, k = base + (i & (refs - 1));
          if (j >= nrow || k >= c.K) continue;
          const int s = sm.shift[j];
          const float u = ub[(size_t)s * c.ldu + k];
          if (!(u < thr) && !(first_group && k == sm.rowarg[s])) sm.live[atomicAdd(sm.count, 1)] = (uint32_t)(k * 8 + j);
        }
        __syncthreads();
        cnt = *sm.count;
      }
      int i0 = 0;
      while (!fine_steps<PREC, NW, Contract, MODE>(a, c, sm, at, cnt, base >= 0, i0, steps)) {
        if (fine_spill(sm, over, item, S)) return;
        steps = INT_MAX;
      }
      if (base >= 0) __syncthreads();  // before the list is written again
      if constexpr (MODE == kFineTighten || (PREC != kFP32 && MODE == kArgmax))
        if (base < 0 && fine_dense<NW>(c, sm, ub, threshold())) return fine_list_dense<0>(c, row0, dense, piece, item);
    }
  }
  if constexpr (MODE == kFineTighten) {
    for (int s = w; s < S; s += NW)
      if (sm.taken[s]) largest_bound(c, row0 + s, 0.f, ln);  // the rows looked at
  } else {
    if (c.row_cc)
      for (int s = tid; s < S; s += kThreads) {
        c.row_cc[(size_t)row0 + s] = value(key_value(sm.key[s]));
        c.row_idx[(size_t)row0 + s] = key_index(sm.key[s]);
      }
    if (tid == 0) write_result(a.m, n, value(key_value(*sm.pbest)), key_index(*sm.pbest));
  }
  __syncthreads();  // before the next particle's keys
}

constexpr int kOverRefs = 32;
// One unit of a particle left to the whole chip (entry e of the list): the
// pairs of its g-th row tile and kOverRefs references that reach the
// particle's best so far.
template <int PREC, int NW, class Contract, int MODE>
__device__ __forceinline__ void fine_unit(const FineArgs& a, CorrArgs c, int n, const FineOver& over, int e, int unit,
                                          float* smem) {
  static_assert(PREC != kFP32 && 8 * kOverRefs <= 64 * NW, "a pair per thread");
  const FineSmem sm(smem, c.S, NW);
  const int tid = threadIdx.x, ln = tid & 63;
  const int S = c.S, row0 = n * S, nw = (c.K + kOverRefs - 1) / kOverRefs;
  const int g = unit / nw, base = (unit - g * nw) * kOverRefs;
  const int first = ((row0 >> 3) + g) * 8 - row0;
  if (first >= S) return;
  const float* ub = c.ub + (size_t)row0 * c.ldu;
  c.A = reinterpret_cast<const float*>(reinterpret_cast<const uint16_t*>(c.A) +
                                       (size_t)(row0 >> 3) * (kSlots * c.R4 * 64));
  const FineAt at{n, row0, S, MODE == kRunnerUp ? c.excl[n] : -1, ub};
  if (tid == 0) {
    // (the best of other workgroups: any earlier value only leaves more pairs)
    *sm.pbest = __hip_atomic_load(&over.best[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *sm.count = 0;
  }
  __syncthreads();
  const float thr = part_thr(key_value(*sm.pbest), a.margin);
  const int s = first + (ln & 7);
  const bool live = ln < 8 && s >= 0 && s < S && !(key_value(c.rowkey[row0 + (s >= 0 && s < S ? s : 0)]) < thr);
  const uint32_t m = (uint32_t)__ballot(live);
  const int nrow = __popc(m);
  if (nrow == 0) {  // (the same in every wave)
    __syncthreads();  // every wave has read the best
    return;
  }
  const int top = first + __ffs(m) - 1;
  if (tid < 8) {
    if (live) {
      sm.shift[__popc(m & ((1u << ln) - 1u))] = s;
      sm.key[s] = 0ull;
    }
    if (ln >= nrow) sm.shift[ln] = top;  // rows past the live ones repeat the first
  }
  __syncthreads();
  if (tid < 8 * kOverRefs) {
    const int j = tid / kOverRefs, k = base + tid % kOverRefs;
    if (j < nrow && k < c.K && !(ub[(size_t)sm.shift[j] * c.ldu + k] < thr))
      sm.live[atomicAdd(sm.count, 1)] = (uint32_t)(k * 8 + j);
  }
  __syncthreads();
  const int cnt = *sm.count;
  if (cnt > 0) {
    int i0 = 0, steps = INT_MAX;
    fine_steps<PREC, NW, Contract, MODE>(a, c, sm, at, cnt, true, i0, steps);
    if (tid < nrow) {
      const unsigned long long key = sm.key[sm.shift[tid]];
      if (key) atomicMax(&over.row[(size_t)e * over.pitch + sm.shift[tid]], key);
    }
    if (tid == 0) atomicMax(&over.best[e], *sm.pbest);
  }
  __syncthreads();  // before the next unit's lists
}

// 16-bit operands: 4 waves, FP32: 8 (as the resampler)
constexpr int fine_waves(int prec) { return prec == kFP32 ? 8 : 4; }
template <int PREC, int MAXR>
struct FineContract {
  typedef typename std::conditional<
      PREC == kFP32, FineContract32<MAXR>,
      FineContract16<PREC == kFP32 ? kBF16 : PREC, MAXR, fine_waves(kBF16)>>::type type;
};

// Item -> piece and particle.
struct FineOne {
  FineArgs a;
  __device__ __forceinline__ int items() const { return a.m.n_part; }
  __device__ __forceinline__ int find(int item, int& n) const {
    n = item;
    return 0;
  }
  __device__ __forceinline__ const FineArgs& piece(int) const { return a; }
};
static_assert(sizeof(FineBatch) + sizeof(FineOver) + sizeof(FineDense) <= 4096, "kernel arguments");
struct FineMany {
  FineBatch b;
  __device__ __forceinline__ int items() const { return b.start[b.n]; }
  __device__ __forceinline__ int find(int item, int& n) const {
    int p = 0;
    while (p + 1 < b.n && b.start[p + 1] <= item) ++p;
    n = item - b.start[p];
    return p;
  }
  __device__ __forceinline__ const FineArgs& piece(int p) const { return b.piece[p]; }
};

// at most 128 registers: four waves per SIMD
template <int PREC, int MAXR, int MODE, class Items>
__global__ __launch_bounds__(64 * fine_waves(PREC), 4) void k_fine(Items it, FineOver over, FineDense dense) {
  extern __shared__ float smem[];
  for (int item = blockIdx.x; item < it.items(); item += gridDim.x) {
    int n;
    const int p = it.find(item, n);
    const FineArgs& a = it.piece(p);
    CorrArgs c = a.c;
    if (PREC == kFP32) c.A += (size_t)blockIdx.x * a.scratch_floats;
    fine_particle<PREC, fine_waves(PREC), typename FineContract<PREC, MAXR>::type, MODE>(a, c, n, over, dense, p, item,
                                                                                         smem);
  }
}

// The particles left over, each spread over over.units workgroups.
template <int PREC, int MAXR, int MODE, class Items>
__global__ __launch_bounds__(64 * fine_waves(PREC), 4) void k_fine_over(Items it, FineOver over) {
  extern __shared__ float smem[];
  const int cnt = min(*over.count, over.cap);
  if (cnt == 0) return;
  int last = -1;
  for (int u = blockIdx.x; u < cnt * over.units; u += gridDim.x) {
    const int e = u % cnt;
    int n;
    const FineArgs& a = it.piece(it.find(over.item[e], n));
    CorrArgs c = a.c;
    if (c.S != last) {  // the places of the table and of pmax depend on S
      const FineSmem sm(smem, c.S, fine_waves(PREC));
      if (threadIdx.x < kFinePairs) sm.pmax[threadIdx.x] = 0u;
      for (int i = threadIdx.x; i < kNphi; i += 64 * fine_waves(PREC)) sm.tw[i] = w256c(c.cs32, i);
      last = c.S;
      __syncthreads();
    }
    fine_unit<PREC, fine_waves(PREC), typename FineContract<PREC, MAXR>::type, MODE>(a, c, n, over, e, u / cnt, smem);
  }
}
// Their results, and those of the dense particles: a wave each.  After tightening:
// the rows' largest bounds, a wave per row; what is still dense goes to list 1.
template <int PREC, int MODE, class Items>
__global__ __launch_bounds__(MODE == kFineTighten ? 256 : 64) void k_fine_done(Items it, FineOver over, FineDense dense) {
  const int n_over = min(*over.count, over.cap), total = n_over + dense.count[1], ln = threadIdx.x & 63;
  for (int e = blockIdx.x; e < total; e += gridDim.x) {
    const int item = e < n_over ? over.item[e] : dense.item[0][e - n_over];
    int n;
    const int p = it.find(item, n);
    const FineArgs& a = it.piece(p);
    const CorrArgs& c = a.c;
    const int row0 = n * c.S;
    if constexpr (MODE == kFineTighten) {
      __shared__ int pairs;
      if (threadIdx.x == 0) pairs = 0;
      __syncthreads();
      unsigned long long best = 0ull;  // (of a particle left over its rows' are not kept, and not needed)
      if (e >= n_over)
        for (int s = 0; s < c.S; ++s) best = max(best, dense_rows(c)[row0 + s]);
      int live = 0;
      for (int s = threadIdx.x >> 6; s < c.S; s += 4) live += largest_bound(c, row0 + s, key_value(best), ln);
      if (e >= n_over) {
        atomicAdd(&pairs, live);
        __syncthreads();
        if ((int64_t)pairs * kDenseShare32 > (int64_t)c.S * c.K) fine_list_dense<1>(c, row0, dense, p, item);
      }
      __syncthreads();
    } else {
      unsigned long long* rows = e < n_over ? over.row + (size_t)e * over.pitch : dense_rows(c) + row0;
      finish_rows<PREC>(a, n, rows, e >= n_over, ln);
    }
  }
}

// The dense particles: every pair of their rows, row tile by row tile, each
// against all references or, where there are fewer row tiles than workgroups, a part
// of them: the contraction and inverse FFTs of k_corr, 64 pairs at a time with the
// rows' operand in registers.  16-bit forms read the operand of the bounds; FP32 makes
// that of the tile's rows in the workgroup's scratch tile first.  One workgroup of 8
// waves per CU (the state of 64 pairs takes 128 KiB of LDS), as many as CUs: a launch
// that finds none ends at once (about 5 us).  76 px, 100 references that are particles,
// +-3, 10 000 particles, whole call: FP32 171.7 ms with every pair in steps of 16,
// 34.9 here; BF16 165.5 and 28.5 (every pair in k_corr, without bounds: 43.8 and 24.4).
template <int PREC, class Contract, int MODE, class Items>
__global__ __launch_bounds__(512) void k_dense(Items it, FineDense dense) {
  extern __shared__ float smem[];
  const CorrSmem<8> sm(smem);
  constexpr int kList = PREC == kFP32 ? 1 : 0;
  const int cnt = dense.count[2 * kList];
  if (cnt == 0) return;
  const int parts = max(1, (int)gridDim.x / cnt), tid = threadIdx.x;
  for (int u = blockIdx.x; u < cnt * parts; u += gridDim.x) {
    const int2 at = dense.tile[kList][u % cnt];
    const FineArgs& a = it.piece(at.x);
    CorrArgs c = a.c;
    const int per = (c.n_ref_tiles + parts - 1) / parts, kt0 = u / cnt * per, kt1 = min(kt0 + per, c.n_ref_tiles);
    if (kt0 >= kt1) continue;
    const uint32_t rows = (dense_mask(c)[at.y] >> (8 * kList)) & 0xffu;
    c.rowkey = dense_rows(c);
    int a_tile = at.y;
    if constexpr (PREC == kFP32) {
      c.A += (size_t)blockIdx.x * a.scratch_floats;
      a_tile = 0;
      const int row0 = at.y * kRowTile;
      for (int n = row0 / c.S; n * c.S < min(row0 + kRowTile, c.rows); ++n) {
        const int first = max(n * c.S - row0, 0), last = min((n + 1) * c.S - row0, kRowTile);
        if (!((rows >> first) & 1u)) continue;
        const int S = c.S, s0 = row0 - n * S;
        fine_operand<Contract::LAYOUT == kRingPerm>(a, n, [=](int r) { return min(max(s0 + r, 0), S - 1); }, first, last,
                                                    smem, const_cast<float*>(c.A));
        __syncthreads();  // the tile is written and the work area free
      }
    }
    if (tid < kNphi) sm.tw[tid] = w256c(c.cs32, tid);
    Contract con;
    corr_tile<PREC, 8, Contract, MODE, true>(c, at.y, a_tile, rows, kt0, kt1, sm, con);
    __syncthreads();  // before the next unit's work area
  }
}

// A launch: one piece (a) or several (b).
struct FineLaunch {
  FineMode mode;
  int R4max;             // largest ring count of the pieces (one ring bucket)
  const FineArgs* a;
  const FineBatch* b;
  FineOver over;
  FineDense dense;
  int grid;
  size_t lds, work;      // LDS of the evaluation; of the FP32 operand's preparation
  hipStream_t st;
};

// The resident form of k_corr where there is one (FP32: up to 9 rings per lane group).
template <int PREC, int MAXR>
struct DenseContract {
  typedef typename std::conditional<
      PREC == kFP32, Fp32Contract<8, MAXR <= 9 ? 9 : 16, (MAXR <= 9), false>,
      Half16Contract<PREC == kFP32 ? kBF16 : PREC, 8, MAXR == 9 ? 10 : MAXR, true>>::type type;
};

template <int PREC, int MAXR, int MODE, class Items>
inline void fine_launch(const Items& it, const FineOver& over, const FineDense& dense, int grid, size_t lds, size_t work,
                        hipStream_t st) {
  const dim3 t(64 * fine_waves(PREC));
  auto go_dense = [&] {
    const size_t state = CorrSmem<8>::bytes();
    hipLaunchKernelGGL((k_dense<PREC, typename DenseContract<PREC, MAXR>::type, MODE, Items>), dim3(dense.grid), dim3(512),
                       state > work ? state : work, st, it, dense);
  };
  if constexpr (PREC == kFP32) go_dense();
  hipLaunchKernelGGL((k_fine<PREC, MAXR, MODE, Items>), dim3(grid), t, lds, st, it, over, dense);
  if constexpr (PREC != kFP32) {
    hipLaunchKernelGGL((k_fine_over<PREC, MAXR, MODE, Items>), dim3(over.grid), t, lds, st, it, over);
    go_dense();
    hipLaunchKernelGGL((k_fine_done<PREC, MODE, Items>), dim3(over.cap), dim3(MODE == kFineTighten ? 256 : 64), 0, st, it,
                       over, dense);
  }
}
template <int PREC, int MAXR, int MODE>
inline void fine_mode(const FineLaunch& f) {
  if (f.b) fine_launch<PREC, MAXR, MODE>(FineMany{*f.b}, f.over, f.dense, f.grid, f.lds, f.work, f.st);
  else fine_launch<PREC, MAXR, MODE>(FineOne{*f.a}, f.over, f.dense, f.grid, f.lds, f.work, f.st);
}
// TIGHTEN: only the tightening of FP32 bounds, else every other mode
template <int PREC, int MAXR, bool TIGHTEN>
inline void fine_go(const FineLaunch& f) {
  if constexpr (TIGHTEN) return fine_mode<PREC, MAXR, kFineTighten>(f);
  else if (f.mode == kFineRunnerUp) return fine_mode<PREC, MAXR, kRunnerUp>(f);
  else return fine_mode<PREC, MAXR, kArgmax>(f);
}

void fine_dispatch_fp32(const FineLaunch& f);
void fine_dispatch_bf16(const FineLaunch& f);
void fine_dispatch_fp16(const FineLaunch& f);
void fine_dispatch_tighten(const FineLaunch& f);

template <int PREC, bool TIGHTEN>
inline void fine_dispatch_16(const FineLaunch& f) {
  if (f.R4max <= 8) return fine_go<PREC, 8, TIGHTEN>(f);
  if (f.R4max <= 10) return fine_go<PREC, 10, TIGHTEN>(f);
  if (f.R4max <= 12) return fine_go<PREC, 12, TIGHTEN>(f);
  return fine_go<PREC, 16, TIGHTEN>(f);
}

}  // namespace mra
