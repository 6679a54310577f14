// Host side of libmra.so: contexts, resident reference sets, validation,
// chunk planning and the launch sequence of one MRA pass (Algorithm 1).
// Every entry point is extern "C", catches everything, and reports through
// an int status plus a per-context message (see include/mra.h).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "mra.h"
#include "mra_common.h"

using namespace mra;

namespace {

constexpr size_t kLdsMax = 160 * 1024;

// Device scratch of mra_align_noalloc (callers that cannot allocate): the
// per-chunk particle operand and row results live here instead of the
// context's workspace.  Each device holds its own copy for the life of the
// process; host code reaches it only through the address that
// hipGetSymbolAddress returns for the device (scratch_ptr), never through
// the symbol itself.
constexpr size_t kScratchBytes = 256ull << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

struct DevBuf {
  void* p = nullptr;
  size_t bytes = 0;
  bool keep = false;   // lives across the steps of the present call
};

struct Refset {
  mra_geom g{};
  int K = 0, R = 0, R4 = 0, NS = 0, n_kt = 0;
  float* B32 = nullptr;
  uint16_t* B16 = nullptr;  // the 16-bit forms' operand; FP32: the FP16 one of the bounds
  float* bnorm = nullptr;   // FP32: norm of each reference's operand
  float2* G1 = nullptr;    // K = 1: spectrum table of the fused single-reference kernel
  float* qhat = nullptr;
  double* norm = nullptr;
  Stencil* stencil = nullptr;
  float b_scale = 1.f;
  int dmin = 0, dmax = 0;  // range of stencil floor offsets
  int variant = 0;         // correlation kernel tile configuration
  int chunk = 0;           // particles per chunk (0: from the workspace cap)
  int prune = 1;           // evaluate only the pairs whose bound can win (0: every pair)
  int run_tiles = 0;       // accepted and reported, no longer used
};

struct Fail {
  int code;
  std::string msg;
};

}  // namespace

struct mra_ctx {
  int device = 0;
  hipStream_t stream = nullptr;
  uint64_t cap = 0;
  bool failed = false;
  std::string err;
  std::map<int32_t, Refset> refs;
  Refset spare;                  // buffers of a replaced refset, for the next load of its sizes
  mra::RefInfo* ref_info = nullptr;  // pinned
  double2* cs64 = nullptr;
  float2* cs32 = nullptr;
  std::map<std::string, DevBuf> ws;
  int n_cu = 256;
  void* scratch = nullptr; // this device's copy of the no-allocation scratch
  bool profiling = false;
  std::map<std::string, std::vector<std::pair<hipEvent_t, hipEvent_t>>> prof;
};

namespace {

void hip_check(mra_ctx* c, hipError_t e, const char* what) {
  if (e != hipSuccess) {
    c->failed = true;
    throw Fail{MRA_E_DEVICE, std::string(what) + ": " + hipGetErrorString(e)};
  }
}

// Address of the no-allocation scratch on c's device (current at the call):
// resolved once per device, kept for every later context on it.
void* scratch_ptr(mra_ctx* c) {
  if (c->device < 0 || c->device >= kMaxDevices) throw Fail{MRA_E_INVAL, "device ordinal out of range"};
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  void*& p = g_scratch_ptr[c->device];
  if (!p) {
    void* q = nullptr;
    hip_check(c, hipGetSymbolAddress(&q, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)");
    if (!q) throw Fail{MRA_E_DEVICE, "no device address for the scratch array"};
    p = q;
  }
  return p;
}

void free_refset(Refset& r) {
  for (void* p : {(void*)r.B32, (void*)r.B16, (void*)r.bnorm, (void*)r.G1, (void*)r.qhat, (void*)r.norm, (void*)r.stencil})
    if (p) (void)hipFree(p);
  r = Refset{};
}

void* alloc(mra_ctx* c, size_t bytes, const char* what) {
  void* p = nullptr;
  hipError_t e = hipMalloc(&p, bytes < 16 ? 16 : bytes);
  if (e == hipErrorOutOfMemory && c->spare.stencil) {  // a replaced refset's buffers are given back first
    (void)hipGetLastError();
    hip_check(c, hipStreamSynchronize(c->stream), "sync");
    free_refset(c->spare);
    e = hipMalloc(&p, bytes < 16 ? 16 : bytes);
  }
  if (e == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    throw Fail{MRA_E_NOMEM, std::string("out of device memory allocating ") + what};
  }
  hip_check(c, e, what);
  return p;
}

// A workspace buffer, grown on demand.
void* ws_get(mra_ctx* c, const std::string& name, size_t bytes, bool keep = false) {
  DevBuf& b = c->ws[name];
  b.keep = keep;
  if (b.bytes < bytes) {
    uint64_t total = bytes;  // the workspace after this buffer grows
    for (const auto& kv : c->ws)
      if (&kv.second != &b) total += kv.second.bytes;
    if (total > c->cap)
      throw Fail{MRA_E_NOMEM, "workspace cap of " + std::to_string(c->cap) + " bytes is too small (" + name +
                                  " needs " + std::to_string(bytes) + " bytes)"};
    if (b.p) hip_check(c, hipFree(b.p), "hipFree");
    b.p = nullptr;
    b.bytes = 0;
    b.p = alloc(c, bytes, name.c_str());
    b.bytes = bytes;
  }
  return b.p;
}

// Before a step (a reference preparation, an alignment chunk, a batched wave, an
// average update) takes the buffers `need`: buffers stay for later steps as long as
// the cap has room; where it has not, all but the kept ones are given back, so that
// a step that fits the cap by itself is never refused for what others left.
typedef std::vector<std::pair<std::string, size_t>> WsNeed;
void ws_step(mra_ctx* c, const WsNeed& need) {
  uint64_t total = 0;  // the workspace with the step's buffers grown
  for (const auto& kv : c->ws) total += kv.second.bytes;
  for (const auto& n : need) {
    const auto it = c->ws.find(n.first);
    const size_t have = it == c->ws.end() ? 0 : it->second.bytes;
    if (n.second > have) total += n.second - have;
  }
  if (total <= c->cap) return;
  hip_check(c, hipStreamSynchronize(c->stream), "sync");
  for (auto& kv : c->ws) {
    if (kv.second.keep || !kv.second.p) continue;
    hip_check(c, hipFree(kv.second.p), "hipFree");
    kv.second = DevBuf{};
  }
}

// Workspace that no step gives back.
uint64_t ws_kept(const mra_ctx* c) {
  uint64_t total = 0;
  for (const auto& kv : c->ws)
    if (kv.second.keep) total += kv.second.bytes;
  return total;
}

// Runs `launch` between two events on the context stream when profiling.
template <class F>
void timed(mra_ctx* c, const char* group, F&& launch) {
  if (!c->profiling) {
    launch();
    return;
  }
  hipEvent_t a, b;
  hip_check(c, hipEventCreate(&a), "hipEventCreate");
  hip_check(c, hipEventCreate(&b), "hipEventCreate");
  hip_check(c, hipEventRecord(a, c->stream), "hipEventRecord");
  launch();
  hip_check(c, hipEventRecord(b, c->stream), "hipEventRecord");
  c->prof[group].emplace_back(a, b);
}

void clear_profile(mra_ctx* c) {
  for (auto& kv : c->prof)
    for (auto& e : kv.second) {
      (void)hipEventDestroy(e.first);
      (void)hipEventDestroy(e.second);
    }
  c->prof.clear();
}

// cos / sin of 2 pi j / n built from the first octant so that the table is
// exactly symmetric (cos even, sin odd, quarter turns exact).
void build_cs(int n, std::vector<double>& c, std::vector<double>& s) {
  c.assign(n, 0.0);
  s.assign(n, 0.0);
  const double two_pi = 6.283185307179586476925286766559;
  const int q = n / 4, e = n / 8;
  std::vector<double> c0(q + 1), s0(q + 1);
  for (int j = 0; j <= e; ++j) {
    c0[j] = std::cos(two_pi * j / n);
    s0[j] = std::sin(two_pi * j / n);
  }
  for (int j = e + 1; j <= q; ++j) {
    c0[j] = s0[q - j];
    s0[j] = c0[q - j];
  }
  for (int j = 0; j < n; ++j) {
    int jj = j, sc = 1, ss = 1;
    if (jj > n / 2) { jj = n - jj; ss = -1; }          // theta -> -theta
    if (jj > q) { jj = n / 2 - jj; sc = -1; }          // theta -> pi - theta
    c[j] = sc * c0[jj];
    s[j] = ss * s0[jj];
  }
}

void check_geom(const mra_geom* g) {
  auto bad = [](const char* m) { throw Fail{MRA_E_INVAL, m}; };
  if (!g) bad("geometry is NULL");
  if (g->L < 8 || g->L > 160) bad("L must be in [8, 160]");
  if (g->r_min < 1 || g->r_max < g->r_min || g->r_max > 64) bad("need 1 <= r_min <= r_max <= 64");
  if (g->n_phi != kNphi) bad("n_phi must be 256 (the only angular sampling the kernels implement)");
  if (g->shift_max < 0 || g->shift_max > 8) bad("shift_max must be in [0, 8]");
  if (g->mirror != 0 && g->mirror != 1) bad("mirror must be 0 or 1");
  if (g->precision < 0 || g->precision > 2) bad("precision must be MRA_FP32, MRA_BF16 or MRA_FP16");
  if (g->normalize != 0 && g->normalize != 1) bad("normalize must be 0 or 1");
  if (g->rescore_rows < 0 || g->rescore_rows > 8) bad("rescore_rows must be in [0, 8]");
}

// The flat candidate index iota = (((k M + m) S1 + sy) S1 + sx) n_phi + a is
// an int32 in every kernel and 0x7fffffff marks "no candidate", so
// K * M * S * n_phi must stay below 2^31.
void check_index_range(int64_t K, int M, int T) {
  const int64_t S1 = 2 * (int64_t)T + 1;
  if (K * M * S1 * S1 * kNphi > (int64_t)INT32_MAX)
    throw Fail{MRA_E_INVAL, "K * mirrors * (2 shift_max + 1)^2 * n_phi must be below 2^31 (int32 candidate index); "
                            "split the references into several refsets"};
}

Refset& get_refset(mra_ctx* c, int32_t id) {
  auto it = c->refs.find(id);
  if (it == c->refs.end()) throw Fail{MRA_E_NOREF, "refset " + std::to_string(id) + " is not loaded"};
  return it->second;
}

struct Plan {
  int T, S1, S, M, pad, Lp, cx;
  int lo, hi;       // lowest and highest pixel index the single-precision resamplers touch
  int pad_r, Lp_r;  // border and side for the kernels that sample with the FP64 stencil table
};

Plan plan_for(const Refset& rs, int T) {
  if (T < 0 || T > 8) throw Fail{MRA_E_INVAL, "shift_max must be in [0, 8]"};
  check_index_range(rs.K, rs.g.mirror ? 2 : 1, T);
  Plan p;
  p.T = T;
  p.S1 = 2 * T + 1;
  p.S = p.S1 * p.S1;
  p.M = rs.g.mirror ? 2 : 1;
  p.cx = rs.g.L / 2;
  // lowest and highest pixel index touched; the resamplers that take the
  // floor of single-precision positions reach one pixel further either side
  const int lo = p.cx - T + rs.dmin;
  const int hi = p.cx + T + rs.dmax + 1;
  p.pad_r = std::max(0, std::max(-lo, hi - (rs.g.L - 1)));
  p.Lp_r = rs.g.L + 2 * p.pad_r;
  p.lo = lo - 1;
  p.hi = hi + 1;
  p.pad = std::max(0, std::max(-p.lo, p.hi - (rs.g.L - 1)));
  p.Lp = rs.g.L + 2 * p.pad;
  if (polar_lds_bytes(p.Lp) > kLdsMax)
    throw Fail{MRA_E_INVAL, "box plus search range too large for the LDS-staged resampler"};
  return p;
}

void check_result(const mra_result* r) {
  if (!r || !r->ref || !r->shift_x || !r->shift_y || !r->psi || !r->mirror || !r->cc)
    throw Fail{MRA_E_INVAL, "result arrays must be non-NULL (cc2, flat_index may be NULL)"};
}

// The two ways through a chunk.  Pruned: the 16-bit operand of every row
// (FP16 for FP32 alignment), a bound of every (row, reference) pair, then the
// evaluation of the pairs that can win; FP32 makes the FP32 operand of the
// rows it evaluates in a scratch tile per workgroup.  Unpruned (prune = 0, the
// debug CC table, or a workspace too small for the bounds): the operand of
// every row in the contraction's own type, every pair evaluated.
int operand_layout(const Refset& rs, bool pruned) {
  return pruned ? (int)kRingPerm16 : a_layout_for(rs.g.precision, rs.variant);
}
size_t tile_bytes_of(const Refset& rs, bool pruned) {
  return (size_t)kSlots * rs.R4 * 64 * a_elem_bytes(operand_layout(rs, pruned));
}
size_t scratch_tile_bytes(const Refset& rs) { return (size_t)kSlots * rs.R4 * 64 * sizeof(float); }
int ub_pitch(const Refset& rs) { return rs.n_kt * kRefTile; }
// the operand's FP16 scale is kept per particle
bool scaled_operand(const Refset& rs, bool pruned) {
  return rs.g.precision == kFP16 || (pruned && rs.g.precision == kFP32);
}
// row results are written out for the re-ranking
bool row_results(const Refset& rs) { return rs.g.precision != kFP32 && rs.g.rescore_rows >= 2; }

// Device buffers of one alignment chunk of nc particles.
struct ChunkBufs {
  float* A = nullptr;        // particle operand, ceil(nc S / 8) row tiles
  float* ub = nullptr;       // pruned: [nc S][ub_pitch] bounds
  float* ub_hi = nullptr;    // pruned: a half of them before they are added
  unsigned long long* rowkey = nullptr;  // [nc S] largest bound (pruned; then dense_rows, dense_mask) or best CC per row
  float* rownorm = nullptr;  // pruned FP32: [2][nc S] norm of the row's operand
  float* scratch = nullptr;  // pruned FP32: one operand tile per evaluation workgroup
  int grid = 0;              // evaluation workgroups
  FineOver over{};           // the particles left to the whole chip
  FineDense dense{};         // those of which every pair is evaluated
  float* rcc = nullptr;      // [nc S] best CC per row
  int* ridx = nullptr;       // [nc S] its flat index
  float* maxabs = nullptr;   // FP16 operand: [nc] max |pixel|
  int32_t* win = nullptr;    // cc2: [nc] chunk-local winner copy
};

// The lists of particles that an evaluation of nc particles (of at most S shifts
// and `units` units of work each, in `tiles` row tiles) leaves to the whole chip,
// and of those whose every pair is evaluated (their launch: dense.grid, set here).
template <class Take>
void take_lists(int64_t nc, size_t tiles, int S, int units, int n_cu, FineOver& o, FineDense& d, Take take) {
  o.cap = (int)std::min<int64_t>(nc, kFineOverCap);
  o.steps = fine_over_steps(nc, units, n_cu);
  o.pitch = S;
  o.units = units;
  o.grid = fine_grid(kFP16, INT32_MAX, n_cu);
  const size_t keys = (size_t)o.cap * (1 + S) * sizeof(unsigned long long), dtile = 2 * tiles * sizeof(int2);
  char* p = (char*)take("over", keys + dtile + (size_t)(kFineCounts + o.cap + 2 * nc) * sizeof(int));
  if (!p) return;  // (only measured)
  o.best = (unsigned long long*)p;
  o.row = o.best + o.cap;
  d.tile[0] = (int2*)(p + keys);
  d.tile[1] = d.tile[0] + tiles;
  o.count = (int*)(p + keys + dtile);
  d.count = o.count + 2;
  o.item = o.count + kFineCounts;
  d.item[0] = o.item + o.cap;
  d.item[1] = d.item[0] + nc;
}

// Workgroups of the evaluation of every pair of a launch's dense particles, one per
// CU (FP32: each with a scratch tile; few particles, fewer tiles).
int dense_grid(int prec, int grid, int n_cu) { return prec == kFP32 ? std::min(n_cu, 2 * grid) : n_cu; }

// Calls take(name, bytes) for every buffer of an nc-particle chunk.
template <class Take>
ChunkBufs layout_chunk(const Refset& rs, const Plan& p, int64_t nc, bool pruned, bool cc2, int n_cu, Take take) {
  ChunkBufs b;
  const size_t rows = (size_t)nc * p.S;
  const size_t tiles = (rows + kRowTile - 1) / kRowTile;
  b.A = (float*)take("A", tiles * tile_bytes_of(rs, pruned));
  if (pruned) {
    b.grid = fine_grid(rs.g.precision, nc, n_cu);
    b.ub = (float*)take("ub", rows * ub_pitch(rs) * sizeof(float));
    b.ub_hi = (float*)take("ub_hi", rows * ub_pitch(rs) * sizeof(float));
    b.dense.grid = dense_grid(rs.g.precision, b.grid, n_cu);
    if (rs.g.precision == kFP32) {
      b.rownorm = (float*)take("rownorm", 2 * rows * sizeof(float));
      b.scratch = (float*)take("scratch", std::max(b.grid, b.dense.grid) * scratch_tile_bytes(rs));
    }
    take_lists(nc, tiles, p.S, fine_units(p.S, rs.K), n_cu, b.over, b.dense, take);
  }
  b.rowkey = (unsigned long long*)take("rowkey", rowkey_bytes(rows, pruned));
  if (row_results(rs)) {
    b.rcc = (float*)take("row_cc", rows * sizeof(float));
    b.ridx = (int*)take("row_idx", rows * sizeof(int));
  }
  if (scaled_operand(rs, pruned)) b.maxabs = (float*)take("maxabs", (size_t)nc * sizeof(float));
  if (cc2) b.win = (int32_t*)take("win", (size_t)nc * sizeof(int32_t));
  return b;
}

// Lays the buffers of an nc-particle chunk out from `base` (256-byte
// aligned pieces); returns the bytes used.  base = nullptr only measures.
size_t carve_chunk(const Refset& rs, const Plan& p, int64_t nc, bool pruned, bool cc2, int n_cu, char* base,
                   ChunkBufs* b) {
  size_t off = 0;
  const ChunkBufs got = layout_chunk(rs, p, nc, pruned, cc2, n_cu, [&](const char*, size_t bytes) -> void* {
    char* q = base ? base + off : nullptr;
    off += (bytes + 255) & ~(size_t)255;
    return q;
  });
  if (b) *b = got;
  return off;
}

// Buffers of a chunk from the context's workspace (grown on demand).
ChunkBufs ws_chunk(mra_ctx* c, const Refset& rs, const Plan& p, int64_t nc, bool pruned, const mra_result* out) {
  WsNeed need;
  layout_chunk(rs, p, nc, pruned, out && out->cc2, c->n_cu, [&](const char* name, size_t bytes) -> void* {
    need.emplace_back(name, bytes);
    return nullptr;
  });
  ws_step(c, need);
  return layout_chunk(rs, p, nc, pruned, out && out->cc2, c->n_cu,
                      [&](const char* name, size_t bytes) { return ws_get(c, name, bytes); });
}

// bytes of operand and bounds per particle
uint64_t particle_bytes(const Refset& rs, const Plan& p, bool pruned) {
  const uint64_t row = tile_bytes_of(rs, pruned) / kRowTile + (pruned ? 2 * ub_pitch(rs) * sizeof(float) : 0);
  return (uint64_t)p.S * row;
}

int64_t chunk_particles(mra_ctx* c, const Refset& rs, const Plan& p, bool pruned) {
  if (rs.chunk > 0) return rs.chunk;
  const uint64_t budget = c->cap / 2;
  return std::max<int64_t>(1, (int64_t)(budget / particle_bytes(rs, p, pruned)));
}

// Tile pairs (of 8 rows and 8 references) that cost what a particle's bounds and its steps of
// evaluation do.  (The more rings, the shorter those steps are beside a tile pair: fewer pairs
// stay live.  Up to 12 rings the bounds' own contraction is short; FP32 from 37 rings on,
// a tile pair's operand is streamed; with the runner-up every pair is evaluated twice.)
int particle_tiles(const Refset& rs, const Plan& p, bool cc2) {
  if (rs.g.precision == kFP32) return cc2 ? 2 : (rs.R4 <= 9 ? 4 : 1);
  if (cc2) return 2;
  return p.S <= 9 ? 3 : (rs.R4 > 3 && rs.R4 <= 7 ? 12 : 5);
}

// Few pairs per particle, at any number of particles.  In 16 bits one or two reference tiles
// are, up to +-3: on particles of these references the two ways take about the same, on
// others', which keep more pairs live, the bounds take longer (4000 particles, 10
// references, bounds / every pair, ms, of these references and of 80: BF16 64 px, +-2 1.74 /
// 1.65 and 2.11 / 1.64; 90 px, 36 rings, +-3 3.20 / 3.52 and 4.43 / 3.74; 100 000 particles of
// 200: 109 / 90; FP32 146 / 147; with the runner-up 3.88 / 5.24; 24 px, 9 rings, +-2: 0.77 /
// 1.01).  Without shifts a step holds at most 8 pairs, of one row: 64 px, 5000
// references, 2000 particles FP32 8.0 / 6.5 ms, BF16 6.7 / 4.3.
bool few_each(const Refset& rs, const Plan& p, bool cc2) {
  const int pairs = p.S * rs.n_kt;
  return p.S == 1 || pairs <= particle_tiles(rs, p, cc2) * kRowTile ||
         (rs.g.precision != kFP32 && rs.R4 > 3 && !cc2 && rs.n_kt <= 2 && pairs <= 100);
}

// A call of few pairs, or of few pairs per particle, takes the unpruned way: with
// every pair of a few row and reference tiles spread over the CUs it ends before the
// pruned way's chain of dependent steps does.  The lines were fitted to 4000 calls drawn over
// boxes of 40 to 128 px, rings out to a third of the box up to all of it, +-1 to +-5, 5 to 300
// references, SNR 0.05 and 0.1, particles of these references and (30 %) of others, 4 to
// 250 tile pairs per CU (2 to 3 % above the faster way on the former, 5 on the latter), and
// checked on 3000 with rings out to the box (1 to 2 %).  Fewer rings leave more pairs live
// (and, FP32, a tile pair costs less).  Pruned over unpruned, geometric means at 8 to
// 16, 32 to 64 and 128 to 260 tile pairs per CU: FP32 17 to 20 rings 2.4, 1.3, 0.92; 25 to
// 28: 1.7, 0.93, 0.70; 33 to 36: 1.3, 0.75, 0.60; 45 to 48: 0.83, 0.46, 0.36; 16 bits 17 to 20
// rings 1.8, 1.2, 1.1; 25 to 28: 1.4, 1.1, 0.80; 33 to 36: 1.2, 0.99, 0.75.  (Up to 12 rings:
// 24 px, 9 rings, 100 references, 600 particles, 95 tile pairs per CU: FP32 1.1, BF16 0.54.)
bool few_tiles(const mra_ctx* c, const Refset& rs, const Plan& p, int64_t tiles, int64_t N, bool cc2) {
  const int cube = rs.R4 * rs.R4 * rs.R4;
  const int per_cu = rs.g.precision == kFP32
                         ? (cc2 ? std::clamp(5500 / cube, 4, 150) : std::clamp(10000 / cube, 8, 150))
                         : (rs.R4 <= 3 ? 20 : (cc2 ? std::clamp(7000 / cube, 12, 150) : std::clamp(20000 / cube, 20, 150)));
  return tiles <= per_cu * (int64_t)c->n_cu + particle_tiles(rs, p, cc2) * N;
}

int64_t tile_pairs(const Refset& rs, const Plan& p, int64_t N) { return (N * p.S + kRowTile - 1) / kRowTile * rs.n_kt; }

bool few_pairs(const mra_ctx* c, const Refset& rs, const Plan& p, int64_t N, bool cc2) {
  return few_each(rs, p, cc2) || few_tiles(c, rs, p, tile_pairs(rs, p, N), N, cc2);
}

// Largest chunk of at most N particles whose buffers fit `bytes` (0 if not one particle).
int64_t fitting_chunk(const Refset& rs, const Plan& p, int64_t N, bool pruned, bool cc2, int n_cu, size_t bytes) {
  const int64_t most = std::min<int64_t>(INT32_MAX / p.S / 2, N);
  if (carve_chunk(rs, p, most, pruned, cc2, n_cu, nullptr, nullptr) <= bytes) return most;
  if (carve_chunk(rs, p, 1, pruned, cc2, n_cu, nullptr, nullptr) > bytes) return 0;
  // the buffers grow with the chunk: bisect for the largest that fits
  int64_t lo = 1, hi = most;
  while (lo < hi) {
    const int64_t mid = lo + (hi - lo + 1) / 2;
    if (carve_chunk(rs, p, mid, pruned, cc2, n_cu, nullptr, nullptr) <= bytes) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Particles per chunk on the pruned path, or 0 when a chunk is of few pairs or not one
// particle's bounds and scratch fit (the call then takes the unpruned one).  All that a chunk holds
// takes at most half the cap, as the unpruned operand does: the other half is left
// to the steps beside it (reference preparation, averages).
int64_t pruned_chunk(mra_ctx* c, const Refset& rs, const Plan& p, int64_t N, bool cc2) {
  if (!rs.prune || few_pairs(c, rs, p, N, cc2)) return 0;
  const int64_t most = std::min<int64_t>(INT32_MAX / p.S / 2, N);
  const uint64_t room = c->cap - std::min(c->cap, ws_kept(c));
  int64_t n = std::min<int64_t>(rs.chunk, most);
  if (rs.chunk <= 0) n = fitting_chunk(rs, p, N, true, cc2, c->n_cu, std::min(c->cap / 2, room));
  else
    while (n > 0 && carve_chunk(rs, p, n, true, cc2, c->n_cu, nullptr, nullptr) > room) n /= 2;
  return few_pairs(c, rs, p, n, cc2) ? 0 : n;
}

// Sub-step angles of particles n0 .. n0 + nc - 1 from their final parameters.
void refine_chunk(mra_ctx* c, const Refset& rs, const Plan& p, const float* parts, int64_t n0, int64_t nc,
                  const mra_result* out) {
  const int L = rs.g.L;
  const int64_t step = INT32_MAX / 2;
  for (int64_t o = 0; o < nc; o += step) {
    RescoreArgs ra{};
    ra.parts = parts + (size_t)(n0 + o) * L * L;
    ra.n_part = (int)std::min<int64_t>(step, nc - o);
    ra.out_off = n0 + o;
    ra.L = L; ra.R = rs.R; ra.r_min = rs.g.r_min; ra.Lp = p.Lp_r; ra.pad = p.pad_r; ra.cx = p.cx;
    ra.K = rs.K; ra.T = p.T;
    ra.stencil = rs.stencil;
    ra.qhat = rs.qhat;
    ra.ref = out->ref; ra.shift_x = out->shift_x; ra.shift_y = out->shift_y;
    ra.psi = out->psi; ra.mirror = out->mirror;
    ra.psi_frac = out->psi_frac;
    timed(c, "refine", [&] { hip_check(c, launch_refine(ra, c->stream), "refine"); });
  }
}

// Arguments of the launches over particles n0 .. n0 + nc - 1 of a stack.
PolarArgs polar_args(mra_ctx* c, const Refset& rs, const Plan& p, const float* src, int nc) {
  PolarArgs pa{};
  pa.parts = src;
  pa.n_part = nc;
  pa.L = rs.g.L; pa.R = rs.R; pa.R4 = rs.R4; pa.T = p.T; pa.S1 = p.S1; pa.S = p.S;
  pa.cx = p.cx;
  polar_window(pa, p.lo, p.hi);
  pa.r_min = rs.g.r_min;
  pa.prec = rs.g.precision;
  pa.cs64 = c->cs64;
  // (a particle's rows touch up to S / 8 + 1 row groups)
  pa.split = polar_split(nc, rs.R * (p.S / kRowTile + 1), c->n_cu, polar_waves(pa));
  return pa;
}

CorrArgs corr_args(mra_ctx* c, const Refset& rs, const Plan& p, int nc, int layout, const ChunkBufs& b) {
  CorrArgs ca{};
  ca.A = b.A;
  ca.a_layout = layout;
  ca.rows = nc * p.S;
  ca.n_row_tiles = (ca.rows + kRowTile - 1) / kRowTile;
  ca.B32 = rs.B32;
  ca.B16 = rs.B16;
  ca.R = rs.R; ca.R4 = rs.R4; ca.n_ref_tiles = rs.n_kt;
  ca.K = rs.K; ca.S = p.S; ca.M = p.M;
  ca.maxabs = b.maxabs;
  ca.b_scale = rs.b_scale;
  ca.bnorm = rs.bnorm;
  ca.cs32 = c->cs32;
  ca.row_cc = b.rcc;
  ca.row_idx = b.ridx;
  ca.ub = b.ub;
  ca.ub_hi = b.ub_hi;
  ca.rowkey = b.rowkey;
  ca.rownorm = b.rownorm;
  ca.ldu = ub_pitch(rs);
  return ca;
}

ResultArgs result_args(const Plan& p, int64_t n0, int nc, const mra_result* out, const ChunkBufs& b) {
  ResultArgs ra{};
  ra.n_part = nc; ra.S = p.S; ra.S1 = p.S1; ra.T = p.T; ra.M = p.M;
  ra.out_off = n0;
  ra.ref = out->ref; ra.shift_x = out->shift_x; ra.shift_y = out->shift_y;
  ra.psi = out->psi; ra.mirror = out->mirror; ra.flat = out->flat_index;
  ra.cc = out->cc; ra.cc2 = out->cc2;
  ra.win = out->cc2 ? b.win : nullptr;
  return ra;
}

RescoreArgs rescore_args(const Refset& rs, const Plan& p, const float* src, int64_t n0, int nc,
                         const mra_result* out, const ChunkBufs& b) {
  RescoreArgs ra{};
  ra.parts = src;
  ra.n_part = nc;
  ra.out_off = n0;
  ra.L = rs.g.L; ra.R = rs.R; ra.r_min = rs.g.r_min; ra.Lp = p.Lp_r; ra.pad = p.pad_r; ra.cx = p.cx;
  ra.K = rs.K; ra.T = p.T;
  ra.stencil = rs.stencil;
  ra.qhat = rs.qhat;
  ra.ref = out->ref; ra.shift_x = out->shift_x; ra.shift_y = out->shift_y;
  ra.psi = out->psi; ra.mirror = out->mirror;
  ra.cc = out->cc;
  ra.rows = rs.g.rescore_rows;
  ra.margin = rerank_margin(rs.g.precision);
  ra.S1 = p.S1; ra.S = p.S; ra.M = p.M;
  ra.row_cc = b.rcc; ra.row_idx = b.ridx;
  ra.ref_w = out->ref; ra.shift_x_w = out->shift_x; ra.shift_y_w = out->shift_y;
  ra.psi_w = out->psi; ra.mirror_w = out->mirror; ra.flat_w = out->flat_index;
  ra.win = out->cc2 ? b.win : nullptr;
  return ra;
}

// Merge of a chunk's rows, every pair evaluated.
MergeArgs merge_args(const Refset& rs, const Plan& p, int64_t n0, int nc, const mra_result* out, const ChunkBufs& b) {
  MergeArgs ma{};
  ma.r = result_args(p, n0, nc, out, b);
  ma.rowkey = b.rowkey;
  ma.maxabs = rs.g.precision == kFP16 ? b.maxabs : nullptr;
  ma.b_scale = rs.b_scale;
  ma.row_cc = b.rcc;
  ma.row_idx = b.ridx;
  return ma;
}

// Evaluation of a chunk from its operand and bounds (ca, with b's buffers).
FineArgs fine_args(mra_ctx* c, const Refset& rs, const Plan& p, const CorrArgs& ca, const float* src, int64_t n0,
                   int nc, const mra_result* out, const ChunkBufs& b) {
  FineArgs fa{};
  fa.c = ca;
  if (rs.g.precision == kFP32) {
    fa.c.A = b.scratch;
    fa.scratch_floats = (int)(scratch_tile_bytes(rs) / sizeof(float));
  }
  fa.m = result_args(p, n0, nc, out, b);
  fa.margin = rs.g.rescore_rows >= 2 ? rerank_margin(rs.g.precision) : 0.f;
  fa.parts = src;
  fa.L = rs.g.L; fa.Lp = p.Lp; fa.pad = p.pad; fa.cx = p.cx; fa.r_min = rs.g.r_min;
  fa.cs64 = c->cs64;
  return fa;
}

// One chunk of the alignment pass, pruned: resample + FFT -> bounds ->
// evaluation (-> FP32 re-score for 16-bit contractions).
void run_chunk(mra_ctx* c, const Refset& rs, const Plan& p, const float* parts, int64_t n0, int nc,
               const mra_result* out, const ChunkBufs& b) {
  hipStream_t st = c->stream;
  const int prec = rs.g.precision;
  const float* src = parts + (size_t)n0 * rs.g.L * rs.g.L;
  PolarArgs pa = polar_args(c, rs, p, src, nc);
  pa.a_layout = kRingPerm16;
  pa.maxabs = b.maxabs;
  pa.out = b.A;
  timed(c, "polar", [&] { hip_check(c, launch_polar(0, pa, st), "polar"); });
  CorrArgs ca = corr_args(c, rs, p, nc, kRingPerm16, b);
  const int items = bound_items(ca, c->n_cu);
  timed(c, "bound", [&] { hip_check(c, launch_bound(prec, ca, items, b.over.count, st), "bound"); });
  FineArgs fa = fine_args(c, rs, p, ca, src, n0, nc, out, b);
  if (prec == kFP32) {
    FineArgs ta = fa;
    ta.c.A = b.A;
    timed(c, "tighten", [&] {
      hip_check(c, launch_fine(prec, kFineTighten, ta, b.over, b.dense, fine_grid(kFP16, nc, c->n_cu), st), "tighten");
    });
  }
  FineOver over = prec == kFP32 ? FineOver{} : b.over;
  timed(c, "fine", [&] { hip_check(c, launch_fine(prec, kFineArgmax, fa, over, b.dense, b.grid, st), "fine"); });
  if (prec != kFP32)
    timed(c, "rescore", [&] { hip_check(c, launch_rescore(rescore_args(rs, p, src, n0, nc, out, b), st), "rescore"); });
  if (out->cc2) {
    // runner-up: the same bounds, the best over every candidate but the winner
    fa.c.excl = b.win;
    fa.c.row_cc = nullptr;
    fa.m.win = nullptr;
    fa.m.runner_up = 1;
    fa.margin = 0.f;
    if (over.cap) over.count += 1;
    timed(c, "fine2", [&] { hip_check(c, launch_fine(prec, kFineRunnerUp, fa, over, b.dense, b.grid, st), "fine2"); });
  }
  if (out->psi_frac) refine_chunk(c, rs, p, parts, n0, nc, out);
}

// One chunk with every pair evaluated: resample + FFT -> correlation ->
// merge (-> FP32 re-score); table != nullptr: the debug CC table only.
void run_chunk_unpruned(mra_ctx* c, const Refset& rs, const Plan& p, const float* parts, int64_t n0, int nc,
                        const mra_result* out, float* table, const ChunkBufs& b) {
  hipStream_t st = c->stream;
  const int prec = rs.g.precision;
  const float* src = parts + (size_t)n0 * rs.g.L * rs.g.L;
  // (the CC table is written by the form launch_corr picks for it)
  const int layout = a_layout_for(prec, table ? (prec == kFP32 ? 2 : 0) : rs.variant);
  CorrArgs ca = corr_args(c, rs, p, nc, layout, b);
  // rows past the chunk in its last tile are read as zeros
  const size_t tile_bytes = tile_bytes_of(rs, false);
  if (ca.rows % kRowTile)
    hip_check(c, launch_fill_zero((char*)b.A + (size_t)(ca.n_row_tiles - 1) * tile_bytes, tile_bytes, st), "fill");
  PolarArgs pa = polar_args(c, rs, p, src, nc);
  pa.a_layout = layout;
  pa.maxabs = b.maxabs;
  pa.rowkey = b.rowkey;
  pa.out = b.A;
  timed(c, "polar", [&] { hip_check(c, launch_polar(0, pa, st), "polar"); });
  ca.table = table;
  ca.kt_per_wg = corr_tiles_per_wg(ca.n_row_tiles, rs.n_kt, c->n_cu);
  timed(c, "corr", [&] { hip_check(c, launch_corr(prec, rs.variant, table != nullptr, ca, st), "corr"); });
  if (table) return;
  MergeArgs ma = merge_args(rs, p, n0, nc, out, b);
  timed(c, "merge", [&] { hip_check(c, launch_merge(ma, st), "merge"); });
  if (prec != kFP32)
    timed(c, "rescore", [&] { hip_check(c, launch_rescore(rescore_args(rs, p, src, n0, nc, out, b), st), "rescore"); });
  if (out->cc2) {
    // runner-up: the same contraction with each particle's winner left out;
    // the best that remains is the best over every other candidate
    ca.excl = b.win;
    const size_t key_bytes = ((size_t)ca.rows * sizeof(unsigned long long) + 15) & ~(size_t)15;
    hip_check(c, launch_fill_zero(b.rowkey, key_bytes, st), "fill");
    timed(c, "corr2", [&] { hip_check(c, launch_corr_runner_up(prec, rs.variant, ca, st), "corr2"); });
    ma.r.win = nullptr;
    ma.row_cc = nullptr;
    ma.r.runner_up = 1;
    timed(c, "merge", [&] { hip_check(c, launch_merge(ma, st), "merge"); });
  }
  if (out->psi_frac) refine_chunk(c, rs, p, parts, n0, nc, out);
}

// One reference (K = 1): the fused single-reference kernel over the whole
// stack; it needs no workspace.
void run_single(mra_ctx* c, const Refset& rs, const Plan& p, const float* parts, int64_t N, const mra_result* out) {
  const int L = rs.g.L;
  const int64_t step = INT32_MAX / 2;
  for (int64_t n0 = 0; n0 < N; n0 += step) {
    RfaArgs ra{};
    ra.parts = parts + (size_t)n0 * L * L;
    ra.n_part = (int)std::min<int64_t>(step, N - n0);
    ra.out_off = n0;
    ra.L = L; ra.R = rs.R; ra.T = p.T; ra.S1 = p.S1; ra.S = p.S; ra.M = p.M;
    ra.Lp = p.Lp; ra.pad = p.pad; ra.cx = p.cx; ra.r_min = rs.g.r_min;
    ra.stencil = rs.stencil;
    ra.cs64 = c->cs64;
    ra.G = rs.G1;
    ra.ref = out->ref; ra.shift_x = out->shift_x; ra.shift_y = out->shift_y;
    ra.psi = out->psi; ra.mirror = out->mirror; ra.flat = out->flat_index;
    ra.cc = out->cc; ra.cc2 = out->cc2;
    timed(c, "rfa", [&] { hip_check(c, launch_rfa(ra, c->stream), "rfa"); });
  }
  if (out->psi_frac) refine_chunk(c, rs, p, parts, 0, N, out);
}

// Particles first .. first + N - 1 of a stack chunk by chunk, in the context's workspace.
void align_stack(mra_ctx* c, const Refset& rs, const Plan& p, const float* parts, int64_t first, int64_t N,
                 const mra_result* out, float* table) {
  int64_t step = table ? 0 : pruned_chunk(c, rs, p, N, out->cc2 != nullptr);
  const bool pruned = step > 0;
  if (!pruned) step = std::min<int64_t>(chunk_particles(c, rs, p, false), (int64_t)(INT32_MAX / p.S / 2));
  for (int64_t n0 = first; n0 < first + N; n0 += step) {
    const int nc = (int)std::min<int64_t>(step, first + N - n0);
    const ChunkBufs b = ws_chunk(c, rs, p, nc, pruned, out);
    if (pruned)
      run_chunk(c, rs, p, parts, n0, nc, out, b);
    else
      run_chunk_unpruned(c, rs, p, parts, n0, nc, out,
                         table ? table + (size_t)n0 * rs.K * p.M * p.S * kNphi : nullptr, b);
  }
}

// noalloc: the chunk buffers come from the device scratch array instead of
// the workspace, so nothing is allocated (the path of mra_align_noalloc).
void align_impl(mra_ctx* c, int32_t id, const float* parts, int64_t N, int T, const mra_result* out,
                float* table, bool noalloc = false) {
  Refset& rs = get_refset(c, id);
  if (N < 0) throw Fail{MRA_E_INVAL, "N must be >= 0"};
  if (N == 0) return;
  if (!parts) throw Fail{MRA_E_INVAL, "parts is NULL"};
  if (!table) check_result(out);
  const Plan p = plan_for(rs, T < 0 ? rs.g.shift_max : T);
  if (rs.K == 1 && !table) {
    run_single(c, rs, p, parts, N, out);
    return;
  }
  if (!noalloc) {
    align_stack(c, rs, p, parts, 0, N, out, table);
    return;
  }
  if (!c->scratch) throw Fail{MRA_E_DEVICE, "no-allocation scratch not resolved on this device"};
  int64_t step = rs.prune ? fitting_chunk(rs, p, N, true, out->cc2 != nullptr, c->n_cu, kScratchBytes) : 0;
  const bool pruned = step > 0 && !few_pairs(c, rs, p, step, out->cc2 != nullptr);
  if (!pruned) step = fitting_chunk(rs, p, N, false, out->cc2 != nullptr, c->n_cu, kScratchBytes);
  if (step < 1)
    throw Fail{MRA_E_INVAL, "one particle's operand exceeds the " + std::to_string(kScratchBytes >> 20) +
                                " MiB no-allocation scratch"};
  for (int64_t n0 = 0; n0 < N; n0 += step) {
    const int nc = (int)std::min<int64_t>(step, N - n0);
    ChunkBufs b;
    carve_chunk(rs, p, nc, pruned, out->cc2 != nullptr, c->n_cu, (char*)c->scratch, &b);
    if (pruned) run_chunk(c, rs, p, parts, n0, nc, out, b);
    else run_chunk_unpruned(c, rs, p, parts, n0, nc, out, nullptr, b);
  }
}

// One piece of a stack inside a batched wave.
struct Piece {
  int stack;
  const Refset* rs;
  Plan p;
  int64_t n0;
  int nc;
  bool every;  // evaluate every pair
};

// Device buffers of a batched wave, those of the pieces end to end.
struct WaveBufs {
  size_t parts = 0, tile = 0;  // particles, largest scratch tile
  int grid = 0;                // evaluation workgroups
  char* A = nullptr;
  float *ub = nullptr, *ub_hi = nullptr, *rownorm = nullptr, *scratch = nullptr, *rcc = nullptr, *maxabs = nullptr;
  unsigned long long* rowkey = nullptr;
  int* ridx = nullptr;
  FineOver over{};
  FineDense dense{};
};

// 8-byte words of a piece's row keys
size_t wave_rowkeys(size_t rows, bool pruned) { return (rowkey_bytes(rows, pruned) + 7) / 8; }

// Calls take(name, bytes) for every buffer of a wave.
template <class Take>
WaveBufs layout_wave(const std::vector<Piece>& w, int n_cu, Take take) {
  WaveBufs b;
  const int prec = w[0].rs->g.precision;
  size_t a_bytes = 0, ub_floats = 0, rows = 0, keys = 0, tiles = 0;
  int max_S = 0, units = 0;
  for (const Piece& pc : w) {
    const size_t r = (size_t)pc.nc * pc.p.S, t = (r + kRowTile - 1) / kRowTile;
    a_bytes += t * tile_bytes_of(*pc.rs, true);
    keys += wave_rowkeys(r, true);
    tiles += t;
    ub_floats += r * ub_pitch(*pc.rs);
    rows += r;
    b.parts += pc.nc;
    max_S = std::max(max_S, pc.p.S);
    units = std::max(units, fine_units(pc.p.S, pc.rs->K));
    b.tile = std::max(b.tile, scratch_tile_bytes(*pc.rs));
  }
  b.grid = fine_grid(prec, (int64_t)b.parts, n_cu);
  b.A = (char*)take("A", a_bytes);
  b.ub = (float*)take("ub", ub_floats * sizeof(float));
  b.ub_hi = (float*)take("ub_hi", ub_floats * sizeof(float));
  b.rowkey = (unsigned long long*)take("rowkey", keys * sizeof(unsigned long long));
  b.dense.grid = dense_grid(prec, b.grid, n_cu);
  if (prec == kFP32) {
    b.rownorm = (float*)take("rownorm", 2 * rows * sizeof(float));
    b.scratch = (float*)take("scratch", std::max(b.grid, b.dense.grid) * b.tile);
  } else {
    b.rcc = (float*)take("row_cc", rows * sizeof(float));
    b.ridx = (int*)take("row_idx", rows * sizeof(int));
  }
  take_lists((int64_t)b.parts, tiles, max_S, units, n_cu, b.over, b.dense, take);
  if (prec != kBF16) b.maxabs = (float*)take("maxabs", b.parts * sizeof(float));
  return b;
}

// The same for a wave whose every pair is evaluated.
template <class Take>
WaveBufs layout_every(const std::vector<Piece>& w, Take take) {
  WaveBufs b;
  size_t a_bytes = 0, keys = 0, rows = 0;
  for (const Piece& pc : w) {
    const size_t r = (size_t)pc.nc * pc.p.S;
    a_bytes += (r + kRowTile - 1) / kRowTile * tile_bytes_of(*pc.rs, false);
    keys += wave_rowkeys(r, false);
    rows += r;
    b.parts += pc.nc;
  }
  b.A = (char*)take("A", a_bytes);
  b.rowkey = (unsigned long long*)take("rowkey", keys * sizeof(unsigned long long));
  if (w[0].rs->g.precision != kFP32) {
    b.rcc = (float*)take("row_cc", rows * sizeof(float));
    b.ridx = (int*)take("row_idx", rows * sizeof(int));
  }
  if (w[0].rs->g.precision == kFP16) b.maxabs = (float*)take("maxabs", b.parts * sizeof(float));
  return b;
}

// A wave with every pair evaluated: one launch each of resample + FFT, correlation,
// merge and (16-bit forms) re-score.  Rows past a piece in its last tile keep what
// is there: they take no part in any result.
void launch_every(mra_ctx* c, const mra_stack* stacks, const std::vector<Piece>& w) {
  hipStream_t st = c->stream;
  uint64_t total = ws_kept(c);
  WsNeed need;
  layout_every(w, [&](const char* name, size_t bytes) -> void* {
    total += bytes;
    need.emplace_back(name, bytes);
    return nullptr;
  });
  if (w.size() == 1 || total > c->cap) {
    for (const Piece& pc : w)
      align_stack(c, *pc.rs, pc.p, stacks[pc.stack].parts, pc.n0, pc.nc, &stacks[pc.stack].out, nullptr);
    return;
  }
  ws_step(c, need);
  WaveBufs b = layout_every(w, [&](const char* name, size_t bytes) { return ws_get(c, name, bytes); });
  const int prec = w[0].rs->g.precision, variant = w[0].rs->variant, np = (int)w.size();
  const int layout = a_layout_for(prec, variant);
  int64_t tiles = 0;
  for (const Piece& pc : w) tiles += ((int64_t)pc.nc * pc.p.S + kRowTile - 1) / kRowTile;
  PolarBatch pb{};
  CorrBatch cb{};
  MergeBatch mb{};
  RescoreBatch rb{};
  pb.n = cb.n = mb.n = rb.n = np;
  int part = 0, items = 0, pitems = 0;
  for (int i = 0; i < np; ++i) {
    const Piece& pc = w[i];
    const Refset& rs = *pc.rs;
    const mra_stack& sk = stacks[pc.stack];
    const size_t r = (size_t)pc.nc * pc.p.S;
    const float* src = sk.parts + (size_t)pc.n0 * rs.g.L * rs.g.L;
    ChunkBufs cbuf;
    cbuf.A = (float*)b.A;
    cbuf.rowkey = b.rowkey;
    cbuf.maxabs = b.maxabs ? b.maxabs + part : nullptr;
    if (row_results(rs)) {
      cbuf.rcc = b.rcc;
      cbuf.ridx = b.ridx;
    }
    PolarArgs& pa = pb.piece[i] = polar_args(c, rs, pc.p, src, pc.nc);
    pa.split = polar_split((int)b.parts, rs.R * (pc.p.S / kRowTile + 1), c->n_cu, polar_waves(pa));
    pa.a_layout = layout;
    pa.maxabs = cbuf.maxabs;
    pa.rowkey = cbuf.rowkey;
    pa.out = cbuf.A;
    CorrArgs& ca = cb.piece[i] = corr_args(c, rs, pc.p, pc.nc, layout, cbuf);
    ca.kt_per_wg = corr_tiles_per_wg((int)std::min<int64_t>(tiles, INT32_MAX), rs.n_kt, c->n_cu);
    mb.piece[i] = merge_args(rs, pc.p, pc.n0, pc.nc, &sk.out, cbuf);
    rb.piece[i] = rescore_args(rs, pc.p, src, pc.n0, pc.nc, &sk.out, cbuf);
    pb.start[i] = pitems;
    pitems += pc.nc * pa.split;
    cb.start[i] = items;
    items += corr_items(ca);
    mb.start[i] = rb.start[i] = part;
    part += pc.nc;
    b.A += (r + kRowTile - 1) / kRowTile * tile_bytes_of(rs, false);
    b.rowkey += wave_rowkeys(r, false);
    if (b.rcc) {
      b.rcc += r;
      b.ridx += r;
    }
  }
  pb.start[np] = pitems;
  cb.start[np] = items;
  mb.start[np] = rb.start[np] = part;
  timed(c, "polar", [&] { hip_check(c, launch_polar_batch(pb, st), "polar batch"); });
  timed(c, "corr", [&] { hip_check(c, launch_corr_batch(prec, variant, cb, st), "corr batch"); });
  timed(c, "merge", [&] { hip_check(c, launch_merge_batch(mb, st), "merge batch"); });
  if (prec != kFP32) timed(c, "rescore", [&] { hip_check(c, launch_rescore_batch(rb, st), "rescore batch"); });
}

void launch_wave(mra_ctx* c, const mra_stack* stacks, const std::vector<Piece>& w) {
  if (w[0].every) return launch_every(c, stacks, w);
  hipStream_t st = c->stream;
  uint64_t total = ws_kept(c);
  WsNeed need;
  layout_wave(w, c->n_cu, [&](const char* name, size_t bytes) -> void* {
    total += bytes;
    need.emplace_back(name, bytes);
    return nullptr;
  });
  // one piece is a call of its own (the way its size takes); so are all where what a
  // wave holds besides its operand and bounds does not fit
  if (w.size() == 1 || total > c->cap) {
    for (const Piece& pc : w)
      align_stack(c, *pc.rs, pc.p, stacks[pc.stack].parts, pc.n0, pc.nc, &stacks[pc.stack].out, nullptr);
    return;
  }
  const int prec = w[0].rs->g.precision, np = (int)w.size();
  ws_step(c, need);
  const WaveBufs wb = layout_wave(w, c->n_cu, [&](const char* name, size_t bytes) { return ws_get(c, name, bytes); });
  const size_t parts = wb.parts, tile = wb.tile;
  const int grid = wb.grid;
  const FineOver over = wb.over;
  char* A = wb.A;
  float *ub = wb.ub, *ub_hi = wb.ub_hi, *rownorm = wb.rownorm, *scratch = wb.scratch, *rcc = wb.rcc;
  float* maxabs = wb.maxabs;
  unsigned long long* rowkey = wb.rowkey;
  int* ridx = wb.ridx;

  PolarBatch pb{};
  CorrBatch cb{};
  FineBatch fb{};
  RescoreBatch rb{};
  pb.n = cb.n = fb.n = rb.n = np;
  int part = 0, items = 0, pitems = 0;
  for (int i = 0; i < np; ++i) {
    const Piece& pc = w[i];
    const Refset& rs = *pc.rs;
    const mra_stack& sk = stacks[pc.stack];
    const size_t r = (size_t)pc.nc * pc.p.S;
    const float* src = sk.parts + (size_t)pc.n0 * rs.g.L * rs.g.L;
    ChunkBufs b;
    b.A = (float*)A;
    b.ub = ub;
    b.ub_hi = ub_hi;
    b.rowkey = rowkey;
    b.rownorm = rownorm;
    b.scratch = scratch;
    b.grid = grid;
    b.maxabs = maxabs ? maxabs + part : nullptr;
    if (row_results(rs)) {
      b.rcc = rcc;
      b.ridx = ridx;
    }
    pb.piece[i] = polar_args(c, rs, pc.p, src, pc.nc);
    pb.piece[i].split = polar_split((int)parts, rs.R * (pc.p.S / kRowTile + 1), c->n_cu, polar_waves(pb.piece[i]));
    pb.piece[i].a_layout = kRingPerm16;
    pb.piece[i].maxabs = b.maxabs;
    pb.piece[i].out = b.A;
    cb.piece[i] = corr_args(c, rs, pc.p, pc.nc, kRingPerm16, b);
    cb.start[i] = items;
    items += bound_items(cb.piece[i], 0);
    fb.piece[i] = fine_args(c, rs, pc.p, cb.piece[i], src, pc.n0, pc.nc, &sk.out, b);
    if (scratch) fb.piece[i].scratch_floats = (int)(tile / sizeof(float));
    rb.piece[i] = rescore_args(rs, pc.p, src, pc.n0, pc.nc, &sk.out, b);
    pb.start[i] = pitems;
    pitems += pc.nc * pb.piece[i].split;
    fb.start[i] = rb.start[i] = part;
    A += (r + kRowTile - 1) / kRowTile * tile_bytes_of(rs, true);
    ub += r * ub_pitch(rs);
    ub_hi += r * ub_pitch(rs);
    rowkey += wave_rowkeys(r, true);
    if (rownorm) rownorm += 2 * r;
    if (rcc) {
      rcc += r;
      ridx += r;
    }
    part += pc.nc;
  }
  pb.start[np] = pitems;
  fb.start[np] = rb.start[np] = part;
  cb.start[np] = items;
  timed(c, "polar", [&] { hip_check(c, launch_polar_batch(pb, st), "polar batch"); });
  timed(c, "bound", [&] { hip_check(c, launch_bound_batch(prec, cb, over.count, st), "bound batch"); });
  if (prec == kFP32) {
    FineBatch tb = fb;
    for (int i = 0; i < np; ++i) tb.piece[i].c.A = cb.piece[i].A;
    const int tgrid = fine_grid(kFP16, (int64_t)parts, c->n_cu);
    timed(c, "tighten", [&] { hip_check(c, launch_fine_batch(prec, kFineTighten, tb, over, wb.dense, tgrid, st), "tighten batch"); });
  }
  timed(c, "fine", [&] {
    hip_check(c, launch_fine_batch(prec, kFineArgmax, fb, prec == kFP32 ? FineOver{} : over, wb.dense, grid, st), "fine batch");
  });
  if (prec != kFP32) timed(c, "rescore", [&] { hip_check(c, launch_rescore_batch(rb, st), "rescore batch"); });
}

void run_batch(mra_ctx* c, const mra_stack* stacks, int n, const std::vector<Plan>& plans) {
  const uint64_t budget = c->cap / 2;
  // Stacks that share the kernels' instantiations are packed into the same waves; within a
  // group the caller's order holds.  A group is of one precision and ring bucket, and of one
  // instance of the correlation kernel if every pair is evaluated: with pruning off, or few
  // pairs (per particle, or in all stacks of the bucket together).  Where the bucket has other
  // stacks, whose waves can take those of few pairs, only if these are of so many rows
  // that what they save is more than launches of their own cost (6 stacks of 100 to 150 particles,
  // two of them of few references, BF16: 688 us in two waves, 506 in one).
  auto bucket = [](const Refset& rs) { return 64 * rs.g.precision + ring_bucket(rs.R4); };
  auto instance = [](const Refset& rs) {
    return 8 + 64 * (rs.g.precision * 4 + rs.variant) + corr_group(rs.g.precision, rs.variant, rs.R4) * 1024;
  };
  struct Total {
    int64_t tiles = 0, parts = 0;
    bool others = false;
  };
  std::map<int, Total> total;       // by bucket
  std::map<int, int64_t> few_rows;  // by instance
  auto shares = [&](int i, const Refset& rs) {
    return stacks[i].N > 0 && !stacks[i].out.cc2 && !stacks[i].out.psi_frac && rs.K > 1 && rs.prune;
  };
  auto few = [&](int i, const Refset& rs) {
    const Total& b = total[bucket(rs)];
    return few_each(rs, plans[i], false) || few_tiles(c, rs, plans[i], b.tiles, b.parts, false);
  };
  for (int pass = 0; pass < 2; ++pass)
    for (int i = 0; i < n; ++i) {
      if (stacks[i].N <= 0) continue;
      const Refset& rs = get_refset(c, stacks[i].refset_id);
      if (!shares(i, rs)) continue;
      Total& b = total[bucket(rs)];
      if (pass == 0) {
        b.tiles += tile_pairs(rs, plans[i], stacks[i].N);
        b.parts += stacks[i].N;
      } else if (few(i, rs)) {
        few_rows[instance(rs)] += stacks[i].N * plans[i].S;
      } else {
        b.others = true;
      }
    }
  auto every = [&](int i) {
    const Refset& rs = get_refset(c, stacks[i].refset_id);
    return !rs.prune || (shares(i, rs) && few(i, rs) &&
                         (!total[bucket(rs)].others || few_rows[instance(rs)] >= 32 * kRowTile * (int64_t)c->n_cu));
  };
  auto key = [&](int i) {
    if (stacks[i].N <= 0) return 0;
    const Refset& rs = get_refset(c, stacks[i].refset_id);
    return every(i) ? instance(rs) : bucket(rs);
  };
  std::vector<int> order(n), keys(n);
  for (int i = 0; i < n; ++i) {
    order[i] = i;
    keys[i] = key(i);
  }
  std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return keys[x] < keys[y]; });
  std::vector<Piece> wave;
  uint64_t used = 0;
  auto flush = [&] {
    if (!wave.empty()) launch_wave(c, stacks, wave);
    wave.clear();
    used = 0;
  };
  for (int i : order) {
    const mra_stack& s = stacks[i];
    if (s.N <= 0) continue;
    const Refset& rs = get_refset(c, s.refset_id);
    const Plan& p = plans[i];
    if (rs.K == 1) {  // one reference: the fused single-reference kernel
      run_single(c, rs, p, s.parts, s.N, &s.out);
      continue;
    }
    // runner-up, refinement, a workspace too small, or every pair of so many particles and
    // rows that their launches fill the chip by themselves, with an operand that stays in the
    // last-level cache (4 stacks of 1000 particles, 8 references, BF16: 2.61 ms in a wave, 2.36
    // one by one): the per-chunk path
    const bool ev = every(i);
    const uint64_t per = particle_bytes(rs, p, !ev);
    if (s.out.cc2 || s.out.psi_frac || per > budget / 2 ||
        (ev && s.N >= 2 * c->n_cu && s.N * p.S >= 8 * kRowTile * (int64_t)c->n_cu)) {
      align_stack(c, rs, p, s.parts, 0, s.N, &s.out, nullptr);
      continue;
    }
    const int64_t cap_n = rs.chunk > 0 ? rs.chunk : std::max<int64_t>(1, (int64_t)(budget / per));
    for (int64_t n0 = 0; n0 < s.N;) {
      const bool compatible = wave.empty() || keys[wave[0].stack] == keys[i];
      if (!compatible || (int)wave.size() == kMaxBatchPieces || used + per > budget) flush();
      const int64_t room = std::max<int64_t>(1, (int64_t)((budget - used) / per));
      const int nc = (int)std::min<int64_t>({s.N - n0, room, cap_n, (int64_t)(INT32_MAX / p.S / 2)});
      wave.push_back(Piece{i, &rs, p, n0, nc, ev});
      used += (uint64_t)nc * per + tile_bytes_of(rs, !ev);
      n0 += nc;
    }
  }
  flush();
}

// The buffers of one replaced refset are kept (up to kSpareBytes) for the next
// set of the same sizes: a program that replaces its references on every pass
// then allocates and frees nothing.  What was enqueued against the old set
// comes first on the same stream.
constexpr uint64_t kSpareBytes = 256ull << 20;

uint64_t refset_bytes(const Refset& r) {
  return (uint64_t)r.R * kNphi * (sizeof(Stencil) + r.K * sizeof(float)) +
         (r.B32 ? (uint64_t)r.n_kt * kRefTile * kSlots * 8 * b32_pitch(r.R4) * sizeof(float) : 0) +
         (r.B16 ? (uint64_t)r.n_kt * kSlots * b16_slot_elems(r.R4) * sizeof(uint16_t) : 0);
}

// The set `old` becomes rs, and its buffers the spare ones or nobody's.  (The
// wait, which can fail, comes before any buffer changes hands.)
void replace_refset(mra_ctx* c, Refset& old, const Refset& rs) {
  const bool keep = refset_bytes(old) <= kSpareBytes;
  if ((keep ? c->spare : old).stencil) hip_check(c, hipStreamSynchronize(c->stream), "sync");
  if (keep) std::swap(c->spare, old);
  free_refset(old);
  old = rs;
}

// rs (sizes set, no buffers yet) takes the spare set's buffers if they fit.
bool take_spare(mra_ctx* c, Refset& rs) {
  Refset& o = c->spare;
  if (!o.stencil || o.K != rs.K || o.R != rs.R || o.g.precision != rs.g.precision) return false;
  rs.stencil = o.stencil; rs.norm = o.norm; rs.qhat = o.qhat;
  rs.B32 = o.B32; rs.B16 = o.B16; rs.bnorm = o.bnorm; rs.G1 = o.G1;
  o = Refset{};
  return true;
}

void load_refs_impl(mra_ctx* c, int32_t id, const float* refs, int32_t K, const mra_geom* g) {
  check_geom(g);
  if (K < 1) throw Fail{MRA_E_INVAL, "K must be >= 1"};
  check_index_range(K, g->mirror ? 2 : 1, g->shift_max);
  if (!refs) throw Fail{MRA_E_INVAL, "refs is NULL"};
  Refset rs;
  rs.g = *g;
  rs.K = K;
  rs.R = g->r_max - g->r_min + 1;
  rs.R4 = (rs.R + 3) / 4;
  rs.NS = (rs.R4 + 7) / 8;
  rs.n_kt = (K + kRefTile - 1) / kRefTile;
  rs.variant = corr_default_variant(g->precision, rs.R4);
  hipStream_t st = c->stream;
  try {
    // floor offsets of the sampling positions r (cos, sin): the table holds the
    // quarter turns exactly, so the rings reach from -r_max to r_max
    rs.dmin = -g->r_max;
    rs.dmax = g->r_max;
    // a set of the same sizes that another load replaced lends its buffers
    const bool reuse = take_spare(c, rs);
    auto buf = [&](auto*& ptr, size_t bytes, const char* what) {
      if (!reuse) ptr = (std::remove_reference_t<decltype(ptr)>)alloc(c, bytes, what);
    };
    buf(rs.stencil, (size_t)rs.R * kNphi * sizeof(Stencil), "stencil");
    RefArgs ra{};
    ra.refs = refs;
    ra.K = K; ra.L = g->L; ra.r_min = g->r_min; ra.R = rs.R; ra.R4 = rs.R4; ra.NS = rs.NS;
    ra.n_ref_tiles = rs.n_kt; ra.normalize = g->normalize; ra.prec = g->precision;
    ra.cs64 = c->cs64;
    const WsNeed need = {{"ref_q64", (size_t)K * rs.R * kNphi * sizeof(double)},
                         {"ref_inv", (size_t)K * sizeof(double)},
                         {"ref_Qs", (size_t)K * 129 * rs.R * sizeof(double2)},
                         {"ref_info", 256}};
    ws_step(c, need);
    auto take = [&](int i) { return ws_get(c, need[i].first, need[i].second); };
    ra.q64 = (double*)take(0);
    ra.inv = (double*)take(1);
    ra.Qs = (double2*)take(2);
    ra.info = (RefInfo*)take(3);
    buf(rs.norm, (size_t)K * sizeof(double), "norm");
    buf(rs.qhat, (size_t)K * rs.R * kNphi * sizeof(float), "qhat");
    ra.norm = rs.norm;
    ra.qhat32 = rs.qhat;
    ra.stencil = rs.stencil;
    hip_check(c, launch_ref_stage1(ra, st), "ref stage 1");
    hip_check(c, hipMemcpyAsync(c->ref_info, ra.info, sizeof(RefInfo), hipMemcpyDeviceToHost, st), "memcpy");
    hip_check(c, hipStreamSynchronize(st), "sync");
    const float bmax = c->ref_info->bmax;
    if (g->normalize && c->ref_info->bad < K)
      throw Fail{MRA_E_DEGENERATE,
                 "reference " + std::to_string(c->ref_info->bad) + " has zero weighted ring norm"};
    rs.b_scale = 1.f;
    if (g->precision != kBF16 && bmax > 0.f && std::isfinite(bmax)) {
      // (FP32: only the bounds take it, and references below 2^-113 are better scaled
      // by less than into an infinite scale)
      const int e = 14 - (int)std::ceil(std::log2(bmax));
      rs.b_scale = std::ldexp(1.f, g->precision == kFP32 ? std::min(e, 127) : e);
    }
    ra.b_scale = rs.b_scale;
    // (FP32 with one reference: the fused kernel and the CC table need no bounds)
    if (g->precision == kFP32) buf(rs.B32, (size_t)rs.n_kt * kRefTile * kSlots * 8 * b32_pitch(rs.R4) * sizeof(float), "B32");
    if (g->precision == kFP32 && K > 1) buf(rs.bnorm, (size_t)K * sizeof(float), "bnorm");
    if (g->precision != kFP32 || K > 1)
      buf(rs.B16, (size_t)rs.n_kt * kSlots * b16_slot_elems(rs.R4) * sizeof(uint16_t), "B16");
    ra.B32 = rs.B32;
    ra.B16 = rs.B16;
    ra.bnorm = rs.bnorm;
    if (K == 1) buf(rs.G1, (size_t)rs.R * kSlots * sizeof(float2), "G1");
    ra.G1 = rs.G1;
    hip_check(c, launch_ref_stage2(ra, st), "ref stage 2");
    const auto it = c->refs.find(id);
    if (it == c->refs.end()) c->refs.emplace(id, rs);
    else replace_refset(c, it->second, rs);
  } catch (...) {
    free_refset(rs);
    throw;
  }
}

void averages_core(mra_ctx* c, int K, int L, const float* parts, int64_t N, const mra_result* params,
                   float* averages, int32_t* counts) {
  if (N < 0 || N > (int64_t)INT32_MAX / 2) throw Fail{MRA_E_INVAL, "N out of range"};
  if (!averages || !counts) throw Fail{MRA_E_INVAL, "averages and counts must be non-NULL"};
  if (!params || !params->ref || !params->shift_x || !params->shift_y || !params->psi || !params->mirror)
    throw Fail{MRA_E_INVAL, "params arrays must be non-NULL"};
  if (N > 0 && !parts) throw Fail{MRA_E_INVAL, "parts is NULL"};
  hipStream_t st = c->stream;
  if (N == 0) {
    hip_check(c, hipMemsetAsync(counts, 0, K * sizeof(int32_t), st), "memset");
    return;
  }
  AvgArgs a{};
  a.parts = parts;
  a.N = N;
  a.K = K; a.L = L; a.cx = L / 2;
  a.ref = params->ref; a.shift_x = params->shift_x; a.shift_y = params->shift_y;
  a.psi = params->psi; a.mirror = params->mirror;
  a.cs64 = c->cs64;
  a.n_blk = (int)((N + 1023) / 1024);
  a.max_chunks = (int)((N + kAvgChunk - 1) / kAvgChunk) + K;
  const WsNeed need = {{"avg_blk_cnt", (size_t)a.n_blk * K * sizeof(int)},
                       {"avg_blk_off", (size_t)a.n_blk * K * sizeof(int)},
                       {"avg_cls", (size_t)(K + 1) * sizeof(int)},
                       {"avg_chunk", (size_t)(K + 1) * sizeof(int)},
                       {"avg_order", (size_t)N * sizeof(int)},
                       {"avg_partial", (size_t)a.max_chunks * L * L * sizeof(float)}};
  ws_step(c, need);
  auto take = [&](int i) { return ws_get(c, need[i].first, need[i].second); };
  a.blk_cnt = (int*)take(0);
  a.blk_off = (int*)take(1);
  a.cls_start = (int*)take(2);
  a.chunk_start = (int*)take(3);
  a.order = (int*)take(4);
  a.partial = (float*)take(5);
  a.averages = averages;
  a.counts = counts;
  timed(c, "averages", [&] { hip_check(c, launch_averages(a, st), "averages"); });
}

void update_averages_impl(mra_ctx* c, int32_t id, const float* parts, int64_t N, const mra_result* params,
                          float* averages, int32_t* counts) {
  const Refset& rs = get_refset(c, id);
  averages_core(c, rs.K, rs.g.L, parts, N, params, averages, counts);
}

// The outer repeat: load the averages as references, align, count the
// particles whose key (class, or with by_flat the whole parameter set)
// changed since the previous pass, update the averages.
void iterate_impl(mra_ctx* c, int32_t id, const mra_geom* g, const float* parts, int64_t N, float* averages,
                  int32_t K, int32_t max_iter, double max_changed_frac, const mra_result* out, int32_t* counts,
                  int32_t* n_iter, int64_t* changed, bool by_flat) {
  // a tuning set on this refset id carries over when the geometry matches
  int variant = -1, chunk = 0, prune = 1, run_tiles = 0;
  auto old = c->refs.find(id);
  if (old != c->refs.end() && old->second.K == K && std::memcmp(&old->second.g, g, sizeof(mra_geom)) == 0) {
    variant = old->second.variant;
    chunk = old->second.chunk;
    prune = old->second.prune;
    run_tiles = old->second.run_tiles;
  }
  hipStream_t st = c->stream;
  mra_result o = *out;
  if (by_flat && !o.flat_index) o.flat_index = (int32_t*)ws_get(c, "iter_flat", (size_t)N * sizeof(int32_t), true);
  const int32_t* key = by_flat ? o.flat_index : o.ref;
  int32_t* prev = (int32_t*)ws_get(c, "iter_prev", (size_t)N * sizeof(int32_t), true);
  int* cnt = (int*)ws_get(c, "iter_count", 256, true);
  *n_iter = 0;
  for (int it = 1; it <= max_iter; ++it) {
    load_refs_impl(c, id, averages, K, g);
    if (variant >= 0) {
      Refset& rs = c->refs[id];
      rs.variant = variant;
      rs.chunk = chunk;
      rs.prune = prune;
      rs.run_tiles = run_tiles;
    }
    align_impl(c, id, parts, N, -1, &o, nullptr);
    int64_t n_changed = N;
    if (it == 1) {
      hip_check(c, hipMemcpyAsync(prev, key, (size_t)N * sizeof(int32_t), hipMemcpyDeviceToDevice, st), "memcpy");
    } else {
      int h = 0;
      hip_check(c, hipMemsetAsync(cnt, 0, sizeof(int), st), "memset");
      hip_check(c, launch_count_changed(key, prev, (int)N, cnt, st), "count changed");
      hip_check(c, hipMemcpyAsync(&h, cnt, sizeof(int), hipMemcpyDeviceToHost, st), "memcpy");
      hip_check(c, hipStreamSynchronize(st), "sync");
      n_changed = h;
    }
    update_averages_impl(c, id, parts, N, &o, averages, counts);
    if (changed) changed[it - 1] = n_changed;
    *n_iter = it;
    if (it > 1 && (double)n_changed <= max_changed_frac * (double)N) break;
  }
  hip_check(c, hipStreamSynchronize(st), "sync");
}

void check_loop_args(const mra_geom* g, const float* parts, int64_t N, const float* averages, int32_t max_iter,
                     double max_changed_frac, const mra_result* out, const int32_t* n_iter) {
  check_geom(g);
  if (N < 1 || N > (int64_t)INT32_MAX / 2) throw Fail{MRA_E_INVAL, "N out of range"};
  if (!parts || !averages || !n_iter) throw Fail{MRA_E_INVAL, "NULL argument"};
  if (max_iter < 1) throw Fail{MRA_E_INVAL, "max_iter must be >= 1"};
  if (!(max_changed_frac >= 0.0 && max_changed_frac <= 1.0))
    throw Fail{MRA_E_INVAL, "max_changed_frac must lie in [0, 1]"};
  check_result(out);
}

template <class F>
int guard(mra_ctx* c, F&& fn) {
  if (!c) return MRA_E_INVAL;
  if (c->failed) {
    c->err = "context failed after an earlier device error";
    return MRA_E_DEVICE;
  }
  try {
    hip_check(c, hipSetDevice(c->device), "hipSetDevice");
    for (auto& kv : c->ws) kv.second.keep = false;
    fn();
    return MRA_OK;
  } catch (const Fail& f) {
    c->err = f.msg;
    return f.code;
  } catch (const std::bad_alloc&) {
    c->err = "host out of memory";
    return MRA_E_NOMEM;
  } catch (...) {
    c->err = "unexpected internal error";
    return MRA_E_INVAL;
  }
}

}  // namespace

extern "C" {

int mra_create(mra_ctx** out, int device, void* hip_stream, uint64_t workspace_cap_bytes) {
  if (!out) return MRA_E_INVAL;
  *out = nullptr;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) {
    (void)hipGetLastError();
    return MRA_E_INVAL;
  }
  mra_ctx* c = new (std::nothrow) mra_ctx;
  if (!c) return MRA_E_NOMEM;
  c->device = device;
  c->stream = (hipStream_t)hip_stream;
  c->cap = workspace_cap_bytes ? workspace_cap_bytes : (32ull << 30);
  int rc = guard(c, [&] {
    std::vector<double> cs, sn;
    build_cs(kNphi, cs, sn);
    std::vector<double2> h64(kNphi);
    std::vector<float2> h32(kNphi);
    for (int j = 0; j < kNphi; ++j) {
      h64[j] = make_double2(cs[j], sn[j]);
      h32[j] = make_float2((float)cs[j], (float)sn[j]);
    }
    int ncu = 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess && ncu > 0)
      c->n_cu = ncu;
    c->scratch = scratch_ptr(c);
    hip_check(c, hipHostMalloc((void**)&c->ref_info, sizeof(RefInfo), hipHostMallocDefault), "hipHostMalloc");
    c->cs64 = (double2*)alloc(c, kNphi * sizeof(double2), "cs64");
    c->cs32 = (float2*)alloc(c, kNphi * sizeof(float2), "cs32");
    hip_check(c, hipMemcpy(c->cs64, h64.data(), kNphi * sizeof(double2), hipMemcpyHostToDevice), "memcpy");
    hip_check(c, hipMemcpy(c->cs32, h32.data(), kNphi * sizeof(float2), hipMemcpyHostToDevice), "memcpy");
  });
  if (rc != MRA_OK) {
    if (c->ref_info) (void)hipHostFree(c->ref_info);
    delete c;
    return rc;
  }
  *out = c;
  return MRA_OK;
}

int mra_destroy(mra_ctx* c) {
  if (!c) return MRA_E_INVAL;
  (void)hipSetDevice(c->device);
  (void)hipStreamSynchronize(c->stream);
  clear_profile(c);
  for (auto& kv : c->refs) free_refset(kv.second);
  free_refset(c->spare);
  if (c->ref_info) (void)hipHostFree(c->ref_info);
  for (auto& kv : c->ws)
    if (kv.second.p) (void)hipFree(kv.second.p);
  if (c->cs64) (void)hipFree(c->cs64);
  if (c->cs32) (void)hipFree(c->cs32);
  delete c;
  return MRA_OK;
}

int mra_load_refs(mra_ctx* c, int32_t id, const float* refs, int32_t K, const mra_geom* g) {
  return guard(c, [&] { load_refs_impl(c, id, refs, K, g); });
}

int mra_check_geom(const mra_geom* g, int32_t K, int32_t shift_max) {
  try {
    check_geom(g);
    if (K < 1) return MRA_E_INVAL;
    const int T = shift_max < 0 ? g->shift_max : shift_max;
    if (T > 8) return MRA_E_INVAL;
    check_index_range(K, g->mirror ? 2 : 1, T);
    Refset rs;
    rs.g = *g;
    rs.K = K;
    rs.dmin = -g->r_max;
    rs.dmax = g->r_max;
    (void)plan_for(rs, T);
    return MRA_OK;
  } catch (const Fail& f) {
    return f.code;
  } catch (...) {
    return MRA_E_INVAL;
  }
}

int mra_unload_refs(mra_ctx* c, int32_t id) {
  return guard(c, [&] {
    Refset& rs = get_refset(c, id);
    hip_check(c, hipStreamSynchronize(c->stream), "sync");
    free_refset(rs);
    free_refset(c->spare);
    c->refs.erase(id);
  });
}

int mra_refset_info(mra_ctx* c, int32_t id, int32_t* K, mra_geom* g) {
  return guard(c, [&] {
    Refset& rs = get_refset(c, id);
    if (K) *K = rs.K;
    if (g) *g = rs.g;
  });
}

int mra_align(mra_ctx* c, int32_t id, const float* parts, int64_t N, mra_result* out) {
  return guard(c, [&] { align_impl(c, id, parts, N, -1, out, nullptr); });
}

int mra_align_noalloc(mra_ctx* c, int32_t id, const float* parts, int64_t N, mra_result* out) {
  return guard(c, [&] { align_impl(c, id, parts, N, -1, out, nullptr, true); });
}

int mra_align_batch(mra_ctx* c, const mra_stack* stacks, int32_t n) {
  return guard(c, [&] {
    if (n < 0 || (n > 0 && !stacks)) throw Fail{MRA_E_INVAL, "bad stack list"};
    std::vector<Plan> plans(n);
    for (int i = 0; i < n; ++i) {  // validate everything before enqueueing anything
      const mra_stack& s = stacks[i];
      Refset& rs = get_refset(c, s.refset_id);
      if (s.N < 0) throw Fail{MRA_E_INVAL, "stack N must be >= 0"};
      plans[i] = plan_for(rs, s.shift_max < 0 ? rs.g.shift_max : s.shift_max);
      if (s.N > 0) {
        if (!s.parts) throw Fail{MRA_E_INVAL, "stack parts is NULL"};
        check_result(&s.out);
        if (s.N * (int64_t)plans[i].S > INT32_MAX / 2) throw Fail{MRA_E_INVAL, "stack too large"};
      }
    }
    run_batch(c, stacks, n, plans);
  });
}

int mra_update_averages(mra_ctx* c, int32_t id, const float* parts, int64_t N, const mra_result* params,
                        float* averages, int32_t* counts) {
  return guard(c, [&] { update_averages_impl(c, id, parts, N, params, averages, counts); });
}

int mra_classify(mra_ctx* c, int32_t id, const mra_geom* g, const float* parts, int64_t N, float* averages,
                 int32_t K, int32_t max_iter, double max_changed_frac, mra_result* out, int32_t* counts,
                 int32_t* n_iter, int64_t* changed) {
  return guard(c, [&] {
    check_loop_args(g, parts, N, averages, max_iter, max_changed_frac, out, n_iter);
    if (K < 1) throw Fail{MRA_E_INVAL, "K must be >= 1"};
    if (!counts) throw Fail{MRA_E_INVAL, "counts is NULL"};
    iterate_impl(c, id, g, parts, N, averages, K, max_iter, max_changed_frac, out, counts, n_iter, changed, false);
  });
}

int mra_rfa(mra_ctx* c, int32_t id, const mra_geom* g, const float* parts, int64_t N, float* average,
            int32_t start_from_mean, int32_t max_iter, double max_changed_frac, mra_result* out, int32_t* n_iter,
            int64_t* changed) {
  return guard(c, [&] {
    check_loop_args(g, parts, N, average, max_iter, max_changed_frac, out, n_iter);
    int32_t* cnt = (int32_t*)ws_get(c, "rfa_count", 256, true);
    if (start_from_mean) {  // the plain mean: the average update with every parameter zero
      hipStream_t st = c->stream;
      for (int32_t* p : {out->ref, out->shift_x, out->shift_y, out->psi, out->mirror})
        hip_check(c, hipMemsetAsync(p, 0, (size_t)N * sizeof(int32_t), st), "memset");
      averages_core(c, 1, g->L, parts, N, out, average, cnt);
    }
    iterate_impl(c, id, g, parts, N, average, 1, max_iter, max_changed_frac, out, cnt, n_iter, changed, true);
  });
}

int mra_debug_polar(mra_ctx* c, int32_t id, const float* parts, int64_t N, float* out) {
  return guard(c, [&] {
    Refset& rs = get_refset(c, id);
    if (N < 0 || N > INT32_MAX || (N > 0 && (!parts || !out))) throw Fail{MRA_E_INVAL, "bad arguments"};
    const Plan p = plan_for(rs, rs.g.shift_max);
    PolarArgs pa{};
    pa.parts = parts; pa.n_part = (int)N;
    pa.L = rs.g.L; pa.R = rs.R; pa.R4 = rs.R4; pa.T = p.T; pa.S1 = p.S1; pa.S = p.S;
    pa.cx = p.cx; pa.r_min = rs.g.r_min; pa.cs64 = c->cs64; pa.out = out;
    polar_window(pa, p.lo, p.hi);
    pa.split = 1;
    hip_check(c, launch_polar(1, pa, c->stream), "polar");
  });
}

int mra_debug_spectra(mra_ctx* c, int32_t id, const float* parts, int64_t N, float* out) {
  return guard(c, [&] {
    Refset& rs = get_refset(c, id);
    if (N < 0 || N > INT32_MAX || (N > 0 && (!parts || !out))) throw Fail{MRA_E_INVAL, "bad arguments"};
    const Plan p = plan_for(rs, rs.g.shift_max);
    PolarArgs pa{};
    pa.parts = parts; pa.n_part = (int)N;
    pa.L = rs.g.L; pa.R = rs.R; pa.R4 = rs.R4; pa.T = p.T; pa.S1 = p.S1; pa.S = p.S;
    pa.cx = p.cx; pa.r_min = rs.g.r_min; pa.cs64 = c->cs64; pa.out = out;
    polar_window(pa, p.lo, p.hi);
    pa.split = 1;
    hip_check(c, launch_polar(2, pa, c->stream), "polar");
  });
}

int mra_debug_cctable(mra_ctx* c, int32_t id, const float* parts, int64_t N, float* out) {
  return guard(c, [&] {
    if (N > 0 && !out) throw Fail{MRA_E_INVAL, "out is NULL"};
    align_impl(c, id, parts, N, -1, nullptr, out);
  });
}

int mra_debug_refs(mra_ctx* c, int32_t id, float* qhat, double* norm) {
  return guard(c, [&] {
    Refset& rs = get_refset(c, id);
    if (qhat)
      hip_check(c, hipMemcpyAsync(qhat, rs.qhat, (size_t)rs.K * rs.R * kNphi * sizeof(float), hipMemcpyDeviceToDevice, c->stream), "memcpy");
    if (norm)
      hip_check(c, hipMemcpyAsync(norm, rs.norm, (size_t)rs.K * sizeof(double), hipMemcpyDeviceToDevice, c->stream), "memcpy");
  });
}

int mra_set_tuning(mra_ctx* c, int32_t id, const mra_tuning* t) {
  return guard(c, [&] {
    Refset& rs = get_refset(c, id);
    if (!t) throw Fail{MRA_E_INVAL, "tuning is NULL"};
    const int v = t->corr_variant < 0 ? corr_default_variant(rs.g.precision, rs.R4) : t->corr_variant;
    if (!corr_variant_ok(rs.g.precision, v, rs.R4)) throw Fail{MRA_E_INVAL, "variant cannot serve this geometry"};
    if (t->chunk_particles < 0) throw Fail{MRA_E_INVAL, "chunk_particles must be >= 0"};
    if (t->prune < -1 || t->prune > 1) throw Fail{MRA_E_INVAL, "prune must be -1, 0 or 1"};
    if (t->run_tiles < 0 || t->run_tiles > 64) throw Fail{MRA_E_INVAL, "run_tiles must be in [0, 64]"};
    rs.variant = v;
    rs.chunk = t->chunk_particles;
    rs.prune = t->prune != 0;
    rs.run_tiles = t->run_tiles;
  });
}

int mra_get_tuning(mra_ctx* c, int32_t id, mra_tuning* t) {
  return guard(c, [&] {
    Refset& rs = get_refset(c, id);
    if (!t) throw Fail{MRA_E_INVAL, "tuning is NULL"};
    t->corr_variant = rs.variant;
    t->chunk_particles = rs.chunk;
    t->prune = rs.prune;
    t->run_tiles = rs.run_tiles;
  });
}

int mra_profile(mra_ctx* c, int enable) {
  return guard(c, [&] {
    hip_check(c, hipStreamSynchronize(c->stream), "sync");
    if (enable) clear_profile(c);
    c->profiling = enable != 0;
  });
}

int mra_profile_read(mra_ctx* c, const char* kernel, double* total_ms, int64_t* launches) {
  return guard(c, [&] {
    if (!kernel) throw Fail{MRA_E_INVAL, "kernel name is NULL"};
    hip_check(c, hipStreamSynchronize(c->stream), "sync");
    double tot = 0.0;
    int64_t cnt = 0;
    auto it = c->prof.find(kernel);
    if (it != c->prof.end())
      for (auto& e : it->second) {
        float ms = 0.f;
        hip_check(c, hipEventElapsedTime(&ms, e.first, e.second), "hipEventElapsedTime");
        tot += ms;
        ++cnt;
      }
    if (total_ms) *total_ms = tot;
    if (launches) *launches = cnt;
  });
}

const char* mra_last_error(mra_ctx* c) { return c ? c->err.c_str() : "NULL context"; }

const char* mra_strerror(int code) {
  switch (code) {
    case MRA_OK: return "ok";
    case MRA_E_INVAL: return "invalid argument";
    case MRA_E_NOREF: return "refset not loaded";
    case MRA_E_NOMEM: return "out of device memory";
    case MRA_E_DEVICE: return "device error";
    case MRA_E_DEGENERATE: return "degenerate reference (zero norm)";
    default: return "unknown error";
  }
}

}  // extern "C"
