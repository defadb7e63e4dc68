// C ABI of libovl.so: argument validation, handle management and kernel orchestration.
// The declarations and the contract of every entry point are in include/ovl.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <complex>
#include <cstring>
#include <limits>
#include <map>
#include <memory>
#include <type_traits>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/ovl.h"
#include "kernels.hpp"
#include "march.hpp"
#include "small.hpp"
#include "stout.hpp"
#include "solver.hpp"
#include "workspace.hpp"

namespace ovl {
bool cheb_sign_coeffs(int degree, double eps, std::vector<double> &alpha);
double cheb_eval(const std::vector<double> &alpha, double x);
}  // namespace ovl

using namespace ovl;

// ---------------------------------------------------------------------------------------------
// error reporting
namespace {

thread_local char g_err[1024] = "";

int fail(int code, const char *fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

#define HIP_TRY(expr)                                                                     \
  do {                                                                                    \
    hipError_t e_ = (expr);                                                               \
    if (e_ != hipSuccess) {                                                               \
      (void)hipGetLastError();                                                            \
      return fail(e_ == hipErrorOutOfMemory ? OVL_ENOMEM : OVL_EHIP, "%s failed: %s (%s:%d)", \
                  #expr, hipGetErrorString(e_), __FILE__, __LINE__);                      \
    }                                                                                     \
  } while (0)

inline hipStream_t as_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }

int elem_bytes(int dt) { return dt == OVL_F64 ? 16 : dt == OVL_F32 ? 8 : dt == OVL_BF16 ? 4 : 0; }

std::atomic<uint64_t> g_poly_serial{1};

// stream-ordered temporaries: blocks kept between calls, or (small, and while the stream is captured)
// from the device's default pool
std::once_flag g_pool_once[64];
int setup_pool(int dev) {
  hipMemPool_t pool;
  HIP_TRY(hipDeviceGetDefaultMemPool(&pool, dev));
  uint64_t thr = UINT64_MAX;
  HIP_TRY(hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &thr));
  return OVL_OK;
}

struct Scratch {
  void *p = nullptr;
  hipStream_t s = nullptr;
  Block block;  // p's block, unless p is the pool's
  ~Scratch() {
    if (block.p) block_cache().give(block, s);
    else if (p) (void)hipFreeAsync(p, s);
  }
};

int scratch_alloc(Scratch &sc, size_t bytes, hipStream_t s) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  if (dev >= 0 && dev < 64) {
    int rc = OVL_OK;
    std::call_once(g_pool_once[dev], [&] { rc = setup_pool(dev); });
    if (rc != OVL_OK) return rc;
  }
  sc.s = s;
  auto from_pool = [&] { return hipMallocAsync(&sc.p, std::max<size_t>(bytes, 256), s); };
  hipError_t e = hipSuccess;
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (bytes >= kKeepBlock) HIP_TRY(hipStreamIsCapturing(s, &cap));
  if (bytes >= kKeepBlock && cap == hipStreamCaptureStatusNone) {
    e = block_cache().take(bytes, s, sc.block);
    sc.p = sc.block.p;
  } else {
    e = from_pool();
    // (a captured allocation happens at the replay: nothing to give back now)
    if (e == hipErrorOutOfMemory && hipStreamIsCapturing(s, &cap) == hipSuccess &&
        cap == hipStreamCaptureStatusNone) {
      (void)hipGetLastError();
      e = block_cache().with_room(from_pool);
    }
  }
  HIP_TRY(e);
  return OVL_OK;
}

// kernel timing of the fused Chebyshev step (see ovl_timing_enable): one event pair brackets the
// n consecutive plain step launches of one sign evaluation
// kinds of timed launch runs (ovl_timing_read)
enum : int { TK_STEP = 0, TK_VJP = 1, TK_COUNT = 2 };
struct TimedRun {
  hipEvent_t e0, e1;
  int n;
  int kind = TK_STEP;
};
std::atomic<int> g_timing{0};
std::mutex g_timing_mu;
std::vector<TimedRun> g_timing_events;
std::vector<hipEvent_t> g_event_pool;

hipEvent_t pool_event() {
  if (!g_event_pool.empty()) {
    hipEvent_t e = g_event_pool.back();
    g_event_pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

}  // namespace

// ---------------------------------------------------------------------------------------------
// handles
struct ovl_gauge {
  Geom g;
  int store_dt;
  int device;
  uint64_t serial;    // unique per handle (keys the step-graph cache)
  int lstride;        // elements between link components inside a block (kLinkBlock)
  Block mem;          // links and flags
  void *links;        // [ceil(V / 64)][4 * 3 * 3][64] complex in store_dt
  uint32_t *flags;    // sticky device flags
  int r12 = 0;        // kernels read two rows per link and complete the third (SU(3) fields)
};

struct ovl_poly {
  std::vector<double> alpha;
  double lmax, m_W;
  double bound;       // sup_{|x| <= 1} |p(x)| (sampled, with margin)
  uint64_t serial;
};

struct ovl_defl {
  Geom g;
  int n_ev;
  int store_dt;
  double2 *phi64;     // [n_ev][12][V] orthonormal, FP64
  void *phi_store;    // same in store_dt (== phi64 for F64)
  std::vector<double> lambda;
  // Eigenvalue-correction weights w_i = sign(lambda_i) - p(lambda_i / lmax) of the last few
  // polynomials used with this basis: slot k holds the weights of the polynomial with serial
  // w_serial[k] in w_dev + k n_ev, uploaded from pinned staging w_pin + k n_ev on the caller's
  // stream (event w_evt[k] marks the upload), so a call never waits for the device and a new
  // polynomial never overwrites weights another polynomial's pending work reads.
  static constexpr int kWSlots = 8;
  double *w_dev;
  double *w_pin;
  hipEvent_t w_evt[kWSlots];
  bool w_evt_live[kWSlots];
  uint64_t w_serial[kWSlots];
  uint64_t w_stamp[kWSlots];
  double w_absmax[kWSlots];  // max |w_i|, for the norm bound of the final check
  uint64_t w_clock;
  std::mutex mu;
};

namespace {

int check_dims(const int32_t dims[4], Geom &g) {
  if (!dims) return fail(OVL_EINVAL, "dims is NULL");
  int64_t v = 1;
  for (int i = 0; i < 4; ++i) {
    if (dims[i] < 1 || dims[i] > (1 << 24))
      return fail(OVL_EDIMS, "lattice extent dims[%d] = %d out of range [1, 2^24]", i, dims[i]);
    v *= dims[i];
    if (v > (int64_t)INT32_MAX) return fail(OVL_EDIMS, "lattice volume exceeds 2^31 - 1 sites");
  }
  g.V = (int)v;
  int st = 1;
  for (int i = 0; i < 4; ++i) {
    g.L[i] = dims[i];
    g.stride[i] = st;
    st *= dims[i];
  }
  return OVL_OK;
}

// operator precision of (spinor dtype, link storage) pairs
enum Prec { P_F64 = 0, P_F32 = 1, P_F32_BF16 = 2, P_BAD = -1 };
Prec precision(int spin_dt, int store_dt) {
  if (spin_dt == OVL_F64 && store_dt == OVL_F64) return P_F64;
  if (spin_dt == OVL_F32 && store_dt == OVL_F32) return P_F32;
  if (spin_dt == OVL_F32 && store_dt == OVL_BF16) return P_F32_BF16;
  return P_BAD;
}

// Elements between consecutive link components inside a 64-site block (see link_lane).
constexpr int kLinkBlock = 64;

// workgroups of the stream probes: 32 per compute unit of a 256-CU device, grid-stride
constexpr unsigned kStreamBlocks = 256 * 32;

// every array a kernel addresses through one buffer resource must span < 4 GiB
bool fits_u32(uint64_t n_elems, int dt) { return n_elems * (uint64_t)elem_bytes(dt) < (1ull << 32); }

int check_spinor_call(const ovl_gauge *g, const void *out, const void *in, int nrhs, int spin_dt,
                      Prec &prec) {
  if (!g) return fail(OVL_EINVAL, "gauge handle is NULL");
  if (!out || !in) return fail(OVL_EINVAL, "spinor pointer is NULL");
  if (nrhs < 1 || nrhs > 65535) return fail(OVL_EINVAL, "nrhs = %d out of range [1, 65535]", nrhs);
  if (spin_dt != OVL_F64 && spin_dt != OVL_F32)
    return fail(OVL_EDTYPE, "spinor dtype %d not supported (F64 or F32)", spin_dt);
  if (!fits_u32(12ull * g->g.V, spin_dt))
    return fail(OVL_EDIMS, "one right-hand side of %d sites exceeds 4 GiB", g->g.V);
  prec = precision(spin_dt, g->store_dt);
  if (prec == P_BAD)
    return fail(OVL_EDTYPE, "spinor dtype %d cannot be combined with link storage %d", spin_dt,
                g->store_dt);
  const size_t bytes = (size_t)nrhs * 12 * g->g.V * elem_bytes(spin_dt);
  const char *o = (const char *)out, *i = (const char *)in;
  if (o < i + bytes && i < o + bytes)
    return fail(OVL_EALIAS, "output overlaps the input (the stencil reads neighbour sites)");
  return OVL_OK;
}

int grid_blocks(int V) { return (V + kBlock - 1) / kBlock; }

// Fused step kernel launch shape, as sites per workgroup: 8 (one wave, eight threads per site:
// the forward and backward hops on separate threads) under 4K site-right-hand-sides, where one
// wave's latency chain is the step (8% faster than 16 at 4^4, no faster at 8^3 x 16, slower at
// 12^3 x 24); 16 (one wave, four threads per site) under 64K so that the work spreads over more
// compute units, else 64 (four waves, one site per lane); from 512K site-right-hand-sides with
// FP32 links 128 (four waves, two x-adjacent sites per lane; even Lx, 16-byte aligned vectors),
// which measured 5-7% faster there and slower for smaller lattices and BF16 links.
int launch_spb(int64_t site_rhs) {
  return site_rhs >= 64 * 1024 ? 64 : site_rhs >= 4 * 1024 ? 16 : 8;
}
int item_blocks(int V, int spb) { return (V + spb - 1) / spb; }

// t-streaming tile (ty, tz) of the step kernel's workgroup order: the largest candidate whose
// slice Lx ty tz splits into whole workgroups and holds at most 1.25 MB of links and spinor data
void step_tile(const Geom &g, int spb, int site_bytes, int &ty, int &tz) {
  ty = tz = 0;
  if (spb < 64 || g.V < 64 * 1024) return;
  static const int cand[][2] = {{8, 8}, {8, 4}, {4, 4}, {4, 2}, {2, 2}};
  for (const auto &c : cand) {
    const int64_t slice = (int64_t)g.L[0] * c[0] * c[1];
    if (g.L[1] % c[0] || g.L[2] % c[1] || slice % spb) continue;
    if (slice * site_bytes > 1280 * 1024) continue;
    ty = c[0];
    tz = c[1];
    return;
  }
}

// Launch configuration of the fused step kernel: sites per workgroup, workgroup order (memory
// order, t-streaming tiles where a tile fits, the LDS slab, or plain steps in the t-marching form with
// the final step in tiles), the XCD-contiguous workgroup remap and the right-hand-side block
// (right-hand sides per thread sharing one link read).
// Default rules unless ovl_autotune measured a better one for the same problem set: the
// precision and the (extents, right-hand-side count) of every item of the launch, in order.
struct LaunchCfg {
  int spb, tiles, remap, rb;
};
constexpr int kMaxBatch = 16;  // items of a launch
constexpr int kMarch = 3;  // LaunchCfg::tiles of the t-marching form (spb 64, rb 1)
struct TuneKey {
  int prec;
  int r12;                                // two-row link reads (every item's field allows them)
  std::vector<std::array<int, 5>> items;  // Lx Ly Lz Lt nrhs per item
  bool operator<(const TuneKey &o) const {
    return prec < o.prec || (prec == o.prec && (r12 < o.r12 || (r12 == o.r12 && items < o.items)));
  }
};
std::mutex g_tune_mu;
std::map<TuneKey, LaunchCfg> g_tuned;

bool march_ok(const StepItem *items, int n) {
  int ty, tz;
  for (int i = 0; i < n; ++i)
    if (!march_tile(items[i].g, ty, tz)) return false;
  return true;
}

// bytes of nvec vectors and the links of a launch's steps
int64_t step_set_bytes(int prec, const StepItem *items, int n, int nvec) {
  const int link = prec == P_F64 ? 16 : prec == P_F32 ? 8 : 4;
  int64_t bytes = 0;
  for (int i = 0; i < n; ++i)
    bytes += (int64_t)nvec * 12 * items[i].g.V * items[i].nrhs * (prec == P_F64 ? 16 : 8) +
             (int64_t)36 * items[i].g.V * link;
  return bytes;
}

// Where the t-marching form is the default: the vectors that the step touches (nvec: three in a recurrence,
// two in K) and the links reach the 256 MB last-level cache, and most sites lie in tiles of kMarchThreads
// sites.  Measured, one fused step in the default form / t-marching, us: 16^3 x 32 FP64 3 vectors (302 MB
// with the links) 79.8 / 79.7, 4 110 / 91, 12 341 / 263; FP32 8 vectors 105 / 96, 12 166 / 142; 16-bit
// links 4 vectors (170 MB) 43.3 / 38.6, 2 (94 MB) 25.0 / 27.7, 12 169 / 124; 16^3 x 64 FP64 1 vector
// (302 MB) 64.4 / 54.0.  Below the cache size the form has too few workgroups (8^3 x 16, 12 FP64
// vectors: 18.8 / 29.0), and 192-site tiles leave a quarter of the threads idle (12^3 x 24, 24 FP32
// vectors: 93 / 103).
// FP64 and FP32 links: at 256 MB this holds for lattices of at least 12 MB a vector in equal chunks of four or
// more slices (they gain most: the other forms re-read the t neighbours of such lattices from beyond L2;
// 16^3 x 32 to 16 x 20 x 20 x 40, 3 vectors 288 to 360 MB: 0.99 to 1.27 times as fast).  Smaller lattices,
// chunks of unequal lengths and t extents below four need more, measured over 31 lattices in steps of two and
// three vectors as the time of the default form over this one:
// - three t slices: a shorter lattice's chunk reads more slices before and after it than its own (16^3 x 1,
//   533 vectors, default / t-marching: FP64 360 / 397, FP32 183 / 219; 16^3 x 2, 266 FP32 vectors 197 / 209);
// - bytes: FP64 256 MB, 384 MB with unequal chunks (16^3 x 17 0.86 to 0.93 at 267 to 293 MB, 1.16 at 395); FP32
//   320 and 560 MB (8^3 x 16 0.94 at 263, 1.05 at 311; 8 x 16 x 16 x 13 0.87 to 1.0 up to 504);
// - up to five rounds of workgroups (one a compute unit in FP64, two in FP32), a last round four fifths full on
//   average: 16 x 4 x 4 x 8 FP64 1.11 at 285 MB and 2.0 rounds, 0.91 at 310 MB and 2.1 rounds.
bool march_pays(int prec, const StepItem *items, int n, int nvec) {
  constexpr int64_t MB = (int64_t)1 << 20;
  StepItem plan[kMaxBatch];
  const int64_t bytes = step_set_bytes(prec, items, n, nvec);
  if (n > kMaxBatch || bytes < 256 * MB) return false;
  for (int i = 0; i < n; ++i) {
    int ty, tz;
    if (!march_tile(items[i].g, ty, tz)) return false;
    plan[i] = items[i];
  }
  const int blocks = march_plan(plan, n);
  int64_t sites = 0, full = 0, even = 0, big = 0;  // all; in whole tiles; in equal chunks; of large lattices
  for (int i = 0; i < n; ++i) {
    const Geom &g = items[i].g;
    const int64_t s = (int64_t)g.V * items[i].nrhs;
    const bool eq = g.L[3] >= 4 && g.L[3] % plan[i].nt == 0;
    sites += s;
    if (g.L[0] * plan[i].mty * plan[i].mtz == kMarchThreads && (g.L[3] >= 3 || prec == P_F32_BF16)) full += s;
    if (eq) even += s;
    if (eq && (int64_t)12 * g.V * (prec == P_F64 ? 16 : 8) >= 12 * MB) big += s;
  }
  if (2 * full < sites) return false;
  if (prec == P_F32_BF16 || 2 * big >= sites) return true;
  const bool eq = 2 * even >= sites;
  if (bytes < (prec == P_F64 ? (eq ? 256 : 384) : (eq ? 320 : 560)) * MB) return false;
  const int slots = prec == P_F64 ? 256 : 512, rounds = (blocks + slots - 1) / slots;
  return rounds > 5 || (int64_t)blocks * 5 > (int64_t)4 * rounds * slots;
}

// Right-hand sides whose workgroups for a site block run side by side: up to 16, else groups of kRhsGroup
// (rhs_group_blocks).
constexpr int kRhsGroup = 4;
int rhs_together(int nrhs) { return nrhs <= 16 ? nrhs : kRhsGroup; }

// Launch form without a measured one.  16-bit links run in memory order while the step's vectors and
// links fit the last-level cache with room (120 MB) and what lies between a site and its t neighbour, the
// links, input and output of a t slice, fits an XCD's 4 MB L2 with room (2.6 MB): the tiles save L2 misses
// that cost little there and lose on their shorter XCD ranges (tiles / memory order, us per step: 16^3 x 32,
// slices of 1.3 MB, 16.3 / 14.9; 8 x 16^2 x 32 10.4 / 9.3; 20^3 x 32, 2.6 MB, 28.2 / 26.6; with larger slices
// 24^2 x 16 x 20, 3.0 MB, 20.5 / 21.4; 24^3 x 20, 4.4 MB, 27.1 / 29.6; 32^2 x 16^2, 5.3 MB, 26.7 / 29.3;
// larger sets: 16^3 x 32 3 vectors 132 MB 35.5 / 36.3, 24^3 x 48 285 MB 66.1 / 69.0).  FP32 is even there
// (16^3 x 32 18.6 / 18.5), FP64 faster in tiles (32.6 / 35.5).
LaunchCfg default_cfg(int64_t work, int prec, const StepItem *items, int n) {
  const int spb = (prec == P_F32 && work >= 512 * 1024) ? 128 : launch_spb(work);
  bool tiles = prec != P_F32_BF16 || step_set_bytes(prec, items, n, 3) >= (int64_t)120 << 20;
  for (int i = 0; i < n; ++i) {
    const Geom &g = items[i].g;
    const int64_t slice = (int64_t)g.L[0] * g.L[1] * g.L[2] * (36 * 4 + 2 * 96 * rhs_together(items[i].nrhs));
    tiles = tiles || slice * 10 > (int64_t)26 << 20;
  }
  return LaunchCfg{spb, tiles, 1, 1};
}

TuneKey tune_key(int prec, const StepItem *items, int n) {
  TuneKey k;
  k.prec = prec;
  k.r12 = 1;
  for (int i = 0; i < n; ++i) k.r12 = k.r12 && items[i].r12 != 0;
  for (int i = 0; i < n; ++i)
    k.items.push_back({items[i].g.L[0], items[i].g.L[1], items[i].g.L[2], items[i].g.L[3],
                       items[i].nrhs});
  return k;
}

// nvec: vectors that a step of the launch touches
LaunchCfg lookup_cfg(int prec, const StepItem *items, int n, int64_t work, int nvec) {
  const TuneKey k = tune_key(prec, items, n);
  std::lock_guard<std::mutex> lk(g_tune_mu);
  auto it = g_tuned.find(k);
  if (it != g_tuned.end()) {
    if (it->second.tiles != kMarch || march_ok(items, n)) return it->second;
    return default_cfg(work, prec, items, n);
  }
  return march_pays(prec, items, n, nvec) ? LaunchCfg{64, kMarch, 1, 1} : default_cfg(work, prec, items, n);
}

// two sites per lane need FP32 spinors, an even Lx (pairs never straddle an x line) and 16-byte
// aligned vectors
bool aligned16(const void *ptr) { return ((uintptr_t)ptr & 15u) == 0; }
bool pairs_ok(Prec prec, const StepItem *items, int n) {
  if (prec == P_F64) return false;
  for (int i = 0; i < n; ++i) {
    const StepItem &it = items[i];
    if (it.g.L[0] % 2 || !aligned16(it.psi) || !aligned16(it.phi)) return false;
    for (int k = 0; k < 3; ++k)
      if (!aligned16(it.buf[k])) return false;
    if (it.twin) {
      if (!aligned16(it.twin_psi)) return false;
      for (int k = 0; k < 3; ++k)
        if (!aligned16(it.twin_buf[k])) return false;
    }
  }
  return true;
}
// right-hand-side blocks exist for the one-site forms with four threads per site (16 and 64
// sites per workgroup) in the memory and tile orders
bool rb_ok(const LaunchCfg &c) {
  return c.rb == 1 || ((c.rb == 2 || c.rb == 4) && (c.spb == 16 || c.spb == 64) && c.tiles < 2);
}
LaunchCfg fit_cfg(LaunchCfg c, bool pairs) {
  if (c.spb == 128 && !pairs && c.tiles != 2) c.spb = 64;
  if (!rb_ok(c)) c.rb = 1;
  return c;
}

// slab order (tiles == 2): whole x lines, SPB = 64 NW sites = Lx ny with ny | Ly, NW = 1..4,
// single problems only
bool slab_ok(const Geom &g, int spb, Prec prec) {
  if (spb % 64 || spb < 64 || spb > 256 || spb % g.L[0] || g.L[1] % (spb / g.L[0])) return false;
  const int bytes = prec == P_F64 ? slab_lds_bytes<double>(spb, g.L[0]) : slab_lds_bytes<float>(spb, g.L[0]);
  return bytes <= 160 * 1024 - 512;
}
LaunchCfg fit_slab(LaunchCfg c, const StepItem &it, Prec prec, int64_t work, bool pairs) {
  if (c.tiles == 2 && !slab_ok(it.g, c.spb, prec)) return fit_cfg(default_cfg(work, prec, &it, 1), pairs);
  return c;
}

// Right-hand-side groups of the workgroup order, in right-hand-side blocks (0: one group).  Up
// to 16 right-hand sides form one group: their workgroups for a site block run side by side and
// share the links through L2 (grouping the 12 right-hand sides of the batched workload measured
// no faster).  More right-hand sides (the eigen-solve's blocks of 64 to 256 vectors) run in
// groups of kRhsGroup, so that between a site and its t neighbour only one group's spinors pass
// through L2 (K on 128 FP64 vectors of 16^3 x 32 in the default configuration: 4.38 ms as one
// group, 3.63 / 3.57 / 3.54 / 3.63 ms in groups of 1 / 2 / 4 / 8).
int rhs_group_blocks(int nrhs, int rb) {
  return nrhs <= 16 ? 0 : std::max(1, kRhsGroup / rb);
}

int site_bytes_of(Prec prec);

// workgroup order and first workgroup of every item, into the launch's arguments: the plan of the
// step kernels and, with cfg.tiles == kMarch, that of the t-marching form of the plain steps
template <bool TABLE>
void plan_launch(StepArgs<TABLE> &p, StepItem *items, int n, const LaunchCfg &cfg, Prec prec) {
  const int site_bytes = site_bytes_of(prec);
  int total = 0;
  for (int i = 0; i < n; ++i) {
    StepItem &it = items[i];
    it.blk0 = total;
    it.ty = it.tz = 0;
    it.rgroup = rhs_group_blocks(it.nrhs, cfg.rb);
    // the slice budget covers every right-hand side of a group: they all pass through L2 between
    // a site and its t neighbour
    const int grhs = it.rgroup > 0 ? std::min(it.nrhs, it.rgroup * cfg.rb) : it.nrhs;
    if (cfg.tiles == 1 || cfg.tiles == kMarch)
      step_tile(it.g, cfg.spb, site_bytes * grhs, it.ty, it.tz);
    it.nt = 0;
    total += item_blocks(it.g.V, cfg.spb) * ((it.nrhs + cfg.rb - 1) / cfg.rb);
  }
  p.total_blocks = total;
  p.remap = cfg.remap;
  p.march_blocks = 0;
  if (cfg.tiles != kMarch) return;
  p.march_blocks = march_plan(items, n);
}

int site_bytes_of(Prec prec) {
  return prec == P_F64 ? 36 * 16 + 12 * 16 : prec == P_F32 ? 36 * 8 + 12 * 8 : 36 * 4 + 12 * 8;
}

int64_t items_work(const StepItem *items, int n) {
  int64_t w = 0;
  for (int i = 0; i < n; ++i) w += (int64_t)items[i].g.V * items[i].nrhs;
  return w;
}

// Lets a kernel use `bytes` of dynamic LDS on the current device; `done` (one per kernel) remembers the
// devices where it may.
int allow_lds(const void *kernel, int bytes, std::atomic<uint64_t> &done) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  const uint64_t bit = dev >= 0 && dev < 64 ? uint64_t(1) << dev : 0;
  if (done.load(std::memory_order_relaxed) & bit) return OVL_OK;
  HIP_TRY(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
  done.fetch_or(bit, std::memory_order_relaxed);
  return OVL_OK;
}

// launch one step; a single-problem launch plans its item here, a table launch was planned when
// its table was written (p.total_blocks, spb)
template <class C, class SE, class LE, int NW, bool R12>
int launch_slab(StepArgs<false> &p, hipStream_t s) {
  const int bytes = slab_lds_bytes<C>(64 * NW, p.item.g.L[0]);
  static std::atomic<uint64_t> done{0};
  const int rc = allow_lds((const void *)step_slab_kernel<C, SE, LE, NW, false, R12>, 160 * 1024 - 512, done);
  if (rc) return rc;
  step_slab_kernel<C, SE, LE, NW, false, R12><<<p.total_blocks, 256 * NW, bytes, s>>>(p);
  HIP_TRY(hipGetLastError());
  return OVL_OK;
}

template <class C, class SE, class LE, bool TABLE, bool R12, int SPB>
int launch_rb(StepArgs<TABLE> &p, int rb, hipStream_t s) {
  switch (rb) {
    case 1: step_kernel<C, SE, LE, SPB, TABLE, 4, R12, 1><<<p.total_blocks, 4 * SPB, 0, s>>>(p); break;
    case 2: step_kernel<C, SE, LE, SPB, TABLE, 4, R12, 2><<<p.total_blocks, 4 * SPB, 0, s>>>(p); break;
    case 4: step_kernel<C, SE, LE, SPB, TABLE, 4, R12, 4><<<p.total_blocks, 4 * SPB, 0, s>>>(p); break;
    default: return fail(OVL_EINVAL, "no right-hand-side block of %d", rb);
  }
  return OVL_OK;
}

// Plain steps of single problems in the 8- and 16-site forms take step_small_kernel: its reciprocals
// hold 16 bits (fewer than 64K sites and workgroups) and its workgroup order is one right-hand-side
// group (up to 16).  Faster than step_kernel at every size measured below the line (4^4 FP64 4.2 / 3.3 us
// per step, 12^3 x 24 FP32 8.5 / 7.6); above it the default is the 64-site form.
bool small_ok(const StepArgs<false> &p) {
  const StepItem &I = p.item;
  return p.mode == MODE_STEP && !I.twin && I.nrhs <= 16 && I.g.V < 64 * 1024 &&
         p.total_blocks < 64 * 1024;
}
template <class C, class SE, class LE, bool R12>
void launch_small(const StepArgs<false> &p, int spb, hipStream_t s) {
  const StepItem &I = p.item;
  auto vec = [&](int role) { return role == ROLE_PSI ? I.psi : I.buf[role - 1]; };
  SmallArgs<C> a;
  a.U = I.U;
  a.v = vec(p.v_role);
  a.src = p.a != 0.0 ? I.psi : nullptr;
  a.w = p.w_role == ROLE_NONE ? nullptr : vec(p.w_role);
  a.out = const_cast<void *>(vec(p.out_role));
  a.kd = C(p.kd);
  a.kh = C(p.kh);
  a.a = C(p.a);
  a.t = C(p.t);
  a.lx = small_div(I.g.L[0]);
  a.ly = small_div(I.g.L[1]);
  a.lz = small_div(I.g.L[2]);
  a.nrhs = small_div(I.nrhs);
  a.lt = I.g.L[3];
  a.remap = p.remap;
  a.blocks = p.total_blocks;
  a.v_g5 = p.v_g5;
  a.y_g5 = p.y_g5;
  a.src_g5 = p.src_g5;
  if (spb == 8) step_small_kernel<C, SE, LE, 8, 8, R12><<<p.total_blocks, 64, 0, s>>>(a);
  else step_small_kernel<C, SE, LE, 16, 4, R12><<<p.total_blocks, 64, 0, s>>>(a);
}

template <class C, class SE, class LE, bool TABLE, bool R12>
int launch_step_r(StepArgs<TABLE> &p, const LaunchCfg &cfg, hipStream_t s) {
  const int spb = cfg.spb;
  if (cfg.tiles == 2) {
    if constexpr (TABLE) {
      return fail(OVL_EINVAL, "the slab order takes single problems");
    } else {
      switch (spb) {
        case 64: return launch_slab<C, SE, LE, 1, R12>(p, s);
        case 128: return launch_slab<C, SE, LE, 2, R12>(p, s);
        case 192: return launch_slab<C, SE, LE, 3, R12>(p, s);
        case 256:
          if constexpr (sizeof(C) == 4) return launch_slab<C, SE, LE, 4, R12>(p, s);
          return fail(OVL_EINVAL, "FP64 slab of 256 sites does not fit the LDS");
        default: return fail(OVL_EINVAL, "slab of %d sites", spb);
      }
    }
  }
  if (cfg.rb != 1 && spb != 64 && spb != 16)
    return fail(OVL_EINVAL, "right-hand-side blocks need 16 or 64 sites per workgroup");
  int rc = OVL_OK;
  if constexpr (!TABLE)
    if ((spb == 8 || spb == 16) && cfg.rb == 1 && cfg.tiles < 2 && small_ok(p)) {
      launch_small<C, SE, LE, R12>(p, spb, s);
      HIP_TRY(hipGetLastError());
      return OVL_OK;
    }
  if (spb == 128) {
    if constexpr (std::is_same<SE, float2>::value)
      step2_kernel<LE, 64, TABLE, R12><<<p.total_blocks, 256, 0, s>>>(p);
    else
      return fail(OVL_EINVAL, "two sites per lane need FP32 spinors");
  } else if (spb == 64) {
    rc = launch_rb<C, SE, LE, TABLE, R12, 64>(p, cfg.rb, s);
  } else if (spb == 16) {
    rc = launch_rb<C, SE, LE, TABLE, R12, 16>(p, cfg.rb, s);
  } else if (spb == 8) {
    step_kernel<C, SE, LE, 8, TABLE, 8, R12><<<p.total_blocks, 64, 0, s>>>(p);
  } else {
    return fail(OVL_EINVAL, "no step kernel for %d sites per workgroup", spb);
  }
  if (rc) return rc;
  HIP_TRY(hipGetLastError());
  return OVL_OK;
}

// the t-marching form of a plain step
template <class C, class SE, class LE, bool TABLE, bool R12>
int launch_march(StepArgs<TABLE> &p, hipStream_t s) {
  constexpr int bytes = march_lds_bytes<C>();
  static std::atomic<uint64_t> done{0};
  const int rc = allow_lds((const void *)march_kernel<C, SE, LE, TABLE, R12>, bytes, done);
  if (rc) return rc;
  march_kernel<C, SE, LE, TABLE, R12><<<p.march_blocks, kMarchThreads, bytes, s>>>(p);
  HIP_TRY(hipGetLastError());
  return OVL_OK;
}

// two-row link reads where the problem's field allows them (single problem: its handle; a
// table launch: every item's, recorded in p.r12 when the table was written)
template <class C, class SE, class LE, bool TABLE>
int launch_step(StepArgs<TABLE> &p, const LaunchCfg &cfg, hipStream_t s) {
  const bool r12 = TABLE ? p.r12 != 0 : p.item.r12 != 0;
  if (p.march_blocks > 0 && p.mode == MODE_STEP)
    return r12 ? launch_march<C, SE, LE, TABLE, true>(p, s)
               : launch_march<C, SE, LE, TABLE, false>(p, s);
  return r12 ? launch_step_r<C, SE, LE, TABLE, true>(p, cfg, s)
             : launch_step_r<C, SE, LE, TABLE, false>(p, cfg, s);
}

template <bool TABLE>
int dispatch_step(Prec prec, StepArgs<TABLE> &p, const LaunchCfg &cfg, hipStream_t s) {
  switch (prec) {
    case P_F64: return launch_step<double, double2, double2, TABLE>(p, cfg, s);
    case P_F32: return launch_step<float, float2, float2, TABLE>(p, cfg, s);
    case P_F32_BF16: return launch_step<float, float2, bf16c, TABLE>(p, cfg, s);
    default: return fail(OVL_EDTYPE, "bad precision");
  }
}

// single problem: plan its item with the tuned (or default) configuration, then launch
int dispatch_cfg(Prec prec, StepArgs<false> &p, const LaunchCfg &cfg, hipStream_t s) {
  plan_launch(p, &p.item, 1, cfg, prec);
  return dispatch_step(prec, p, cfg, s);
}
// distinct vectors among a single problem's operands
int step_vectors(const StepArgs<false> &p) {
  const StepItem &I = p.item;
  auto vec = [&](int role) { return role == ROLE_PSI ? I.psi : I.buf[role - 1]; };
  const void *v[4] = {vec(p.v_role), vec(p.out_role), p.w_role == ROLE_NONE ? nullptr : vec(p.w_role),
                      p.a != 0.0 ? I.psi : nullptr};
  int n = 0;
  for (int i = 0; i < 4; ++i) {
    bool seen = !v[i];
    for (int j = 0; j < i; ++j) seen = seen || v[j] == v[i];
    n += !seen;
  }
  return n;
}
int dispatch_single(Prec prec, StepArgs<false> &p, hipStream_t s) {
  const int64_t work = items_work(&p.item, 1);
  const bool pairs = pairs_ok(prec, &p.item, 1);
  const LaunchCfg cfg = fit_slab(
      fit_cfg(lookup_cfg((int)prec, &p.item, 1, work, step_vectors(p)), pairs), p.item, prec,
      work, pairs);
  return dispatch_cfg(prec, p, cfg, s);
}

void fill_item(StepItem &it, const ovl_gauge *g, int nrhs) {
  std::memset(&it, 0, sizeof(it));
  it.U = g->links;
  it.g = g->g;
  it.lstride = g->lstride;
  it.r12 = g->r12;
  it.nrhs = nrhs;
}

template <bool TABLE>
void clear_args(StepArgs<TABLE> &p) {
  std::memset(&p, 0, sizeof(p));
  p.v_role = ROLE_PSI;
  p.w_role = ROLE_NONE;
  p.out_role = ROLE_B0;
  p.mode = MODE_STEP;
  p.remap = 1;
}

// a one-problem launch: psi = src, buf = {b0, b1, b2}
StepArgs<false> single_args(const ovl_gauge *g, int nrhs) {
  StepArgs<false> p;
  clear_args(p);
  fill_item(p.item, g, nrhs);
  p.n_items = 1;
  return p;
}

// c[r][i] = phi_i^+ psi_r (FP64 result), scratch `partial` of n_blocks * nrhs * n_ev double2.
// workgroups of the two projection kernels; the partial buffer holds project_blocks(V) of either
int project_blocks_valu(int V) { return std::min(grid_blocks(V), 1024); }
int project_blocks_mfma(int V) {  // about 1024 reals per workgroup: many short FP32 sums
  return (int)std::min<int64_t>(((int64_t)24 * V + 1023) / 1024, 2048);
}
int project_blocks(int V) { return std::max(project_blocks_valu(V), project_blocks_mfma(V)); }

// Matrix-core projection: tiles of 16 vectors x 8 right-hand sides, up to 2 x 2 per workgroup.
template <class SE>
int project_mfma(const SE *phi, int n_ev, const SE *psi, int psi_g5, int nrhs, int V,
                 double2 *partial, int nblk, double2 *c, hipStream_t s) {
  const int64_t K = (int64_t)24 * V;
  nblk = std::min(nblk, project_blocks_mfma(V));
  // reals per workgroup: a multiple of 64 (4 waves x 4 lane groups x 4 reals)
  int64_t chunk = (K + nblk - 1) / nblk;
  chunk = (chunk + 63) / 64 * 64;
  const int blocks = (int)((K + chunk - 1) / chunk);
  const int te = n_ev > 16 ? 2 : 1, tr = nrhs > 8 ? 2 : 1;
  const dim3 grid(blocks, (n_ev + 16 * te - 1) / (16 * te), (nrhs + 8 * tr - 1) / (8 * tr));
  auto go = [&](auto kernel) {
    kernel<<<grid, 256, 0, s>>>(phi, n_ev, psi, nrhs, psi_g5, V, (int)chunk, partial);
  };
  if (te == 1 && tr == 1) go(project_mfma_kernel<SE, 1, 1>);
  else if (te == 2 && tr == 1) go(project_mfma_kernel<SE, 2, 1>);
  else if (te == 1) go(project_mfma_kernel<SE, 1, 2>);
  else go(project_mfma_kernel<SE, 2, 2>);
  HIP_TRY(hipGetLastError());
  const int count = nrhs * n_ev;
  project_reduce_kernel<<<count, 64, 0, s>>>(partial, blocks, count, c);
  HIP_TRY(hipGetLastError());
  return OVL_OK;
}

// FP64 storage: one right-hand side takes the VALU kernel with FP64 products (each basis vector is
// read once whatever the kernel), and so do several on a few modes of a larger lattice, where its more
// numerous workgroups count for more than a basis read once per right-hand side (VALU / matrix cores, us:
// 16^3 x 32, 1 mode, 2 right-hand sides 25 / 71, 12 sides 69 / 125, 4 modes and 4 sides 50 / 75, 6 and 2
// 54 / 75; 24^3 x 48, 2 modes and 2 sides 123 / 311; 12^3 x 16, 1 mode, 12 sides 24 / 40, 4 sides 25 / 25, but 5
// modes and 2 sides 36 / 28; 16 x 24^2 x 32, 3 modes and 6 sides 192 / 153, 8 and 2 188 / 161).
// The others take the FP64 matrix cores, where one read of the basis serves 16 right-hand sides
// and one read of a right-hand side 32 vectors.
int project(const double2 *phi, int n_ev, const double2 *psi, int psi_g5, int nrhs, int V,
            double2 *partial, int nblk, double2 *c, hipStream_t s) {
  const bool few = n_ev == 1 ? (int64_t)V * nrhs >= 128 * 1024
                             : V >= 49152 && ((n_ev <= 4 && nrhs <= 4) || (n_ev <= 6 && n_ev * nrhs <= 12));
  if (nrhs > 1 && !few) return project_mfma(phi, n_ev, psi, psi_g5, nrhs, V, partial, nblk, c, s);
  nblk = std::min(nblk, project_blocks_valu(V));
  auto go = [&](auto kernel, int ch) {
    const dim3 grid(nblk, (n_ev + ch - 1) / ch, nrhs);
    kernel<<<grid, kBlock, 0, s>>>(phi, n_ev, psi, psi_g5, V, partial);
  };
  if (nrhs == 1) go(project_partial_kernel<double2, 8, false>, 8);
  else if (n_ev == 1) go(project_partial_kernel<double2, 1, true>, 1);
  else if (n_ev == 2) go(project_partial_kernel<double2, 2, true>, 2);
  else if (n_ev <= 4) go(project_partial_kernel<double2, 4, true>, 4);
  else go(project_partial_kernel<double2, 8, true>, 8);
  HIP_TRY(hipGetLastError());
  const int count = nrhs * n_ev;
  project_reduce_kernel<<<count, 64, 0, s>>>(partial, nblk, count, c);
  HIP_TRY(hipGetLastError());
  return OVL_OK;
}

// FP32 storage: the FP32 matrix cores with FP64 running sums
int project(const float2 *phi, int n_ev, const float2 *psi, int psi_g5, int nrhs, int V,
            double2 *partial, int nblk, double2 *c, hipStream_t s) {
  if (!fits_u32(12ull * V * nrhs, OVL_F32))
    return fail(OVL_EDIMS, "%d right-hand sides of %d sites exceed 4 GiB", nrhs, V);
  return project_mfma(phi, n_ev, psi, psi_g5, nrhs, V, partial, nblk, c, s);
}

// Device weights w_i = sign(lambda_i) - p(lambda_i / lmax) (FP64, Sec. 2, eq. 3) of polynomial p
// for basis d: the slot already holding them, else the least recently used slot, refilled on
// stream s.  *w_out receives the device pointer, *absmax the largest |w_i|.
int defl_weights(ovl_defl *d, const ovl_poly *p, hipStream_t s, const double **w_out,
                 double *absmax) {
  std::lock_guard<std::mutex> lk(d->mu);
  int k = -1;
  for (int i = 0; i < ovl_defl::kWSlots; ++i)
    if (d->w_serial[i] == p->serial) k = i;
  if (k < 0) {
    k = 0;
    for (int i = 1; i < ovl_defl::kWSlots; ++i)
      if (d->w_stamp[i] < d->w_stamp[k]) k = i;
    // the staging of slot k may still feed an upload that has not run yet
    if (d->w_evt_live[k]) HIP_TRY(hipEventSynchronize(d->w_evt[k]));
    double *wp = d->w_pin + (size_t)k * d->n_ev;
    double m = 0.0;
    for (int i = 0; i < d->n_ev; ++i) {
      const double l = d->lambda[i];
      const double sg = l > 0 ? 1.0 : (l < 0 ? -1.0 : 0.0);
      wp[i] = sg - cheb_eval(p->alpha, l / p->lmax);
      m = std::max(m, std::fabs(wp[i]));
    }
    d->w_serial[k] = 0;
    HIP_TRY(hipMemcpyAsync(d->w_dev + (size_t)k * d->n_ev, wp, sizeof(double) * d->n_ev,
                           hipMemcpyHostToDevice, s));
    HIP_TRY(hipEventRecord(d->w_evt[k], s));
    d->w_evt_live[k] = true;
    d->w_serial[k] = p->serial;
    d->w_absmax[k] = m;
  }
  d->w_stamp[k] = ++d->w_clock;
  *w_out = d->w_dev + (size_t)k * d->n_ev;
  *absmax = d->w_absmax[k];
  return OVL_OK;
}

// One problem of a sign / overlap evaluation.
struct SignJob {
  const ovl_gauge *g;
  ovl_defl *d;  // nullable
  const void *in;
  void *out;
  int nrhs;
};


// ---------------------------------------------------------------------------------------------
// Step graphs.  A small single-problem evaluation is bound by the launch rate (its steps take a
// few microseconds each), and a HIP graph replays a sequence of kernels faster than the same
// launches made one by one.  The plain recurrence steps k = N-1 .. 1 of a repeated evaluation
// (same gauge field, polynomial, source and output buffers, precision, source gamma5 and launch
// configuration) are captured on its second occurrence and replayed from then on; the graph
// owns the one work vector the steps use, so no allocation or memset is captured.  The deflation
// projection, the final fused step and the norm check are launched directly around it.
std::atomic<int> g_graphs{1};

struct GraphKey {
  int device;
  uint64_t g_serial, p_serial;
  const void *in;
  void *out;
  int nrhs, prec, src_g5, spb, tiles, remap, rb;
  bool operator==(const GraphKey &o) const {
    return device == o.device && g_serial == o.g_serial && p_serial == o.p_serial && in == o.in &&
           out == o.out && nrhs == o.nrhs && prec == o.prec && src_g5 == o.src_g5 &&
           spb == o.spb && tiles == o.tiles && remap == o.remap && rb == o.rb;
  }
};
struct GraphEntry {
  GraphKey key;
  void *work = nullptr;  // the odd-k recurrence vector
  hipGraphExec_t exec = nullptr;
  int uses = 0;
  bool failed = false;  // capture or instantiation failed: launch directly
  uint64_t stamp = 0;
};
constexpr int kGraphCache = 8;
std::mutex g_graph_mu;
std::vector<GraphEntry> g_graph_cache;
uint64_t g_graph_clock = 0;

void graph_release(GraphEntry &e) {
  if (e.exec) (void)hipGraphExecDestroy(e.exec);
  if (e.work) (void)hipFree(e.work);  // synchronises the device: eviction only
  e.exec = nullptr;
  e.work = nullptr;
}

// the cache entry for `key` (created with its work vector when absent, evicting the least
// recently used); nullptr when the work vector cannot be allocated
GraphEntry *graph_entry(const GraphKey &key, size_t work_bytes) {
  for (auto &e : g_graph_cache)
    if (e.key == key) {
      e.stamp = ++g_graph_clock;
      return &e;
    }
  if ((int)g_graph_cache.size() >= kGraphCache) {
    auto lru = std::min_element(g_graph_cache.begin(), g_graph_cache.end(),
                                [](const GraphEntry &a, const GraphEntry &b) { return a.stamp < b.stamp; });
    graph_release(*lru);
    g_graph_cache.erase(lru);
  }
  GraphEntry e;
  e.key = key;
  if (block_cache().with_room([&] { return hipMalloc(&e.work, work_bytes); }) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  e.stamp = ++g_graph_clock;
  g_graph_cache.push_back(e);
  return &g_graph_cache.back();
}

// a private stream per device on which step sequences are captured (capture executes nothing)
hipStream_t capture_stream(int device) {
  static std::mutex mu;
  static std::map<int, hipStream_t> streams;
  std::lock_guard<std::mutex> lk(mu);
  auto it = streams.find(device);
  if (it != streams.end()) return it->second;
  hipStream_t cs = nullptr;
  if (hipStreamCreateWithFlags(&cs, hipStreamNonBlocking) != hipSuccess) return nullptr;
  streams[device] = cs;
  return cs;
}

// Clenshaw evaluation of sum_m alpha_m T_m(X) in + deflation, final combine by `mode`, for up to
// NI problems that share the polynomial, in one launch per K application.
// b_k = alpha_k src + 2 X b_{k+1} - b_{k+2}, k = N-1 .. 1 (b_N = alpha_N src and b_{N+1} = 0
// are folded into the first two steps), result = alpha_0 src + X b_1 - b_2.  b_k lives in
// `out` for even k and in one scratch vector for odd k; every step updates b_{k+2} in place.
// Work space of one evaluation: the caller's fixed buffer (fixed != nullptr: the entry point that
// allocates nothing; sizes above fixed_cap are rejected) or a stream-ordered allocation.
struct SignSpace {
  void *fixed = nullptr;
  size_t fixed_cap = 0;
};

// The launch configuration of an evaluation of these problems: the tuned one for the same
// problem set (ovl_autotune), else the default rules, fitted to what the vectors allow.
template <bool TABLE>
LaunchCfg sign_cfg(const SignJob *jobs, int nj, Prec prec) {
  int64_t work = 0;
  for (int j = 0; j < nj; ++j) work += (int64_t)jobs[j].g->g.V * jobs[j].nrhs;
  bool pairs = prec != P_F64;
  for (int j = 0; j < nj; ++j)
    pairs = pairs && jobs[j].g->g.L[0] % 2 == 0 && aligned16(jobs[j].in) && aligned16(jobs[j].out) &&
            (!jobs[j].d || aligned16(jobs[j].d->phi_store));
  StepItem key_items[kMaxBatch];
  for (int j = 0; j < nj; ++j) fill_item(key_items[j], jobs[j].g, jobs[j].nrhs);
  LaunchCfg cfg = fit_cfg(lookup_cfg((int)prec, key_items, nj, work, 3), pairs);
  if (TABLE) return cfg.tiles == 2 ? fit_cfg(default_cfg(work, prec, key_items, nj), pairs) : cfg;
  return fit_slab(cfg, key_items[0], prec, work, pairs);
}

template <bool TABLE>
int run_sign_jobs(const SignJob *jobs, int nj, const ovl_poly *p, int mode, double mu, int src_g5,
                  int spin_dt, Prec prec, hipStream_t s, const SignSpace &space = SignSpace()) {
  const int N = (int)p->alpha.size() - 1;
  const LaunchCfg cfg = sign_cfg<TABLE>(jobs, nj, prec);
  const int spb = cfg.spb;
  const bool slab = cfg.tiles == 2;
  // scratch: [item table] then per job [vector][norm partials][projection partials][c]
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  size_t off[kMaxBatch][4];
  size_t total = TABLE ? up(sizeof(StepItem) * nj) : 0;
  for (int j = 0; j < nj; ++j) {
    const int V = jobs[j].g->g.V, nrhs = jobs[j].nrhs;
    const int n_ev = jobs[j].d ? jobs[j].d->n_ev : 0;
    off[j][0] = total;
    total += N >= 2 ? up((size_t)nrhs * 12 * V * elem_bytes(spin_dt)) : 0;
    off[j][1] = total;
    total += up(sizeof(double) * 2 * (size_t)item_blocks(V, spb) * nrhs);
    off[j][2] = total;
    total += up(sizeof(double2) * (size_t)project_blocks(V) * nrhs * n_ev);
    off[j][3] = total;
    total += up(sizeof(double2) * (size_t)nrhs * n_ev);
  }
  if (space.fixed && total > space.fixed_cap)
    return fail(OVL_EINVAL, "the evaluation needs %zu bytes of work space, above the %zu-byte "
                "fixed buffer", total, space.fixed_cap);
  const double *wdev[kMaxBatch] = {};
  double wmax[kMaxBatch] = {};
  for (int j = 0; j < nj; ++j)
    if (jobs[j].d) {
      int rc = defl_weights(jobs[j].d, p, s, &wdev[j], &wmax[j]);
      if (rc) return rc;
    }
  Scratch sc;
  int rc = OVL_OK;
  if (!space.fixed) {
    rc = scratch_alloc(sc, total, s);
    if (rc) return rc;
  }
  char *base = space.fixed ? (char *)space.fixed : (char *)sc.p;
  // step graph for a small single problem.  The graph lock is held until the final step, which
  // reads the graph's work vector, is enqueued: an eviction by another thread frees that vector.
  std::unique_lock<std::mutex> glk(g_graph_mu, std::defer_lock);
  GraphEntry *ge = nullptr;
  if (!TABLE && !space.fixed && N >= 3 && spb < 64 && !slab && g_graphs.load() != 0) {
    GraphKey key{jobs[0].g->device, jobs[0].g->serial, p->serial, jobs[0].in, jobs[0].out,
                 jobs[0].nrhs, (int)prec, src_g5, cfg.spb, cfg.tiles, cfg.remap, cfg.rb};
    glk.lock();
    ge = graph_entry(key, (size_t)jobs[0].nrhs * 12 * jobs[0].g->g.V * elem_bytes(spin_dt));
    if (!ge) glk.unlock();
  }

  StepItem items[kMaxBatch];
  for (int j = 0; j < nj; ++j) {
    const SignJob &J = jobs[j];
    StepItem &it = items[j];
    fill_item(it, J.g, J.nrhs);
    it.psi = J.in;
    it.buf[0] = J.out;
    it.buf[1] = ge ? ge->work : base + off[j][0];
    it.norm_partial = (double *)(base + off[j][1]);
    if (J.d) {
      const int V = J.g->g.V;
      double2 *partial = (double2 *)(base + off[j][2]);
      double2 *cvec = (double2 *)(base + off[j][3]);
      if (prec == P_F64)
        rc = project((const double2 *)J.d->phi_store, J.d->n_ev, (const double2 *)J.in, src_g5,
                     J.nrhs, V, partial, project_blocks(V), cvec, s);
      else
        rc = project((const float2 *)J.d->phi_store, J.d->n_ev, (const float2 *)J.in, src_g5,
                     J.nrhs, V, partial, project_blocks(V), cvec, s);
      if (rc) return rc;
      it.phi = J.d->phi_store;
      it.n_ev = J.d->n_ev;
      it.c = cvec;
      it.wdefl = wdev[j];
    }
  }
  StepArgs<TABLE> args;
  clear_args(args);
  args.n_items = nj;
  plan_launch(args, items, nj, cfg, prec);
  args.r12 = 1;
  for (int j = 0; j < nj; ++j) args.r12 = args.r12 && items[j].r12;
  if (TABLE) {
    StepItem *table = (StepItem *)base;
    for (int j = 0; j < nj; ++j) {
      write_item_kernel<<<1, 64, 0, s>>>(items[j], table + j);
      HIP_TRY(hipGetLastError());
    }
    args.table = table;
  } else {
    args.item = items[0];
  }

  auto role = [](int k) { return (k % 2 == 0) ? ROLE_B0 : ROLE_B1; };
  const double *al = p->alpha.data();
  const double kdiag = 4.0 - p->m_W;
  // timing: one event pair around the plain steps k = N-1 .. 1 (consecutive launches)
  TimedRun run{nullptr, nullptr, N - 1};
  if (g_timing.load() != 0 && N >= 2 && !space.fixed) {
    std::lock_guard<std::mutex> lk(g_timing_mu);
    run.e0 = pool_event();
    run.e1 = pool_event();
  }
  auto set_step = [&](int k) {
    double sfac = (k == 0) ? 1.0 : 2.0;
    double a = al[k];
    if (k + 1 == N) {
      args.v_role = ROLE_PSI;
      args.v_g5 = src_g5;
      sfac *= al[N];
    } else {
      args.v_role = role(k + 1);
      args.v_g5 = 0;
    }
    args.t = 0.0;
    if (k + 2 == N + 1) {
      args.w_role = ROLE_NONE;
    } else if (k + 2 == N) {
      args.w_role = ROLE_NONE;
      a -= al[N];
    } else {
      args.w_role = role(k + 2);
      args.t = -1.0;
    }
    args.src_g5 = src_g5;
    args.a = a;
    args.y_g5 = 1;
    args.kd = sfac * kdiag / p->lmax;
    args.kh = -0.5 * sfac / p->lmax;
    args.out_role = role(k);
    args.mode = (k == 0) ? mode : MODE_STEP;
    args.mu = mu;
  };
  // plain steps k = N-1 .. 1
  if (run.e0) HIP_TRY(hipEventRecord(run.e0, s));
  if (ge && !ge->exec && !ge->failed && ge->uses >= 1) {
    // second occurrence: capture the plain steps once
    hipStream_t cs = capture_stream(jobs[0].g->device);
    if (cs && hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal) == hipSuccess) {
      for (int k = N - 1; k >= 1 && rc == OVL_OK; --k) {
        set_step(k);
        rc = dispatch_step(prec, args, cfg, cs);
      }
      hipGraph_t graph = nullptr;
      const hipError_t ec = hipStreamEndCapture(cs, &graph);
      if (rc == OVL_OK && ec == hipSuccess && graph &&
          hipGraphInstantiate(&ge->exec, graph, nullptr, nullptr, 0) != hipSuccess)
        ge->exec = nullptr;
      if (graph) (void)hipGraphDestroy(graph);
      (void)hipGetLastError();
      if (rc) return rc;
    }
    if (!ge->exec) ge->failed = true;
  }
  if (ge) ++ge->uses;
  if (ge && ge->exec) {
    HIP_TRY(hipGraphLaunch(ge->exec, s));
  } else {
    for (int k = N - 1; k >= 1; --k) {
      set_step(k);
      rc = dispatch_step(prec, args, cfg, s);
      if (rc) return rc;
    }
  }
  if (run.e0 && run.e1) {
    HIP_TRY(hipEventRecord(run.e1, s));
    std::lock_guard<std::mutex> lk(g_timing_mu);
    g_timing_events.push_back(run);
  }
  // final step: deflation correction, combine, norm partials
  set_step(0);
  rc = dispatch_step(prec, args, cfg, s);
  if (rc) return rc;
  for (int j = 0; j < nj; ++j) {
    const SignJob &J = jobs[j];
    const double bound = p->bound + (J.d ? wmax[j] : 0.0);
    norm_check_kernel<<<J.nrhs, kBlock, 0, s>>>(
        items[j].norm_partial, item_blocks(J.g->g.V, spb), J.nrhs, bound * bound, J.g->flags,
        nullptr);
    HIP_TRY(hipGetLastError());
  }
  return OVL_OK;
}

int run_sign(const ovl_gauge *g, const ovl_poly *p, ovl_defl *d, int mode, double mu, int src_g5,
             void *out, const void *in, int nrhs, int spin_dt, Prec prec, hipStream_t s) {
  SignJob j{g, d, in, out, nrhs};
  return run_sign_jobs<false>(&j, 1, p, mode, mu, src_g5, spin_dt, prec, s);
}

// the problems of a batch: every item valid, one operator precision, no output overlapping any
// input or another output (outputs are written while other items' inputs are still read)
int check_batch(const ovl_batch_item *items, int n_items, int spin_dt, SignJob *jobs,
                Prec &prec0) {
  if (!items) return fail(OVL_EINVAL, "items is NULL");
  if (n_items < 1 || n_items > kMaxBatch)
    return fail(OVL_EINVAL, "n_items = %d out of range [1, %d]", n_items, kMaxBatch);
  prec0 = P_BAD;
  for (int i = 0; i < n_items; ++i) {
    Prec prec;
    const int rc = check_spinor_call(items[i].g, items[i].out, items[i].in, items[i].nrhs,
                                     spin_dt, prec);
    if (rc) return fail(rc, "item %d: %s", i, std::string(g_err).c_str());
    if (i > 0 && prec != prec0)
      return fail(OVL_EDTYPE, "item %d: link storage differs from item 0", i);
    prec0 = prec;
    jobs[i] = SignJob{items[i].g, nullptr, items[i].in, items[i].out, items[i].nrhs};
  }
  for (int i = 0; i < n_items; ++i)
    for (int j = 0; j < n_items; ++j) {
      const size_t bi = (size_t)items[i].nrhs * 12 * items[i].g->g.V * elem_bytes(spin_dt);
      const size_t bj = (size_t)items[j].nrhs * 12 * items[j].g->g.V * elem_bytes(spin_dt);
      const char *o = (const char *)items[i].out, *x = (const char *)items[j].in;
      const char *oj = (const char *)items[j].out;
      if (o < x + bj && x < o + bi)
        return fail(OVL_EALIAS, "output of item %d overlaps the input of item %d", i, j);
      if (i != j && o < oj + bj && oj < o + bi)
        return fail(OVL_EALIAS, "outputs of items %d and %d overlap", i, j);
    }
  return OVL_OK;
}

// Tuning cache file: one entry per line,
//   B <prec> <r12> <n_items> (<Lx> <Ly> <Lz> <Lt> <nrhs>) x n_items <spb> <order> <remap> <rb> <us>
// or, for a single problem with full link reads, the short form  <Lx> <Ly> <Lz> <Lt> <prec>
// <nrhs> <spb> <order> <remap> <us>  (right-hand-side block 1).  Returns the entries read or a
// negative status.
bool cfg_valid(const LaunchCfg &c) {
  const bool ok_spb = c.tiles == 2 ? (c.spb == 64 || c.spb == 128 || c.spb == 192 || c.spb == 256)
                                   : (c.spb == 8 || c.spb == 16 || c.spb == 64 || c.spb == 128);
  return ok_spb && c.tiles >= 0 && (c.tiles <= 2 || (c.tiles == kMarch && c.spb == 64)) && rb_ok(c);
}
int load_tune_cache(const char *path) {
  FILE *f = std::fopen(path, "r");
  if (!f) return fail(OVL_EINVAL, "cannot open tuning cache %s", path);
  char line[4096];
  int n = 0;
  while (std::fgets(line, sizeof(line), f)) {
    std::vector<double> v;
    bool batch = false;
    char *q = line;
    while (*q == ' ' || *q == '\t') ++q;
    if (*q == 'B') {
      batch = true;
      ++q;
    }
    char *end = nullptr;
    for (;;) {
      const double x = std::strtod(q, &end);
      if (end == q) break;
      v.push_back(x);
      q = end;
    }
    TuneKey key;
    LaunchCfg c;
    if (batch) {
      if (v.size() < 3) continue;
      const int ni = (int)v[2];
      if (ni < 1 || ni > kMaxBatch || (int)v.size() != 3 + 5 * ni + 5) continue;
      key.prec = (int)v[0];
      key.r12 = v[1] != 0 ? 1 : 0;
      for (int i = 0; i < ni; ++i)
        key.items.push_back({(int)v[3 + 5 * i], (int)v[4 + 5 * i], (int)v[5 + 5 * i],
                             (int)v[6 + 5 * i], (int)v[7 + 5 * i]});
      const int o = 3 + 5 * ni;
      c = LaunchCfg{(int)v[o], (int)v[o + 1], v[o + 2] != 0 ? 1 : 0, (int)v[o + 3]};
    } else {
      if (v.size() != 10) continue;
      key.prec = (int)v[4];
      key.r12 = 0;
      key.items.push_back({(int)v[0], (int)v[1], (int)v[2], (int)v[3], (int)v[5]});
      c = LaunchCfg{(int)v[6], (int)v[7], v[8] != 0 ? 1 : 0, 1};
    }
    bool ok = key.prec >= 0 && key.prec <= 2 && cfg_valid(c);
    for (const auto &it : key.items) ok = ok && it[4] >= 1;
    if (!ok) continue;
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tuned[key] = c;
    ++n;
  }
  std::fclose(f);
  return n;
}
// a cache named by a batch call is read once per process
int load_tune_cache_once(const char *path) {
  static std::mutex mu;
  static std::vector<std::string> loaded;
  std::lock_guard<std::mutex> lk(mu);
  if (std::find(loaded.begin(), loaded.end(), path) != loaded.end()) return OVL_OK;
  const int n = load_tune_cache(path);
  if (n < 0) return n;
  loaded.emplace_back(path);
  return OVL_OK;
}

int check_poly(const ovl_poly *p) {
  if (!p) return fail(OVL_EINVAL, "polynomial handle is NULL");
  return OVL_OK;
}

int check_defl(const ovl_gauge *g, const ovl_defl *d, Prec prec) {
  if (!d) return OVL_OK;
  for (int i = 0; i < 4; ++i)
    if (d->g.L[i] != g->g.L[i]) return fail(OVL_EDIMS, "deflation basis and gauge field differ in extent");
  const int want = (prec == P_F64) ? OVL_F64 : OVL_F32;
  if (d->store_dt != want)
    return fail(OVL_EDTYPE, "deflation basis stored as dtype %d, operator needs %d", d->store_dt, want);
  return OVL_OK;
}

}  // namespace

// ---------------------------------------------------------------------------------------------
extern "C" {

const char *ovl_last_error(void) { return g_err; }

const char *ovl_version(void) { return "ovl 0.1 (gfx950)"; }

// plain device-memory streams of 16-byte elements (the bandwidth ceilings the kernels are
// compared with); enqueued on the caller's stream
int ovl_stream_probe(int kind, void *dst, const void *src, int64_t bytes, void *stream) {
  g_err[0] = 0;
  if (!dst || !src) return fail(OVL_EINVAL, "NULL argument");
  if (bytes <= 0 || bytes % 16 != 0) return fail(OVL_EINVAL, "bytes must be a positive multiple of 16");
  if (!aligned16(dst) || !aligned16(src)) return fail(OVL_EINVAL, "buffers must be 16-byte aligned");
  const int64_t n = bytes / 16;
  const unsigned blocks = kStreamBlocks;
  hipStream_t s = as_stream(stream);
  switch (kind) {
    case 0: stream_read_kernel<<<blocks, 256, 0, s>>>((const uint4 *)src, n, (uint32_t *)dst); break;
    case 1: stream_copy_kernel<<<blocks, 256, 0, s>>>((const uint4 *)src, n, (uint4 *)dst); break;
    case 2: stream_3to1_kernel<<<blocks, 256, 0, s>>>((const uint4 *)src, n, (uint4 *)dst); break;
    default: return fail(OVL_EINVAL, "stream kind %d", kind);
  }
  HIP_TRY(hipGetLastError());
  return OVL_OK;
}

int ovl_gauge_create(ovl_gauge **out, const int32_t dims[4], const void *U_dev, int in_dt,
                     int store_dt, void *stream) {
  g_err[0] = 0;
  if (!out || !U_dev) return fail(OVL_EINVAL, "NULL argument");
  *out = nullptr;
  Geom geo;
  int rc = check_dims(dims, geo);
  if (rc) return rc;
  if (in_dt != OVL_F64 && in_dt != OVL_F32) return fail(OVL_EDTYPE, "link input dtype %d", in_dt);
  if (store_dt != OVL_F64 && store_dt != OVL_F32 && store_dt != OVL_BF16)
    return fail(OVL_EDTYPE, "link storage dtype %d", store_dt);
  const int lstride = kLinkBlock;
  const int64_t nlink = (int64_t)(geo.V + 63) / 64 * 36 * 64;  // elements, whole blocks
  if (!fits_u32((uint64_t)nlink, store_dt))
    return fail(OVL_EDIMS, "links of %d sites exceed 4 GiB", geo.V);
  hipStream_t s = as_stream(stream);
  ovl_gauge *g = new (std::nothrow) ovl_gauge();
  if (!g) return fail(OVL_ENOMEM, "host allocation failed");
  g->g = geo;
  g->store_dt = store_dt;
  g->links = nullptr;
  g->flags = nullptr;
  g->lstride = lstride;
  g->serial = g_poly_serial.fetch_add(1);
  hipError_t e = hipGetDevice(&g->device);
  const int64_t n = (int64_t)36 * geo.V;
  const size_t lbytes = ((size_t)nlink * elem_bytes(store_dt) + 255) / 256 * 256;
  if (e == hipSuccess) e = block_cache().take_handle(lbytes + 256, s, g->mem);
  if (e == hipSuccess) {
    g->links = g->mem.p;
    g->flags = (uint32_t *)((char *)g->mem.p + lbytes);
    e = hipMemsetAsync(g->flags, 0, 256, s);
  }
  if (e == hipSuccess) {
    const int threads = 256;
    const unsigned blocks = (unsigned)((n + threads - 1) / threads);
    const int V = geo.V;
    if (in_dt == OVL_F64) {
      const double2 *src = (const double2 *)U_dev;
      if (store_dt == OVL_F64) pack_links_kernel<<<blocks, threads, 0, s>>>(src, (double2 *)g->links, V);
      else if (store_dt == OVL_F32) pack_links_kernel<<<blocks, threads, 0, s>>>(src, (float2 *)g->links, V);
      else pack_links_kernel<<<blocks, threads, 0, s>>>(src, (bf16c *)g->links, V);
    } else {
      const float2 *src = (const float2 *)U_dev;
      if (store_dt == OVL_F64) pack_links_kernel<<<blocks, threads, 0, s>>>(src, (double2 *)g->links, V);
      else if (store_dt == OVL_F32) pack_links_kernel<<<blocks, threads, 0, s>>>(src, (float2 *)g->links, V);
      else pack_links_kernel<<<blocks, threads, 0, s>>>(src, (bf16c *)g->links, V);
    }
    e = hipGetLastError();
  }
  if (e != hipSuccess) {
    (void)hipGetLastError();
    block_cache().give(g->mem, s);
    delete g;
    return fail(e == hipErrorOutOfMemory ? OVL_ENOMEM : OVL_EHIP, "gauge create: %s",
                hipGetErrorString(e));
  }
  *out = g;
  return OVL_OK;
}

int ovl_gauge_destroy(ovl_gauge *g) {
  g_err[0] = 0;
  if (!g) return OVL_OK;
  block_cache().retire(g->mem);
  delete g;
  return OVL_OK;
}

int ovl_gauge_info(const ovl_gauge *g, int32_t dims_out[4], int *store_dt) {
  if (!g || !dims_out || !store_dt) return fail(OVL_EINVAL, "NULL argument");
  for (int i = 0; i < 4; ++i) dims_out[i] = g->g.L[i];
  *store_dt = g->store_dt;
  return OVL_OK;
}

// Two-row link reads: enable after checking on the device that every stored third row matches
// the one completed from the first two (an SU(3) field up to storage rounding) within tol.
int ovl_gauge_reconstruct(ovl_gauge *g, int on, double tol, double *max_dev, void *stream) {
  g_err[0] = 0;
  if (!g) return fail(OVL_EINVAL, "gauge handle is NULL");
  if (!on) {
    if (g->r12) g->serial = g_poly_serial.fetch_add(1);  // new key for cached step graphs
    g->r12 = 0;
    if (max_dev) *max_dev = 0.0;
    return OVL_OK;
  }
  if (!(tol >= 0.0) || !std::isfinite(tol)) return fail(OVL_EINVAL, "tol must be finite and >= 0");
  const hipStream_t s = as_stream(stream);
  const int V = g->g.V;
  const int nblk = (int)(((int64_t)4 * V + 255) / 256);
  Scratch sc;
  int rc = scratch_alloc(sc, sizeof(double) * nblk, s);
  if (rc) return rc;
  double *partial = (double *)sc.p;
  if (g->store_dt == OVL_F64)
    su3_row2_dev_kernel<<<nblk, 256, 0, s>>>((const double2 *)g->links, V, partial);
  else if (g->store_dt == OVL_F32)
    su3_row2_dev_kernel<<<nblk, 256, 0, s>>>((const float2 *)g->links, V, partial);
  else
    su3_row2_dev_kernel<<<nblk, 256, 0, s>>>((const bf16c *)g->links, V, partial);
  HIP_TRY(hipGetLastError());
  std::vector<double> h(nblk);
  HIP_TRY(hipMemcpyAsync(h.data(), partial, sizeof(double) * nblk, hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  double dev = 0.0;
  for (double v : h) dev = std::isnan(v) ? v : std::max(dev, v);
  if (max_dev) *max_dev = dev;
  if (!(dev <= tol))
    return fail(OVL_EINVAL, "links are not SU(3) within %g: third rows deviate by %g", tol, dev);
  if (!g->r12) g->serial = g_poly_serial.fetch_add(1);
  g->r12 = 1;
  return OVL_OK;
}

int ovl_poly_create(ovl_poly **out, const double *alpha, int n_alpha, double lmax, double m_W) {
  g_err[0] = 0;
  if (!out || !alpha) return fail(OVL_EINVAL, "NULL argument");
  *out = nullptr;
  if (n_alpha < 2 || n_alpha > 100001)
    return fail(OVL_EINVAL, "n_alpha = %d out of range [2, 100001]", n_alpha);
  if (!std::isfinite(lmax) || !std::isfinite(m_W)) return fail(OVL_ENONFINITE, "lmax or m_W not finite");
  if (!(lmax > 0.0)) return fail(OVL_EINVAL, "lmax must be positive");
  for (int i = 0; i < n_alpha; ++i)
    if (!std::isfinite(alpha[i])) return fail(OVL_ENONFINITE, "alpha[%d] is not finite", i);
  ovl_poly *p = new (std::nothrow) ovl_poly();
  if (!p) return fail(OVL_ENOMEM, "host allocation failed");
  p->alpha.assign(alpha, alpha + n_alpha);
  p->lmax = lmax;
  p->m_W = m_W;
  // sup |p| on [-1, 1] sampled finely, plus the sum of |alpha| beyond as a hard cap
  double sup = 0.0, l1 = 0.0;
  for (double a : p->alpha) l1 += std::fabs(a);
  const int ns = std::max(4096, 16 * n_alpha);
  for (int j = 0; j <= ns; ++j) {
    const double x = std::cos(M_PI * j / ns);
    sup = std::max(sup, std::fabs(cheb_eval(p->alpha, x)));
  }
  p->bound = std::min(l1, sup * 1.05 + 1e-3);
  p->serial = g_poly_serial.fetch_add(1);
  *out = p;
  return OVL_OK;
}

int ovl_poly_destroy(ovl_poly *p) {
  delete p;
  return OVL_OK;
}

int ovl_poly_eval(const ovl_poly *p, double lambda, double *value_out) {
  if (!p || !value_out) return fail(OVL_EINVAL, "NULL argument");
  *value_out = cheb_eval(p->alpha, lambda / p->lmax);
  return OVL_OK;
}

int ovl_cheb_sign_coeffs(int degree, double eps, double *alpha_host, int *n_alpha_out) {
  g_err[0] = 0;
  if (!alpha_host || !n_alpha_out) return fail(OVL_EINVAL, "NULL argument");
  if (degree < 1 || degree > 100000) return fail(OVL_EINVAL, "degree %d out of range", degree);
  if (!(eps > 0.0 && eps < 1.0)) return fail(OVL_EINVAL, "eps must lie in (0, 1)");
  std::vector<double> a;
  if (!cheb_sign_coeffs(degree, eps, a)) return fail(OVL_EINVAL, "coefficient rule failed");
  std::memcpy(alpha_host, a.data(), sizeof(double) * a.size());
  *n_alpha_out = (int)a.size();
  return OVL_OK;
}

int ovl_defl_create(ovl_defl **out, const int32_t dims[4], const void *phi_dev, int in_dt,
                    const double *lambda, int n_ev, int store_dt, void *stream) {
  g_err[0] = 0;
  if (!out || !phi_dev || !lambda) return fail(OVL_EINVAL, "NULL argument");
  *out = nullptr;
  Geom geo;
  int rc = check_dims(dims, geo);
  if (rc) return rc;
  if (n_ev < 1 || (int64_t)n_ev > (int64_t)12 * geo.V)
    return fail(OVL_EINVAL, "n_ev = %d out of range [1, 12 V]", n_ev);
  if (in_dt != OVL_F64 && in_dt != OVL_F32) return fail(OVL_EDTYPE, "eigenvector dtype %d", in_dt);
  if (store_dt != OVL_F64 && store_dt != OVL_F32) return fail(OVL_EDTYPE, "basis storage %d", store_dt);
  for (int i = 0; i < n_ev; ++i)
    if (!std::isfinite(lambda[i])) return fail(OVL_ENONFINITE, "lambda[%d] is not finite", i);
  if (!fits_u32(12ull * geo.V, OVL_F64))
    return fail(OVL_EDIMS, "one eigenvector of %d sites exceeds 4 GiB in FP64", geo.V);
  if (store_dt == OVL_F32 && !fits_u32(12ull * geo.V * n_ev, OVL_F32))
    return fail(OVL_EDIMS, "an FP32 basis of %d vectors of %d sites exceeds 4 GiB", n_ev, geo.V);
  hipStream_t s = as_stream(stream);
  ovl_defl *d = new (std::nothrow) ovl_defl();
  if (!d) return fail(OVL_ENOMEM, "host allocation failed");
  d->g = geo;
  d->n_ev = n_ev;
  d->store_dt = store_dt;
  d->phi64 = nullptr;
  d->phi_store = nullptr;
  d->w_dev = nullptr;
  d->w_pin = nullptr;
  d->lambda.assign(lambda, lambda + n_ev);
  d->w_clock = 0;
  for (int k = 0; k < ovl_defl::kWSlots; ++k) {
    d->w_evt[k] = nullptr;
    d->w_evt_live[k] = false;
    d->w_serial[k] = 0;
    d->w_stamp[k] = 0;
    d->w_absmax[k] = 0.0;
  }
  const int V = geo.V;
  const int64_t nv = (int64_t)12 * V;  // complex entries per vector
  const int64_t n = nv * n_ev;
  auto cleanup = [&](int code) {
    if (d->phi_store && d->phi_store != d->phi64) (void)hipFree(d->phi_store);
    if (d->phi64) (void)hipFree(d->phi64);
    if (d->w_dev) (void)hipFree(d->w_dev);
    if (d->w_pin) (void)hipHostFree(d->w_pin);
    for (int k = 0; k < ovl_defl::kWSlots; ++k)
      if (d->w_evt[k]) (void)hipEventDestroy(d->w_evt[k]);
    delete d;
    return code;
  };
  const size_t wbytes = sizeof(double) * (size_t)n_ev * ovl_defl::kWSlots;
  auto alloc = [](auto **p, size_t bytes) {
    return block_cache().with_room([&] { return hipMalloc((void **)p, bytes); });
  };
  hipError_t e = alloc(&d->phi64, n * sizeof(double2));
  if (e == hipSuccess) e = alloc(&d->w_dev, wbytes);
  if (e == hipSuccess) e = hipHostMalloc((void **)&d->w_pin, wbytes, hipHostMallocDefault);
  for (int k = 0; k < ovl_defl::kWSlots && e == hipSuccess; ++k)
    e = hipEventCreateWithFlags(&d->w_evt[k], hipEventDisableTiming);
  if (e != hipSuccess)
    return cleanup(fail(e == hipErrorOutOfMemory ? OVL_ENOMEM : OVL_EHIP, "defl alloc: %s",
                        hipGetErrorString(e)));
  {
    const unsigned blocks = (unsigned)((n + 255) / 256);
    if (in_dt == OVL_F64)
      convert_kernel<<<blocks, 256, 0, s>>>((const double2 *)phi_dev, d->phi64, n);
    else
      convert_kernel<<<blocks, 256, 0, s>>>((const float2 *)phi_dev, d->phi64, n);
  }
  // CGS2 in FP64: for each vector, two passes of v -= Q (Q^+ v) against the previous ones,
  // then v /= ||v||.  norms[2j] = ||v||^2 before, norms[2j+1] = after the two passes.
  const int nblk = project_blocks(V);
  Scratch sc;
  const size_t part_bytes = sizeof(double2) * (size_t)nblk * std::max(n_ev, 1);
  rc = scratch_alloc(sc, part_bytes + sizeof(double2) * (n_ev + 1) + sizeof(double) * 2 * n_ev + 1024, s);
  if (rc) return cleanup(rc);
  double2 *partial = (double2 *)sc.p;
  double2 *cbuf = (double2 *)((char *)sc.p + part_bytes);
  double *norms = (double *)((char *)cbuf + sizeof(double2) * (n_ev + 1));
  const unsigned vblocks = (unsigned)((nv + 255) / 256);
  for (int j = 0; j < n_ev && rc == OVL_OK; ++j) {
    double2 *v = d->phi64 + (int64_t)j * nv;
    rc = project(v, 1, v, 0, 1, V, partial, nblk, cbuf, s);
    if (rc) break;
    record_kernel<<<1, 64, 0, s>>>(cbuf, norms, 2 * j);
    for (int pass = 0; pass < 2 && j > 0 && rc == OVL_OK; ++pass) {
      rc = project(d->phi64, j, v, 0, 1, V, partial, nblk, cbuf, s);
      if (rc) break;
      correct_kernel<double, double2><<<dim3(grid_blocks(V), 1), kBlock, 0, s>>>(
          v, d->phi64, j, cbuf, nullptr, -1.0, V);
    }
    if (rc) break;
    rc = project(v, 1, v, 0, 1, V, partial, nblk, cbuf, s);
    if (rc) break;
    normalize_kernel<<<vblocks, 256, 0, s>>>(v, cbuf, nv, norms, 2 * j + 1);
  }
  if (rc) return cleanup(rc);
  std::vector<double> hn(2 * n_ev);
  e = hipMemcpyAsync(hn.data(), norms, sizeof(double) * 2 * n_ev, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipGetLastError();
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return cleanup(fail(OVL_EHIP, "defl create: %s", hipGetErrorString(e)));
  for (int j = 0; j < n_ev; ++j) {
    if (!std::isfinite(hn[2 * j]) || !std::isfinite(hn[2 * j + 1]))
      return cleanup(fail(OVL_ENONFINITE, "eigenvector %d holds non-finite values", j));
    if (!(hn[2 * j] > 0.0) || hn[2 * j + 1] < 1e-20 * hn[2 * j])
      return cleanup(fail(OVL_EDEFL, "eigenvector %d is numerically dependent on the previous ones", j));
  }
  if (store_dt == OVL_F64) {
    d->phi_store = d->phi64;
  } else {
    e = alloc(&d->phi_store, n * sizeof(float2));
    if (e == hipSuccess) {
      convert_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>((const double2 *)d->phi64,
                                                                 (float2 *)d->phi_store, n);
      e = hipGetLastError();
    }
    if (e != hipSuccess) return cleanup(fail(OVL_EHIP, "defl storage copy: %s", hipGetErrorString(e)));
  }
  *out = d;
  return OVL_OK;
}

int ovl_defl_destroy(ovl_defl *d) {
  if (!d) return OVL_OK;
  (void)hipDeviceSynchronize();
  if (d->phi_store && d->phi_store != d->phi64) (void)hipFree(d->phi_store);
  (void)hipFree(d->phi64);
  (void)hipFree(d->w_dev);
  (void)hipHostFree(d->w_pin);
  for (int k = 0; k < ovl_defl::kWSlots; ++k) (void)hipEventDestroy(d->w_evt[k]);
  delete d;
  return OVL_OK;
}

int ovl_defl_basis(const ovl_defl *d, void *phi_out, void *stream) {
  if (!d || !phi_out) return fail(OVL_EINVAL, "NULL argument");
  HIP_TRY(hipMemcpyAsync(phi_out, d->phi64, sizeof(double2) * (size_t)12 * d->g.V * d->n_ev,
                         hipMemcpyDeviceToDevice, as_stream(stream)));
  return OVL_OK;
}

int ovl_wilson_apply(const ovl_gauge *g, void *out, const void *in, int nrhs, int spin_dt,
                     double m_W, int dagger, void *stream) {
  g_err[0] = 0;
  Prec prec;
  int rc = check_spinor_call(g, out, in, nrhs, spin_dt, prec);
  if (rc) return rc;
  if (!std::isfinite(m_W)) return fail(OVL_ENONFINITE, "m_W is not finite");
  StepArgs<false> p = single_args(g, nrhs);
  p.item.psi = in;
  p.item.buf[0] = out;
  p.v_role = ROLE_PSI;
  p.out_role = ROLE_B0;
  p.v_g5 = dagger ? 1 : 0;
  p.y_g5 = dagger ? 1 : 0;
  p.kd = 4.0 - m_W;
  p.kh = -0.5;
  return dispatch_single(prec, p, as_stream(stream));
}

int ovl_kernel_apply(const ovl_gauge *g, void *out, const void *in, int nrhs, int spin_dt,
                     double m_W, void *stream) {
  g_err[0] = 0;
  Prec prec;
  int rc = check_spinor_call(g, out, in, nrhs, spin_dt, prec);
  if (rc) return rc;
  if (!std::isfinite(m_W)) return fail(OVL_ENONFINITE, "m_W is not finite");
  StepArgs<false> p = single_args(g, nrhs);
  p.item.psi = in;
  p.item.buf[0] = out;
  p.v_role = ROLE_PSI;
  p.out_role = ROLE_B0;
  p.y_g5 = 1;
  p.kd = 4.0 - m_W;
  p.kh = -0.5;
  return dispatch_single(prec, p, as_stream(stream));
}

int ovl_kernel_axpby(const ovl_gauge *g, void *out, const void *in, double c, const void *src,
                     double a, const void *w, double b, int nrhs, int spin_dt, double m_W,
                     void *stream) {
  g_err[0] = 0;
  Prec prec;
  int rc = check_spinor_call(g, out, in, nrhs, spin_dt, prec);
  if (rc) return rc;
  if (!std::isfinite(m_W) || !std::isfinite(c) || !std::isfinite(a) || !std::isfinite(b))
    return fail(OVL_ENONFINITE, "non-finite coefficient");
  if (src == in || w == in) return fail(OVL_EALIAS, "src or w is the stencil input");
  StepArgs<false> p = single_args(g, nrhs);
  p.item.psi = src;
  p.item.buf[0] = const_cast<void *>(in);
  p.item.buf[1] = const_cast<void *>(w);
  p.item.buf[2] = out;
  p.v_role = ROLE_B0;
  p.w_role = w ? ROLE_B1 : ROLE_NONE;
  p.out_role = ROLE_B2;
  p.y_g5 = 1;
  p.kd = c * (4.0 - m_W);
  p.kh = -0.5 * c;
  p.a = src ? a : 0.0;
  p.t = w ? b : 0.0;
  return dispatch_single(prec, p, as_stream(stream));
}

int ovl_sign_apply(const ovl_gauge *g, const ovl_poly *p, const ovl_defl *d, void *out,
                   const void *in, int nrhs, int spin_dt, void *stream) {
  g_err[0] = 0;
  Prec prec;
  int rc = check_spinor_call(g, out, in, nrhs, spin_dt, prec);
  if (rc) return rc;
  if ((rc = check_poly(p)) || (rc = check_defl(g, d, prec))) return rc;
  return run_sign(g, p, const_cast<ovl_defl *>(d), MODE_SIGN, 0.0, 0, out, in, nrhs, spin_dt, prec,
                  as_stream(stream));
}

int ovl_overlap_apply(const ovl_gauge *g, const ovl_poly *p, const ovl_defl *d, double mu,
                      int dagger, void *out, const void *in, int nrhs, int spin_dt, void *stream) {
  g_err[0] = 0;
  Prec prec;
  int rc = check_spinor_call(g, out, in, nrhs, spin_dt, prec);
  if (rc) return rc;
  if ((rc = check_poly(p)) || (rc = check_defl(g, d, prec))) return rc;
  if (!std::isfinite(mu)) return fail(OVL_ENONFINITE, "mu is not finite");
  // D^+ psi = 1/2 ((1 + mu) psi + (1 - mu) sign(K) gamma5 psi)
  return run_sign(g, p, const_cast<ovl_defl *>(d), dagger ? MODE_OVERLAP_DAG : MODE_OVERLAP, mu,
                  dagger ? 1 : 0, out, in, nrhs, spin_dt, prec, as_stream(stream));
}

}  // extern "C"

// ---------------------------------------------------------------------------------------------
// Work space of the entry point that allocates nothing (ovl_overlap_apply_noalloc): one
// file-scope device array, present on every device the library runs on until the process ends.
// Host code never passes the array's name to a kernel or a copy: on the host it is only a
// stand-in for the symbol.  Its device address is looked up once per device, with that device
// current, and kept in g_noalloc_ptr.
namespace {
constexpr size_t kNoAllocBytes = size_t(64) << 20;
__device__ __align__(256) unsigned char scratch[kNoAllocBytes];
constexpr int kMaxDevices = 64;
std::once_flag g_noalloc_once[kMaxDevices];
void *g_noalloc_ptr[kMaxDevices];
hipError_t g_noalloc_err[kMaxDevices];

int noalloc_space(void **ptr) {
  int dev = -1;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(OVL_EINVAL, "device %d out of range", dev);
  std::call_once(g_noalloc_once[dev], [dev] {
    void *p = nullptr;
    g_noalloc_err[dev] = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    g_noalloc_ptr[dev] = g_noalloc_err[dev] == hipSuccess ? p : nullptr;
  });
  HIP_TRY(g_noalloc_err[dev]);
  if (!g_noalloc_ptr[dev]) return fail(OVL_EHIP, "no device address for the static work space");
  *ptr = g_noalloc_ptr[dev];
  return OVL_OK;
}
}  // namespace

extern "C" {

int ovl_overlap_apply_noalloc(const ovl_gauge *g, const ovl_poly *p, const ovl_defl *d, double mu,
                              int dagger, void *out, const void *in, int nrhs, int spin_dt,
                              void *stream) {
  g_err[0] = 0;
  Prec prec;
  int rc = check_spinor_call(g, out, in, nrhs, spin_dt, prec);
  if (rc) return rc;
  if ((rc = check_poly(p)) || (rc = check_defl(g, d, prec))) return rc;
  if (!std::isfinite(mu)) return fail(OVL_ENONFINITE, "mu is not finite");
  SignSpace space;
  if ((rc = noalloc_space(&space.fixed))) return rc;
  space.fixed_cap = kNoAllocBytes;
  SignJob j{g, const_cast<ovl_defl *>(d), in, out, nrhs};
  return run_sign_jobs<false>(&j, 1, p, dagger ? MODE_OVERLAP_DAG : MODE_OVERLAP, mu, dagger ? 1 : 0,
                              spin_dt, prec, as_stream(stream), space);
}

}  // extern "C"

// ---------------------------------------------------------------------------------------------
// overlap inversion
namespace {

// vectors of one solve: FP64 (double2) or FP32 (float2) complex, 12 V elements
struct SolveVecs {
  bool f64;
  int64_t n;  // complex elements
  hipStream_t s;
  double2 *partial;  // projection scratch (dot products)
  int nblk;
  double2 *cdev;
};

unsigned vec_blocks(int64_t n) { return (unsigned)((n + 255) / 256); }

int vaxpby(const SolveVecs &w, const void *x, std::complex<double> a, const void *y,
           std::complex<double> b, void *out) {
  const double2 aa = make_double2(a.real(), a.imag()), bb = make_double2(b.real(), b.imag());
  if (w.f64)
    axpby_kernel<double, double2><<<vec_blocks(w.n), 256, 0, w.s>>>(
        (const double2 *)x, aa, (const double2 *)y, bb, (double2 *)out, w.n);
  else
    axpby_kernel<float, float2><<<vec_blocks(w.n), 256, 0, w.s>>>(
        (const float2 *)x, aa, (const float2 *)y, bb, (float2 *)out, w.n);
  HIP_TRY(hipGetLastError());
  return OVL_OK;
}

// <a, b> = a^+ b with FP64 accumulation, returned to the host (synchronises the stream)
int vdot(const SolveVecs &w, const void *a, const void *b, int V, std::complex<double> &out) {
  int rc = w.f64 ? project((const double2 *)a, 1, (const double2 *)b, 0, 1, V, w.partial, w.nblk,
                           w.cdev, w.s)
                 : project((const float2 *)a, 1, (const float2 *)b, 0, 1, V, w.partial, w.nblk,
                           w.cdev, w.s);
  if (rc) return rc;
  double2 h;
  HIP_TRY(hipMemcpyAsync(&h, w.cdev, sizeof(double2), hipMemcpyDeviceToHost, w.s));
  HIP_TRY(hipStreamSynchronize(w.s));
  out = std::complex<double>(h.x, h.y);
  return OVL_OK;
}

// <a, b> = a^+ b with FP64 accumulation into the device slot dst (no synchronisation)
int vdot_dev(const SolveVecs &w, const void *a, const void *b, int V, double2 *dst) {
  return w.f64 ? project((const double2 *)a, 1, (const double2 *)b, 0, 1, V, w.partial, w.nblk,
                         dst, w.s)
               : project((const float2 *)a, 1, (const float2 *)b, 0, 1, V, w.partial, w.nblk,
                         dst, w.s);
}

// Host-side view of device scalars that lags the stream by a few launches: value i is copied
// into pinned memory behind an event, and read once the stream has passed it, so the host never
// waits for the iteration it has just enqueued.
struct ScalarLag {
  static constexpr int K = 4;
  double *pin = nullptr;
  hipEvent_t ev[K] = {};
  int live = 0;
  ~ScalarLag() {
    for (auto &e : ev)
      if (e) (void)hipEventDestroy(e);
    if (pin) (void)hipHostFree(pin);
  }
  int init() {
    HIP_TRY(hipHostMalloc((void **)&pin, sizeof(double) * K));
    for (auto &e : ev) HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    return OVL_OK;
  }
  // enqueue the copy of slot->x as value number i
  int push(const double2 *slot, int i, hipStream_t s) {
    HIP_TRY(hipMemcpyAsync(pin + i % K, &slot->x, sizeof(double), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipEventRecord(ev[i % K], s));
    return OVL_OK;
  }
  // value number i (waits for its event)
  int get(int i, double &v) {
    HIP_TRY(hipEventSynchronize(ev[i % K]));
    v = pin[i % K];
    return OVL_OK;
  }
};

// CG on D^+ D x = D^+ rhs (x = 0 on entry) in the precision of (g, d); stops when
// ||D^+ (rhs - D x)|| <= tol ||D^+ rhs|| or after max_iter iterations (each two overlap
// applications).  The CG coefficients stay on the device (slots: rr ping-pong, <p, q>); the host
// reads ||r||^2 two iterations behind the stream, so it may run up to two iterations past the
// first one that met the tolerance.  `slots` holds 3 double2, `flag` one int (cleared here).
int cgnr(const SolveVecs &w, const ovl_gauge *g, const ovl_poly *p, const ovl_defl *d, double mu,
         int dt, void *x, const void *rhs, void *r, void *pv, void *q, void *t, double tol,
         int max_iter, int &iters, double2 *slots, int *flag, void *stream) {
  iters = 0;
  const int V = g->g.V;
  hipStream_t s = w.s;
  ScalarLag lag;
  int rc = lag.init();
  if (rc) return rc;
  if ((rc = ovl_overlap_apply(g, p, d, mu, 1, r, rhs, 1, dt, stream))) return rc;  // r = D^+ rhs
  if ((rc = vaxpby(w, nullptr, 0.0, nullptr, 0.0, x))) return rc;                   // x = 0
  if ((rc = vaxpby(w, r, 1.0, nullptr, 0.0, pv))) return rc;                        // p = r
  HIP_TRY(hipMemsetAsync(flag, 0, sizeof(int), s));
  double2 *rr_slot[2] = {slots, slots + 1};
  double2 *pq = slots + 2;
  if ((rc = vdot_dev(w, r, r, V, rr_slot[0]))) return rc;
  if ((rc = lag.push(rr_slot[0], 0, s))) return rc;
  double rr0;
  if ((rc = lag.get(0, rr0))) return rc;
  if (!(rr0 > 0.0)) return OVL_OK;  // D^+ rhs = 0: x = 0 solves it
  if (!std::isfinite(rr0)) return fail(OVL_ENONFINITE, "non-finite right-hand side");
  const double stop = tol * tol * rr0;
  constexpr int kLag = 2;
  const unsigned nb = vec_blocks(w.n);
  bool done = false;
  for (int it = 0; it < max_iter && !done; ++it) {
    if ((rc = ovl_overlap_apply(g, p, d, mu, 0, t, pv, 1, dt, stream))) return rc;  // t = D p
    if ((rc = ovl_overlap_apply(g, p, d, mu, 1, q, t, 1, dt, stream))) return rc;   // q = D^+ t
    if ((rc = vdot_dev(w, pv, q, V, pq))) return rc;
    double2 *ro = rr_slot[it % 2], *rn = rr_slot[(it + 1) % 2];
    if (w.f64) {
      cg_xr_kernel<double, double2><<<nb, 256, 0, s>>>((double2 *)x, (double2 *)r, (const double2 *)pv,
                                                       (const double2 *)q, ro, pq, flag, w.n);
    } else {
      cg_xr_kernel<float, float2><<<nb, 256, 0, s>>>((float2 *)x, (float2 *)r, (const float2 *)pv,
                                                     (const float2 *)q, ro, pq, flag, w.n);
    }
    HIP_TRY(hipGetLastError());
    if ((rc = vdot_dev(w, r, r, V, rn))) return rc;
    if (w.f64)
      cg_p_kernel<double, double2><<<nb, 256, 0, s>>>((double2 *)pv, (const double2 *)r, rn, ro, w.n);
    else
      cg_p_kernel<float, float2><<<nb, 256, 0, s>>>((float2 *)pv, (const float2 *)r, rn, ro, w.n);
    HIP_TRY(hipGetLastError());
    if ((rc = lag.push(rn, it + 1, s))) return rc;
    iters = it + 1;
    if (it + 1 - kLag >= 1) {
      double v;
      if ((rc = lag.get(it + 1 - kLag, v))) return rc;
      done = v <= stop;
    }
  }
  if (!done) {  // the last values, which the loop did not read yet
    for (int i = std::max(1, iters + 1 - kLag); i <= iters && !done; ++i) {
      double v;
      if ((rc = lag.get(i, v))) return rc;
      done = v <= stop;
    }
  }
  int hflag = 0;
  HIP_TRY(hipMemcpyAsync(&hflag, flag, sizeof(int), hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  if (!done && (hflag & SOLVE_FLAG_CURVATURE))
    return fail(OVL_EDIVERGED, "CG lost positivity (<p, D^+ D p> not positive)");
  return OVL_OK;
}

// a copy of p truncated to the lowest odd degree M whose tail sum_{m > M} |alpha_m| is at most
// tol (|T_m| <= 1 on [-1, 1] bounds the truncation error by the tail); nullptr when p itself is
// needed.  The copy has its own serial (its own deflation weights).
ovl_poly *truncated_poly(const ovl_poly *p, double tol) {
  const int N = (int)p->alpha.size() - 1;
  if (!(tol > 0.0)) return nullptr;
  double tail = 0.0;
  int M = N;
  // walk down while the dropped coefficients stay within tol
  while (M > 1) {
    const double drop = std::fabs(p->alpha[M]) + (M - 1 >= 1 ? std::fabs(p->alpha[M - 1]) : 0.0);
    if (tail + drop > tol) break;
    tail += drop;
    M -= 2;
  }
  if (M >= N) return nullptr;
  ovl_poly *q = new (std::nothrow) ovl_poly();
  if (!q) return nullptr;
  q->alpha.assign(p->alpha.begin(), p->alpha.begin() + M + 1);
  q->lmax = p->lmax;
  q->m_W = p->m_W;
  q->bound = p->bound + tail;
  q->serial = g_poly_serial.fetch_add(1);
  return q;
}

}  // namespace

extern "C" {

// D[mu] x = b for one FP64 vector: defect correction in FP64 around CG on the normal equations,
// run in the precision of (g_in, d_in) (FP32 or BF16-link storage) or of (g, d) when g_in is NULL
int ovl_overlap_solve(const ovl_gauge *g, const ovl_poly *p, const ovl_defl *d, double mu,
                      void *x, const void *b, const ovl_gauge *g_in, const ovl_defl *d_in,
                      double tol, int max_iter, int *iters_out, double *resid_out, void *stream) {
  g_err[0] = 0;
  Prec prec;
  int rc = check_spinor_call(g, x, b, 1, OVL_F64, prec);
  if (rc) return rc;
  if (prec != P_F64) return fail(OVL_EDTYPE, "the outer gauge handle must store FP64 links");
  if ((rc = check_poly(p)) || (rc = check_defl(g, d, prec))) return rc;
  if (!std::isfinite(mu)) return fail(OVL_ENONFINITE, "mu is not finite");
  if (!(tol > 0.0) || max_iter < 1) return fail(OVL_EINVAL, "tol must be > 0 and max_iter >= 1");
  const ovl_gauge *gi = g_in ? g_in : g;
  const ovl_defl *di = g_in ? d_in : d;
  if (g_in) {
    if (std::memcmp(g_in->g.L, g->g.L, sizeof(g->g.L)) != 0)
      return fail(OVL_EDIMS, "inner gauge handle has other extents");
    if (g_in->store_dt == OVL_F64) return fail(OVL_EDTYPE, "inner gauge handle stores FP64 links");
    if ((rc = check_defl(g_in, d_in, P_F32))) return rc;
  }
  const bool in64 = gi->store_dt == OVL_F64;
  const int dt_in = in64 ? OVL_F64 : OVL_F32;
  hipStream_t s = as_stream(stream);
  const int V = g->g.V;
  const int64_t n = (int64_t)12 * V;
  const size_t v64 = ((size_t)n * 16 + 255) / 256 * 256;
  const size_t vin = ((size_t)n * (in64 ? 16 : 8) + 255) / 256 * 256;
  const int nblk = project_blocks(V);
  const size_t part = ((size_t)nblk * sizeof(double2) + 255) / 256 * 256;
  Scratch sc;
  if ((rc = scratch_alloc(sc, 2 * v64 + 6 * vin + part + 512, s))) return rc;
  char *base = (char *)sc.p;
  void *r64 = base, *t64 = base + v64;
  char *ib = base + 2 * v64;
  void *rhs = ib, *dx = ib + vin, *r = ib + 2 * vin, *pv = ib + 3 * vin, *q = ib + 4 * vin,
       *t = ib + 5 * vin;
  SolveVecs w64{true, n, s, (double2 *)(ib + 6 * vin), nblk, (double2 *)(ib + 6 * vin + part)};
  double2 *slots = (double2 *)(ib + 6 * vin + part + 256);  // CG scalars (3) and the flag word
  int *flag = (int *)(slots + 4);
  SolveVecs wi = w64;
  wi.f64 = in64;
  std::complex<double> z;
  if ((rc = vdot(w64, b, b, V, z))) return rc;
  const double nb = std::sqrt(z.real());
  if ((rc = vaxpby(w64, nullptr, 0.0, nullptr, 0.0, x))) return rc;
  int total = 0;
  double resid = nb > 0.0 ? 1.0 : 0.0;
  for (int outer = 0; nb > 0.0; ++outer) {
    if (outer == 0) {
      if ((rc = vaxpby(w64, b, 1.0, nullptr, 0.0, r64))) return rc;  // r = b (x = 0)
    } else {
      if ((rc = ovl_overlap_apply(g, p, d, mu, 0, t64, x, 1, OVL_F64, stream))) return rc;
      if ((rc = vaxpby(w64, b, 1.0, t64, -1.0, r64))) return rc;  // r = b - D x
    }
    if ((rc = vdot(w64, r64, r64, V, z))) return rc;
    const double rn = std::sqrt(z.real());
    resid = rn / nb;
    if (resid <= tol || total >= max_iter || outer >= 40) break;
    // inner solve of D dx = r / |r| in the inner precision
    if (in64)
      scale_convert_kernel<double2, double2><<<vec_blocks(n), 256, 0, s>>>((const double2 *)r64, (double2 *)rhs, 1.0 / rn, n);
    else
      scale_convert_kernel<double2, float2><<<vec_blocks(n), 256, 0, s>>>((const double2 *)r64, (float2 *)rhs, 1.0 / rn, n);
    HIP_TRY(hipGetLastError());
    const double floor = in64 ? 1e-14 : 1e-5;
    const double tol_in = std::min(0.1, std::max(0.5 * tol / resid, floor));
    int its = 0;
    if ((rc = cgnr(wi, gi, p, di, mu, dt_in, dx, rhs, r, pv, q, t, tol_in, max_iter - total, its,
                   slots, flag, stream)))
      return rc;
    total += its;
    if (in64)
      accumulate_kernel<double2><<<vec_blocks(n), 256, 0, s>>>((double2 *)x, (const double2 *)dx, rn, n);
    else
      accumulate_kernel<float2><<<vec_blocks(n), 256, 0, s>>>((double2 *)x, (const float2 *)dx, rn, n);
    HIP_TRY(hipGetLastError());
  }
  if (iters_out) *iters_out = total;
  if (resid_out) *resid_out = resid;
  if (!(resid <= tol)) return fail(OVL_EDIVERGED, "relative residual %.3e > %.3e after %d iterations", resid, tol, total);
  return OVL_OK;
}

// D[mu] x = b by GMRESR (generalised conjugate residuals with a variable preconditioner): each
// outer step solves D z = r approximately with CG on the normal equations in the inner precision
// and with a truncated ("relaxed") polynomial, forms c = D z in FP64, orthogonalises c against the
// previous directions (classical Gram-Schmidt twice; z follows with the same coefficients),
// normalises, and takes x += <c, r> z, r -= <c, r> c.  All coefficients stay on the device; the
// host reads ||r|| once per outer step.  With relax, the outer product of step k uses the
// polynomial truncated at tail 0.1 tol ||b|| / ||r_k|| (coarser as the residual falls).  The
// final residual is recomputed with the full polynomial; if it misses tol, GMRESR restarts from
// x without relaxation (at most 3 cycles).
int ovl_overlap_solve_gmresr(const ovl_gauge *g, const ovl_poly *p, const ovl_defl *d, double mu,
                             void *x, const void *b, const ovl_gauge *g_in, const ovl_defl *d_in,
                             double tol, double inner_tol, double inner_poly_tol, int relax,
                             int max_outer, int max_inner, int *outer_out, int *inner_out,
                             double *resid_out, void *stream) {
  g_err[0] = 0;
  Prec prec;
  int rc = check_spinor_call(g, x, b, 1, OVL_F64, prec);
  if (rc) return rc;
  if (prec != P_F64) return fail(OVL_EDTYPE, "the outer gauge handle must store FP64 links");
  if ((rc = check_poly(p)) || (rc = check_defl(g, d, prec))) return rc;
  if (!std::isfinite(mu) || !std::isfinite(tol) || !std::isfinite(inner_tol) ||
      !std::isfinite(inner_poly_tol))
    return fail(OVL_ENONFINITE, "non-finite mu or tolerance");
  if (!(tol > 0.0) || !(inner_tol > 0.0 && inner_tol < 1.0) || !(inner_poly_tol >= 0.0) ||
      max_outer < 1 || max_outer > 1024 || max_inner < 1)
    return fail(OVL_EINVAL, "need tol > 0, 0 < inner_tol < 1, inner_poly_tol >= 0, "
                "1 <= max_outer <= 1024, max_inner >= 1");
  const ovl_gauge *gi = g_in ? g_in : g;
  const ovl_defl *di = g_in ? d_in : d;
  if (g_in) {
    if (std::memcmp(g_in->g.L, g->g.L, sizeof(g->g.L)) != 0)
      return fail(OVL_EDIMS, "inner gauge handle has other extents");
    if (g_in->store_dt == OVL_F64) return fail(OVL_EDTYPE, "inner gauge handle stores FP64 links");
    if ((rc = check_defl(g_in, d_in, P_F32))) return rc;
  }
  const bool in64 = gi->store_dt == OVL_F64;
  const int dt_in = in64 ? OVL_F64 : OVL_F32;
  hipStream_t s = as_stream(stream);
  const int V = g->g.V;
  const int64_t n = (int64_t)12 * V;
  auto up = [](size_t v) { return (v + 255) / 256 * 256; };
  const size_t v64 = up((size_t)n * 16), vin = up((size_t)n * (in64 ? 16 : 8));
  const int nblk = project_blocks(V);
  const size_t part = up((size_t)nblk * max_outer * sizeof(double2));
  const size_t slot_bytes = up(sizeof(double2) * (size_t)(max_outer + 8) + 64);
  // direction bases C and Z: max_outer vectors each, exactly n elements apart (the projection
  // kernels read a basis as one [m][12][V] array)
  const size_t vb = up((size_t)max_outer * n * sizeof(double2));
  Scratch sc;
  if ((rc = scratch_alloc(sc, 2 * v64 + 2 * vb + 6 * vin + part + slot_bytes, s))) return rc;
  char *base = (char *)sc.p;
  double2 *r64 = (double2 *)base, *t64 = (double2 *)(base + v64);
  double2 *Cb = (double2 *)(base + 2 * v64), *Zb = (double2 *)(base + 2 * v64 + vb);
  char *ib = base + 2 * v64 + 2 * vb;
  void *rhs = ib, *dz = ib + vin, *r = ib + 2 * vin, *pv = ib + 3 * vin, *q = ib + 4 * vin,
       *t = ib + 5 * vin;
  double2 *partial = (double2 *)(ib + 6 * vin);
  double2 *slots = (double2 *)(ib + 6 * vin + part);
  // slots: [0, max_outer) Gram-Schmidt coefficients, then |c|^2, <c, r>, |r|^2, CG scalars (3)
  double2 *beta = slots, *cnrm = slots + max_outer, *alph = cnrm + 1, *rr = cnrm + 2,
          *cg_slots = cnrm + 3;
  int *flag = (int *)(cnrm + 7);
  SolveVecs w64{true, n, s, partial, nblk, rr};
  SolveVecs wi = w64;
  wi.f64 = in64;
  const unsigned nb64 = vec_blocks(n);
  // polynomials: the inner one truncated at inner_poly_tol; relaxed outer ones by truncation level
  std::vector<std::unique_ptr<ovl_poly>> owned;
  const ovl_poly *p_in = p;
  if (ovl_poly *q0 = truncated_poly(p, inner_poly_tol)) {
    owned.emplace_back(q0);
    p_in = q0;
  }
  std::map<int, const ovl_poly *> relaxed;  // truncation exponent -> polynomial
  auto outer_poly = [&](double tail) -> const ovl_poly * {
    if (!(tail > 0.0)) return p;
    const int e = (int)std::floor(std::log10(std::min(tail, 0.1)));  // tails 10^e
    auto it = relaxed.find(e);
    if (it != relaxed.end()) return it->second;
    const ovl_poly *pp = p;
    if (ovl_poly *q1 = truncated_poly(p, std::pow(10.0, e))) {
      owned.emplace_back(q1);
      pp = q1;
    }
    relaxed[e] = pp;
    return pp;
  };
  auto host_norm = [&](const void *a, double &out) -> int {
    std::complex<double> z;
    int e = vdot(w64, a, a, V, z);
    out = std::sqrt(std::max(0.0, z.real()));
    return e;
  };
  double nb;
  if ((rc = host_norm(b, nb))) return rc;
  if (!std::isfinite(nb)) return fail(OVL_ENONFINITE, "non-finite right-hand side");
  if ((rc = vaxpby(w64, nullptr, 0.0, nullptr, 0.0, x))) return rc;
  int outer = 0, inner = 0;
  double resid = nb > 0.0 ? 1.0 : 0.0;
  for (int cycle = 0; cycle < 3 && nb > 0.0; ++cycle) {
    // r = b - D x (full polynomial)
    if (cycle == 0) {
      if ((rc = vaxpby(w64, b, 1.0, nullptr, 0.0, r64))) return rc;
    } else {
      if ((rc = ovl_overlap_apply(g, p, d, mu, 0, t64, x, 1, OVL_F64, stream))) return rc;
      if ((rc = vaxpby(w64, b, 1.0, t64, -1.0, r64))) return rc;
    }
    double rn;
    if ((rc = host_norm(r64, rn))) return rc;
    if (rn / nb <= tol) {
      resid = rn / nb;
      break;
    }
    const bool rel = relax != 0 && cycle == 0;
    for (int k = 0; k < max_outer && rn / nb > tol && inner < max_inner; ++k) {
      // inner: D z ~ r / |r| in the inner precision with the truncated polynomial
      if (in64)
        scale_convert_kernel<double2, double2><<<nb64, 256, 0, s>>>(r64, (double2 *)rhs, 1.0 / rn, n);
      else
        scale_convert_kernel<double2, float2><<<nb64, 256, 0, s>>>(r64, (float2 *)rhs, 1.0 / rn, n);
      HIP_TRY(hipGetLastError());
      int its = 0;
      if ((rc = cgnr(wi, gi, p_in, di, mu, dt_in, dz, rhs, r, pv, q, t, inner_tol,
                     max_inner - inner, its, cg_slots, flag, stream)))
        return rc;
      inner += its;
      double2 *ck = Cb + (size_t)k * n;
      double2 *zk = Zb + (size_t)k * n;
      if (in64)
        scale_convert_kernel<double2, double2><<<nb64, 256, 0, s>>>((const double2 *)dz, zk, 1.0, n);
      else
        scale_convert_kernel<float2, double2><<<nb64, 256, 0, s>>>((const float2 *)dz, zk, 1.0, n);
      HIP_TRY(hipGetLastError());
      // c = D z in FP64 (relaxed: truncated polynomial)
      const ovl_poly *pk = rel ? outer_poly(0.1 * tol * nb / rn) : p;
      if ((rc = ovl_overlap_apply(g, pk, d, mu, 0, ck, zk, 1, OVL_F64, stream))) return rc;
      // classical Gram-Schmidt twice against the previous directions
      HIP_TRY(hipMemsetAsync(flag, 0, sizeof(int), s));
      for (int pass = 0; pass < 2 && k > 0; ++pass) {
        if ((rc = project(Cb, k, ck, 0, 1, V, partial, nblk, beta, s))) return rc;
        gcr_orth_kernel<<<nb64, 256, 0, s>>>(ck, Cb, k, beta, n);
        HIP_TRY(hipGetLastError());
        gcr_orth_kernel<<<nb64, 256, 0, s>>>(zk, Zb, k, beta, n);
        HIP_TRY(hipGetLastError());
      }
      if ((rc = project(ck, 1, ck, 0, 1, V, partial, nblk, cnrm, s))) return rc;
      gcr_normalise_kernel<<<nb64, 256, 0, s>>>(ck, zk, cnrm, flag, n);
      HIP_TRY(hipGetLastError());
      if ((rc = project(ck, 1, r64, 0, 1, V, partial, nblk, alph, s))) return rc;
      gcr_update_kernel<<<nb64, 256, 0, s>>>((double2 *)x, r64, zk, ck, alph, n);
      HIP_TRY(hipGetLastError());
      ++outer;
      if ((rc = host_norm(r64, rn))) return rc;
      int hflag = 0;
      HIP_TRY(hipMemcpyAsync(&hflag, flag, sizeof(int), hipMemcpyDeviceToHost, s));
      HIP_TRY(hipStreamSynchronize(s));
      if (hflag) return fail(OVL_EDIVERGED, "GMRESR direction %d is dependent on the previous ones", k);
    }
    // the true residual with the full polynomial
    if ((rc = ovl_overlap_apply(g, p, d, mu, 0, t64, x, 1, OVL_F64, stream))) return rc;
    if ((rc = vaxpby(w64, b, 1.0, t64, -1.0, r64))) return rc;
    double tn;
    if ((rc = host_norm(r64, tn))) return rc;
    resid = tn / nb;
    if (resid <= tol || inner >= max_inner) break;
  }
  if (outer_out) *outer_out = outer;
  if (inner_out) *inner_out = inner;
  if (resid_out) *resid_out = resid;
  if (!(resid <= tol))
    return fail(OVL_EDIVERGED, "relative residual %.3e > %.3e after %d outer / %d inner iterations",
                resid, tol, outer, inner);
  return OVL_OK;
}

int ovl_batch_sign_apply(const ovl_batch_item *items, int n_items, const ovl_poly *p,
                         int spin_dt, const char *tune_cache_path, void *stream) {
  g_err[0] = 0;
  int rc = check_poly(p);
  if (rc) return rc;
  SignJob jobs[kMaxBatch];
  Prec prec;
  if ((rc = check_batch(items, n_items, spin_dt, jobs, prec))) return rc;
  if (tune_cache_path && (rc = load_tune_cache_once(tune_cache_path))) return rc;
  return run_sign_jobs<true>(jobs, n_items, p, MODE_SIGN, 0.0, 0, spin_dt, prec,
                             as_stream(stream));
}

int ovl_defl_project(const ovl_defl *d, double *c_dev, const void *in, int nrhs, int spin_dt,
                     void *stream) {
  g_err[0] = 0;
  if (!d || !c_dev || !in) return fail(OVL_EINVAL, "NULL argument");
  if (nrhs < 1 || nrhs > 65535) return fail(OVL_EINVAL, "nrhs = %d out of range", nrhs);
  const int want = spin_dt;
  if (want != d->store_dt) return fail(OVL_EDTYPE, "spinor dtype %d differs from basis storage %d", spin_dt, d->store_dt);
  hipStream_t s = as_stream(stream);
  const int V = d->g.V;
  const int nblk = project_blocks(V);
  Scratch sc;
  int rc = scratch_alloc(sc, sizeof(double2) * (size_t)nblk * nrhs * d->n_ev, s);
  if (rc) return rc;
  if (spin_dt == OVL_F64)
    return project((const double2 *)d->phi_store, d->n_ev, (const double2 *)in, 0, nrhs, V,
                   (double2 *)sc.p, nblk, (double2 *)c_dev, s);
  return project((const float2 *)d->phi_store, d->n_ev, (const float2 *)in, 0, nrhs, V,
                 (double2 *)sc.p, nblk, (double2 *)c_dev, s);
}

int ovl_defl_correct(const ovl_defl *d, void *inout, const double *c_dev, const double *w_host,
                     int nrhs, int spin_dt, void *stream) {
  g_err[0] = 0;
  if (!d || !c_dev || !inout || !w_host) return fail(OVL_EINVAL, "NULL argument");
  if (nrhs < 1 || nrhs > 65535) return fail(OVL_EINVAL, "nrhs = %d out of range", nrhs);
  if (spin_dt != d->store_dt) return fail(OVL_EDTYPE, "spinor dtype %d differs from basis storage %d", spin_dt, d->store_dt);
  for (int i = 0; i < d->n_ev; ++i)
    if (!std::isfinite(w_host[i])) return fail(OVL_ENONFINITE, "w[%d] is not finite", i);
  hipStream_t s = as_stream(stream);
  const int V = d->g.V;
  // the weights travel in the kernel arguments, kWChunk per launch: nothing is staged on the
  // device and the call returns without waiting
  for (int e0 = 0; e0 < d->n_ev; e0 += kWChunk) {
    const int ne = std::min(kWChunk, d->n_ev - e0);
    WChunk w;
    for (int k = 0; k < kWChunk; ++k) w.v[k] = k < ne ? w_host[e0 + k] : 0.0;
    const int64_t n = (int64_t)12 * V;
    auto go = [&](auto kernel, auto *io, const auto *phi, int rb, int el) {
      const dim3 grid((unsigned)((n + kBlock * el - 1) / (kBlock * el)), (unsigned)((nrhs + rb - 1) / rb));
      kernel<<<grid, kBlock, 0, s>>>(io, phi, e0, ne, d->n_ev, nrhs, (const double2 *)c_dev, w, n);
    };
    // Right-hand sides per thread: the smallest of 1, 4, 16 that holds them (16 a pass beyond).  16 need 800
    // workgroups, else the multiply-adds of a thread are the launch's time: 24 FP64 modes, 16 right-hand
    // sides at 16 / 4: 256 sites 25 / 11 us, 8^3 x 16 34 / 21 (12 and 28 without passes of right-hand sides).
    // FP32 components are 8 bytes: two a thread on large lattices, for loads in flight (4 right-hand sides of
    // 16^3 x 32, 1 mode: 21.7 -> 18.8 us; FP64 components are 16 bytes and gain nothing).
    auto pick = [&](auto zero, auto *io, const auto *phi) {
      using C = decltype(zero);
      using SE = std::remove_reference_t<decltype(*io)>;
      const int64_t blocks = (n + kBlock - 1) / kBlock;
      const bool two = sizeof(C) == 4 && blocks >= 4096;
      if (nrhs == 1 && two) go(correct_w_kernel<C, SE, 1, 2>, io, phi, 1, 2);
      else if (nrhs == 1) go(correct_w_kernel<C, SE, 1, 1>, io, phi, 1, 1);
      else if (nrhs <= 4 && two) go(correct_w_kernel<C, SE, 4, 2>, io, phi, 4, 2);
      else if (nrhs <= 4 || blocks * ((nrhs + 15) / 16) < 800) go(correct_w_kernel<C, SE, 4, 1>, io, phi, 4, 1);
      else go(correct_w_kernel<C, SE, 16, 1>, io, phi, 16, 1);
    };
    if (spin_dt == OVL_F64) pick(0.0, (double2 *)inout, (const double2 *)d->phi_store);
    else pick(0.0f, (float2 *)inout, (const float2 *)d->phi_store);
    HIP_TRY(hipGetLastError());
  }
  return OVL_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------------------------
// link derivatives
namespace {

// One VJP launch over up to two runs of pairs: len0 pairs from (a0, t0), then len - len0 from
// (a1, t1), consecutive pairs step_bytes apart within a run; the first pair carries weight
// coef_first, the others coef_rest.  The sum starts from zero (in_mode 0), from the FP64 running
// buffer G64 (1) or from G (2), and goes to G64 (out_mode 0) or to G (1).  For FP64 spinors G64
// may be G itself.
int launch_vjp(Prec prec, const ovl_gauge *g, void *G, double2 *G64, const void *a0,
               const void *a1, int a_g5, const void *t0, const void *t1, size_t step_bytes,
               int len0, int len, double coef_first, double coef_rest, int in_mode, int out_mode,
               hipStream_t s) {
  if (len <= 0) return OVL_OK;
  const dim3 grid((unsigned)((g->g.V + 63) / 64));
  TimedRun run{nullptr, nullptr, 1, TK_VJP};
  if (g_timing.load() != 0) {
    std::lock_guard<std::mutex> lk(g_timing_mu);
    run.e0 = pool_event();
    run.e1 = pool_event();
  }
  if (run.e0) HIP_TRY(hipEventRecord(run.e0, s));
  // t-streaming tile order where the lattice allows it (whole tiles of 64 sites)
  int ty = 0, tz = 0;
  step_tile(g->g, 64, 2 * 96, ty, tz);
  switch (prec) {
    case P_F64:
      link_vjp_kernel<double, double2, double2><<<grid, 256, 0, s>>>(
          (double2 *)G, G64, (const double2 *)a0, (const double2 *)a1,
          (int64_t)(step_bytes / sizeof(double2)), (const double2 *)t0, (const double2 *)t1,
          (int64_t)(step_bytes / sizeof(double2)), len0, len, coef_first, coef_rest, g->g, a_g5,
          in_mode, out_mode, ty, tz);
      break;
    case P_F32:
    case P_F32_BF16:
      link_vjp_kernel<float, float2, float2><<<grid, 256, 0, s>>>(
          (float2 *)G, G64, (const float2 *)a0, (const float2 *)a1,
          (int64_t)(step_bytes / sizeof(float2)), (const float2 *)t0, (const float2 *)t1,
          (int64_t)(step_bytes / sizeof(float2)), len0, len, coef_first, coef_rest, g->g, a_g5,
          in_mode, out_mode, ty, tz);
      break;
    default:
      return fail(OVL_EDTYPE, "bad precision");
  }
  HIP_TRY(hipGetLastError());
  if (run.e0 && run.e1) {
    HIP_TRY(hipEventRecord(run.e1, s));
    std::lock_guard<std::mutex> lk(g_timing_mu);
    g_timing_events.push_back(run);
  }
  return OVL_OK;
}

// Pairs per link-VJP launch of a force that keeps every t_m: fewer launches read and write the running
// sum of G (FP64, 1152 bytes a site) less often; beyond 64 it is below 2% of a launch's bytes.
constexpr int kForcePairs = 64;

// Whether a force may take `bytes` of work space to keep every t_m: a tenth of the device's memory (read
// once per device: hipMemGetInfo has stalled the host for 10 ms and more here); the allocation itself
// tells whether they are free.  Not while the stream is captured: the graph would hold them.
bool force_may_keep(size_t bytes, hipStream_t s) {
  static std::once_flag once[64];
  static size_t total[64];
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  int dev = -1;
  if (hipStreamIsCapturing(s, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone ||
      hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
    (void)hipGetLastError();
    return false;
  }
  std::call_once(once[dev], [dev] {
    if (hipDeviceTotalMem(&total[dev], dev) != hipSuccess) {
      (void)hipGetLastError();
      total[dev] = 0;
    }
  });
  return bytes <= total[dev] / 10;
}

}  // namespace

extern "C" {

int ovl_wilson_link_vjp(const ovl_gauge *g, void *G, const void *chi, const void *psi, int spin_dt,
                        int accumulate, void *stream) {
  g_err[0] = 0;
  Prec prec;
  if (!G) return fail(OVL_EINVAL, "G is NULL");
  int rc = check_spinor_call(g, G, chi, 1, spin_dt, prec);
  if (rc == OVL_EALIAS) return fail(OVL_EALIAS, "G overlaps chi");
  if (rc) return rc;
  if (!psi) return fail(OVL_EINVAL, "psi is NULL");
  if (!fits_u32(36ull * g->g.V, spin_dt)) return fail(OVL_EDIMS, "G exceeds 4 GiB");
  return launch_vjp(prec, g, G, nullptr, chi, chi, 0, psi, psi, 0, 1, 1, 1.0, 1.0,
                    accumulate ? 2 : 0, 1, as_stream(stream));
}

// dL = Re[<b_1, dX t_0> + 2 sum_{m=1}^{N-1} <b_{m+1}, dX t_m>] with b the Clenshaw vectors of chi
// and t_m = T_m(X) psi; dX = gamma5 dD_W / lmax.  Forward sweep keeps (t_{js}, t_{js+1}) for every
// segment j of length s; the backward sweep walks the segments from the top, regenerates the
// segment's t_m, and advances b_k = alpha_k chi + 2 X b_{k+1} - b_{k+2} downwards.
int ovl_sign_force(const ovl_gauge *g, const ovl_poly *p, void *G, const void *chi,
                   const void *psi, int ckpt_stride, int spin_dt, void *stream) {
  g_err[0] = 0;
  Prec prec;
  if (!G || !chi || !psi) return fail(OVL_EINVAL, "NULL argument");
  int rc = check_spinor_call(g, G, psi, 1, spin_dt, prec);
  if (rc == OVL_EALIAS) return fail(OVL_EALIAS, "G overlaps psi");
  if (rc) return rc;
  if ((rc = check_poly(p))) return rc;
  if (!fits_u32(36ull * g->g.V, OVL_F64))
    return fail(OVL_EDIMS, "the FP64 sum of G over %d sites exceeds 4 GiB", g->g.V);
  if (ckpt_stride < 0) return fail(OVL_EINVAL, "ckpt_stride must be >= 0");
  const int N = (int)p->alpha.size() - 1;
  hipStream_t s = as_stream(stream);
  const size_t vec = (size_t)12 * g->g.V * elem_bytes(spin_dt);
  const size_t vecp = (vec + 255) / 256 * 256;
  const bool f64 = prec == P_F64;
  // Work space of a segment length: checkpoints, the segment buffer of S vectors (+1 spare), a ring of
  // S + 2 Clenshaw vectors and, for FP32 spinors, the FP64 running sum of G across the segments.
  // `keep`: every t_m has a slot of its own (nothing is regenerated, no segment buffer).
  int S = 0, R = 0, nseg = 0, nslot = 0;
  std::vector<int> slot_of;
  size_t nvec = 0, g64_bytes = 0;
  auto plan = [&](int stride, bool keep) {
    S = std::max(1, std::min(stride, N));
    R = S + 2;
    nseg = (N + S - 1) / S;  // segments cover m = 0 .. N-1
    // checkpoint slots: t_{jS} and t_{jS+1} of every segment j (distinct m only, m <= N-1)
    slot_of.assign(N + 1, -1);
    nslot = 0;
    for (int j = 0; j < nseg; ++j)
      for (int m = j * S; m <= (keep ? j * S + S - 1 : j * S + 1) && m <= N - 1; ++m)
        if (slot_of[m] < 0) slot_of[m] = nslot++;
    nvec = (size_t)nslot + (keep ? 0 : S + 1) + R;
    g64_bytes = (!f64 && nseg > 1) ? (size_t)36 * g->g.V * sizeof(double2) : 0;
  };
  // Without a stride from the caller all t_m are kept where they take at most a tenth of the device's
  // memory: the backward sweep then regenerates nothing (24^3 x 48 FP32, degree 299: 23 GB, 94.9 -> 77.5
  // ms).  Otherwise, or where the allocation fails, checkpoints every ceil(sqrt N).
  Scratch sc;
  bool keep = false;
  if (ckpt_stride == 0) {
    plan(kForcePairs, true);
    const size_t bytes = nvec * vecp + g64_bytes;
    if (force_may_keep(bytes, s)) {
      rc = scratch_alloc(sc, bytes, s);
      keep = rc == OVL_OK;
      if (rc != OVL_OK && rc != OVL_ENOMEM) return rc;
    }
  }
  if (!keep) {
    plan(ckpt_stride > 0 ? ckpt_stride : (int)std::ceil(std::sqrt((double)N)), false);
    if ((rc = scratch_alloc(sc, nvec * vecp + g64_bytes, s))) return rc;
  }
  char *base = (char *)sc.p;
  double2 *G64 = f64 ? (double2 *)G : (g64_bytes ? (double2 *)(base + nvec * vecp) : nullptr);
  auto ck = [&](int m) -> void * { return base + (size_t)slot_of[m] * vecp; };
  auto seg = [&](int i) -> void * { return base + ((size_t)nslot + i) * vecp; };
  // b_k lives in ring slot k mod R: a segment touches b_{m0} .. b_{m1+2}, at most S + 2 vectors
  char *ring = base + ((size_t)nslot + (keep ? 0 : S + 1)) * vecp;
  auto bv = [&](int k) -> void * { return ring + (size_t)(k % R) * vecp; };
  const double kdiag = 4.0 - p->m_W;
  const double *al = p->alpha.data();
  // X applied: out = sx * X v + a * src + t * w
  auto xstep = [&](void *out, const void *v, double sx, const void *src, double a, const void *w,
                   double t) -> int {
    StepArgs<false> sp = single_args(g, 1);
    sp.item.psi = src;
    sp.item.buf[0] = const_cast<void *>(v);
    sp.item.buf[1] = const_cast<void *>(w);
    sp.item.buf[2] = out;
    sp.v_role = ROLE_B0;
    sp.w_role = w ? ROLE_B1 : ROLE_NONE;
    sp.out_role = ROLE_B2;
    sp.y_g5 = 1;
    sp.kd = sx * kdiag / p->lmax;
    sp.kh = -0.5 * sx / p->lmax;
    sp.a = src ? a : 0.0;
    sp.t = t;
    return dispatch_single(prec, sp, s);
  };
  // two such steps with the same stencil weight sx and w coefficient t in one launch (the twin
  // recurrence: both read every link once): out = sx X v + a src + t w, out2 likewise
  auto xstep2 = [&](void *out, const void *v, const void *src, double a, const void *w,
                    void *out2, const void *v2, const void *src2, double a2, const void *w2,
                    double sx, double t) -> int {
    StepArgs<false> sp = single_args(g, 2);
    sp.item.twin = 1;
    sp.item.psi = src;
    sp.item.buf[0] = const_cast<void *>(v);
    sp.item.buf[1] = const_cast<void *>(w);
    sp.item.buf[2] = out;
    sp.item.twin_psi = src2;
    sp.item.twin_buf[0] = const_cast<void *>(v2);
    sp.item.twin_buf[1] = const_cast<void *>(w2);
    sp.item.twin_buf[2] = out2;
    sp.item.twin_a = src2 ? a2 : 0.0;
    sp.v_role = ROLE_B0;
    sp.w_role = ROLE_B1;
    sp.out_role = ROLE_B2;
    sp.y_g5 = 1;
    sp.kd = sx * kdiag / p->lmax;
    sp.kh = -0.5 * sx / p->lmax;
    sp.a = src ? a : 0.0;
    sp.t = t;
    return dispatch_single(prec, sp, s);
  };
  // forward sweep: t_0 = psi, t_1 = X psi, t_{m+1} = 2 X t_m - t_{m-1}, keeping the checkpoint
  // vectors; the others rotate through seg(0), seg(1) (never the buffer read as stencil input).
  // It stops at the last checkpoint: the top segment is regenerated by the backward sweep.
  int last_ck = 0;
  for (int m = 0; m <= N - 1; ++m)
    if (slot_of[m] >= 0) last_ck = m;
  HIP_TRY(hipMemcpyAsync(ck(0), psi, vec, hipMemcpyDeviceToDevice, s));
  if (last_ck >= 1) {
    void *t1 = slot_of[1] >= 0 ? ck(1) : seg(0);
    if ((rc = xstep(t1, psi, 1.0, nullptr, 0.0, nullptr, 0.0))) return rc;
    const void *tm1 = ck(0);
    const void *tm = t1;
    int which = (t1 == seg(0)) ? 1 : 0;
    for (int m = 1; m + 1 <= last_ck; ++m) {  // produce t_{m+1} up to the last checkpoint
      void *dst;
      if (slot_of[m + 1] >= 0) {
        dst = ck(m + 1);
      } else {
        dst = seg(which);
        which ^= 1;
      }
      if ((rc = xstep(dst, tm, 2.0, nullptr, 0.0, tm1, -1.0))) return rc;
      tm1 = tm;
      tm = dst;
    }
  }
  // backward sweep, segments from the top.  b_{N+1} = 0 is never formed: the steps that would
  // read it drop that term.  b_N = alpha_N chi (a step whose stencil term has weight zero).
  if ((rc = xstep(bv(N), chi, 0.0, chi, al[N], nullptr, 0.0))) return rc;
  for (int j = nseg - 1; j >= 0; --j) {
    const int m0 = j * S;
    const int m1 = std::min(N - 1, m0 + S - 1);
    // regenerate t_{m0} .. t_{m1} into seg(0..) (ascending) and advance
    // b_m = alpha_m chi + 2 X b_{m+1} - b_{m+2} for m = m1 .. max(m0, 1) (descending; b_{m1+1}
    // and b_{m1+2} come from the segment above or the start values).  The two recurrences are
    // independent, so their steps run as twins, one launch per pair of steps.
    int mt = m0 + 2, mb = m1;
    if (keep) {
      mt = m1 + 1;  // t_{m0} .. t_{m1} are there (consecutive slots)
    } else {
      HIP_TRY(hipMemcpyAsync(seg(0), ck(m0), vec, hipMemcpyDeviceToDevice, s));
      if (m1 >= m0 + 1) HIP_TRY(hipMemcpyAsync(seg(1), ck(m0 + 1), vec, hipMemcpyDeviceToDevice, s));
    }
    const int mb_end = std::max(m0, 1);
    while (mt <= m1 || mb >= mb_end) {
      // b_{N-1} has no b_{N+1} term: it runs alone (the twins share the w coefficient)
      const bool b_next = mb >= mb_end;
      const bool b_w = b_next && mb + 2 <= N;
      if (mt <= m1 && b_w) {
        rc = xstep2(seg(mt - m0), seg(mt - m0 - 1), nullptr, 0.0, seg(mt - m0 - 2),
                    bv(mb), bv(mb + 1), chi, al[mb], bv(mb + 2), 2.0, -1.0);
        ++mt;
        --mb;
      } else if (b_next) {
        rc = xstep(bv(mb), bv(mb + 1), 2.0, chi, al[mb], b_w ? bv(mb + 2) : nullptr, -1.0);
        --mb;
      } else {
        rc = xstep(seg(mt - m0), seg(mt - m0 - 1), 2.0, nullptr, 0.0, seg(mt - m0 - 2), -1.0);
        ++mt;
      }
      if (rc) return rc;
    }
    // pairs (b_{m+1}, t_m), m = m0 .. m1, in one launch: the ring slots of b_{m0+1} .. b_{m1+1}
    // are consecutive up to one wrap (a segment holds at most S < R pairs), so they form at most
    // two runs; the t_m are consecutive in the segment buffer
    const int len = m1 - m0 + 1;
    const int len0 = std::min(len, R - (m0 + 1) % R);
    // FP64 running sum: the top segment starts it, the last one (j = 0) writes G
    const double cf = (m0 == 0 ? 1.0 : 2.0) / p->lmax;
    const int in_mode = j == nseg - 1 ? 0 : 1;
    const int out_mode = j == 0 ? 1 : 0;
    char *tb = (char *)(keep ? ck(m0) : seg(0));
    if ((rc = launch_vjp(prec, g, G, G64, bv(m0 + 1), bv(m0 + 1 + len0), 1, tb, tb + len0 * vecp,
                         vecp, len0, len, cf, 2.0 / p->lmax, in_mode, out_mode, s)))
      return rc;
  }
  return OVL_OK;
}

// ||S (S psi_r) - psi_r|| / ||psi_r|| per right-hand side, S the polynomial sign function with
// deflation.  The exact sign function squares to one (Sec. 2), so this measures the
// approximation: two fused evaluations, S^2 psi - psi in place, and FP64 inner products.
int ovl_sign_residual(const ovl_gauge *g, const ovl_poly *p, const ovl_defl *d, const void *in,
                      int nrhs, int spin_dt, double *r_out, void *stream) {
  g_err[0] = 0;
  if (!r_out) return fail(OVL_EINVAL, "r_out is NULL");
  // argument checks of a one-vector call; the outputs are the library's own vectors, so the
  // placeholder output address below only has to be distinct from any device buffer
  static const char kOwnOutput = 0;
  Prec prec;
  int rc = check_spinor_call(g, &kOwnOutput, in, nrhs, spin_dt, prec);
  if (rc) return rc;
  if ((rc = check_poly(p)) || (rc = check_defl(g, d, prec))) return rc;
  const hipStream_t s = as_stream(stream);
  const int V = g->g.V;
  const size_t one = (size_t)12 * V * elem_bytes(spin_dt);
  const size_t vec = one * nrhs;
  const int nblk = project_blocks(V);
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  Scratch sc;
  if ((rc = scratch_alloc(sc, 2 * up(vec) + up(sizeof(double2) * nblk) +
                                  up(sizeof(double2) * 2 * nrhs), s)))
    return rc;
  char *y1 = (char *)sc.p, *y2 = y1 + up(vec);
  double2 *partial = (double2 *)(y2 + up(vec));
  double2 *cdev = (double2 *)((char *)partial + up(sizeof(double2) * nblk));
  if ((rc = run_sign(g, p, const_cast<ovl_defl *>(d), MODE_SIGN, 0.0, 0, y1, in, nrhs, spin_dt,
                     prec, s)))
    return rc;
  if ((rc = run_sign(g, p, const_cast<ovl_defl *>(d), MODE_SIGN, 0.0, 0, y2, y1, nrhs, spin_dt,
                     prec, s)))
    return rc;
  const SolveVecs w{spin_dt == OVL_F64, (int64_t)nrhs * 12 * V, s, partial, nblk, cdev};
  if ((rc = vaxpby(w, y2, 1.0, in, -1.0, y2))) return rc;  // S^2 psi - psi
  for (int r = 0; r < nrhs; ++r) {
    const char *dr = y2 + (size_t)r * one;
    const char *pr = (const char *)in + (size_t)r * one;
    for (int k = 0; k < 2; ++k) {
      const char *v = k == 0 ? dr : pr;
      rc = spin_dt == OVL_F64
               ? project((const double2 *)v, 1, (const double2 *)v, 0, 1, V, partial, nblk,
                         cdev + 2 * r + k, s)
               : project((const float2 *)v, 1, (const float2 *)v, 0, 1, V, partial, nblk,
                         cdev + 2 * r + k, s);
      if (rc) return rc;
    }
  }
  std::vector<double2> h((size_t)2 * nrhs);
  HIP_TRY(hipMemcpyAsync(h.data(), cdev, sizeof(double2) * 2 * nrhs, hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  for (int r = 0; r < nrhs; ++r) {
    const double num = h[2 * r].x, den = h[2 * r + 1].x;
    if (!std::isfinite(num) || !std::isfinite(den))
      return fail(OVL_ENONFINITE, "non-finite norm for right-hand side %d", r);
    r_out[r] = den > 0.0 ? std::sqrt(std::max(num, 0.0) / den) : 0.0;
  }
  return OVL_OK;
}


}  // extern "C"

// ---------------------------------------------------------------------------------------------
// low modes of K (the deflation basis of Sec. 2, eq. 3)
namespace {

using cplx = std::complex<double>;

// Eigen-decomposition of a Hermitian n x n matrix A (row-major): Householder reduction to
// Hermitian tridiagonal form, a diagonal phase similarity that makes the tridiagonal real, the
// implicit QL iteration with Wilkinson-type shifts on the real tridiagonal (accumulating its
// rotations), and back-transformation.  w ascending; the eigenvectors are the columns of Q
// (row-major).  Returns false if the QL iteration does not converge.
bool hermitian_eigh(int n, std::vector<cplx> A, std::vector<double> &w, std::vector<cplx> &Q) {
  auto a = [&](int i, int j) -> cplx & { return A[(size_t)i * n + j]; };
  std::vector<cplx> hv((size_t)n * n, cplx(0.0, 0.0));  // Householder vector of step k in column k
  std::vector<bool> has(n, false);
  for (int k = 0; k + 2 < n; ++k) {
    const int L = n - k - 1;
    double xn2 = 0.0;
    for (int i = 0; i < L; ++i) xn2 += std::norm(a(k + 1 + i, k));
    const double xn = std::sqrt(xn2);
    if (xn == 0.0) continue;
    const cplx x0 = a(k + 1, k);
    const cplx ph = std::abs(x0) > 0.0 ? x0 / std::abs(x0) : cplx(1.0, 0.0);
    const cplx alpha = -ph * xn;  // H x = alpha e_1
    std::vector<cplx> v(L);
    for (int i = 0; i < L; ++i) v[i] = a(k + 1 + i, k);
    v[0] -= alpha;
    double vn2 = 0.0;
    for (int i = 0; i < L; ++i) vn2 += std::norm(v[i]);
    if (vn2 == 0.0) continue;
    const double vn = std::sqrt(vn2);
    for (int i = 0; i < L; ++i) v[i] /= vn;
    // trailing block B <- H B H with H = 1 - 2 v v^+:  p = B v, beta = v^+ p, w = p - beta v,
    // B <- B - 2 v w^+ - 2 w v^+
    std::vector<cplx> pv(L, 0.0);
    for (int i = 0; i < L; ++i) {
      cplx t = 0.0;
      for (int j = 0; j < L; ++j) t += a(k + 1 + i, k + 1 + j) * v[j];
      pv[i] = t;
    }
    cplx beta = 0.0;
    for (int i = 0; i < L; ++i) beta += std::conj(v[i]) * pv[i];
    for (int i = 0; i < L; ++i) pv[i] -= beta.real() * v[i];
    for (int i = 0; i < L; ++i)
      for (int j = 0; j < L; ++j)
        a(k + 1 + i, k + 1 + j) -= 2.0 * (v[i] * std::conj(pv[j]) + pv[i] * std::conj(v[j]));
    a(k + 1, k) = alpha;
    a(k, k + 1) = std::conj(alpha);
    for (int i = 1; i < L; ++i) a(k + 1 + i, k) = a(k, k + 1 + i) = 0.0;
    for (int i = 0; i < L; ++i) hv[(size_t)(k + 1 + i) * n + k] = v[i];
    has[k] = true;
  }
  // phases that make the sub-diagonal real and non-negative: T' = D^+ T D
  std::vector<cplx> phi(n, cplx(1.0, 0.0));
  std::vector<double> d(n), e(n, 0.0);
  for (int k = 0; k < n; ++k) d[k] = a(k, k).real();
  for (int k = 0; k + 1 < n; ++k) {
    const cplx t = a(k + 1, k);
    const double m = std::abs(t);
    phi[k + 1] = m > 0.0 ? phi[k] * (t / m) : phi[k];
    e[k] = m;
  }
  // implicit QL on (d, e), rotations accumulated into Z (real, row-major)
  std::vector<double> Z((size_t)n * n, 0.0);
  for (int i = 0; i < n; ++i) Z[(size_t)i * n + i] = 1.0;
  const double eps = std::numeric_limits<double>::epsilon();
  for (int l = 0; l < n; ++l) {
    int iter = 0, m;
    do {
      for (m = l; m < n - 1; ++m) {
        const double dd = std::fabs(d[m]) + std::fabs(d[m + 1]);
        if (std::fabs(e[m]) <= eps * dd) break;
      }
      if (m != l) {
        if (iter++ == 100) return false;
        double g = (d[l + 1] - d[l]) / (2.0 * e[l]);
        double r = std::hypot(g, 1.0);
        g = d[m] - d[l] + e[l] / (g + std::copysign(r, g));
        double s2 = 1.0, c = 1.0, p = 0.0;
        int i;
        for (i = m - 1; i >= l; --i) {
          double f = s2 * e[i];
          const double b = c * e[i];
          e[i + 1] = (r = std::hypot(f, g));
          if (r == 0.0) {
            d[i + 1] -= p;
            e[m] = 0.0;
            break;
          }
          s2 = f / r;
          c = g / r;
          g = d[i + 1] - p;
          r = (d[i] - g) * s2 + 2.0 * c * b;
          d[i + 1] = g + (p = s2 * r);
          g = c * r - b;
          for (int k = 0; k < n; ++k) {
            f = Z[(size_t)k * n + i + 1];
            Z[(size_t)k * n + i + 1] = s2 * Z[(size_t)k * n + i] + c * f;
            Z[(size_t)k * n + i] = c * Z[(size_t)k * n + i] - s2 * f;
          }
        }
        if (r == 0.0 && i >= l) continue;
        d[l] -= p;
        e[l] = g;
        e[m] = 0.0;
      }
    } while (m != l);
  }
  // Q = H_0 H_1 ... (D Z), columns ordered by eigenvalue
  std::vector<int> order(n);
  for (int i = 0; i < n; ++i) order[i] = i;
  std::sort(order.begin(), order.end(), [&](int x, int y) { return d[x] < d[y]; });
  Q.assign((size_t)n * n, cplx(0.0, 0.0));
  w.resize(n);
  for (int jn = 0; jn < n; ++jn) {
    w[jn] = d[order[jn]];
    for (int i = 0; i < n; ++i) Q[(size_t)i * n + jn] = phi[i] * Z[(size_t)i * n + order[jn]];
  }
  for (int k = n - 3; k >= 0; --k) {
    if (!has[k]) continue;
    for (int j = 0; j < n; ++j) {  // column j <- (1 - 2 v v^+) column j on rows k+1 ..
      cplx t = 0.0;
      for (int i = k + 1; i < n; ++i) t += std::conj(hv[(size_t)i * n + k]) * Q[(size_t)i * n + j];
      for (int i = k + 1; i < n; ++i) Q[(size_t)i * n + j] -= 2.0 * hv[(size_t)i * n + k] * t;
    }
  }
  return true;
}

// device block algebra of the eigen-solve
struct BlockOps {
  hipStream_t s;
  int64_t n;           // complex elements per vector (12 V)
  double2 *partial;    // Gram slices
  size_t partial_cap;  // elements
  double2 *gdev;       // Gram result / rotation matrix (m x m)
  double *rpart;       // residual partials [m][kResBlocks]
};
constexpr int kResBlocks = 512;

// H[i][j] = <A_i, B_j> on the host (synchronises the stream)
int block_gram(BlockOps &o, const double2 *A, int ma, const double2 *B, int mb,
               std::vector<cplx> &H) {
  const int gx = (ma + kGramT - 1) / kGramT, gy = (mb + kGramT - 1) / kGramT;
  const int64_t tiles = (int64_t)gx * gy;
  int nslice = (int)std::max<int64_t>(1, std::min<int64_t>(512, 4096 / tiles));
  nslice = (int)std::min<int64_t>(nslice, (o.partial_cap / (tiles * kGramT * kGramT)));
  nslice = std::max(nslice, 1);
  int64_t slice = (o.n + nslice - 1) / nslice;
  slice = (slice + kGramKC - 1) / kGramKC * kGramKC;
  nslice = (int)((o.n + slice - 1) / slice);
  gram_partial_kernel<<<dim3(gx, gy, nslice), 256, 0, o.s>>>(A, ma, B, mb, o.n, slice, o.partial);
  HIP_TRY(hipGetLastError());
  gram_reduce_kernel<<<(ma * mb + 255) / 256, 256, 0, o.s>>>(o.partial, ma, mb, nslice, o.gdev);
  HIP_TRY(hipGetLastError());
  std::vector<double2> h((size_t)ma * mb);
  HIP_TRY(hipMemcpyAsync(h.data(), o.gdev, sizeof(double2) * h.size(), hipMemcpyDeviceToHost, o.s));
  HIP_TRY(hipStreamSynchronize(o.s));
  H.assign((size_t)ma * mb, cplx(0.0, 0.0));
  for (int j = 0; j < mb; ++j)
    for (int i = 0; i < ma; ++i) H[(size_t)i * mb + j] = cplx(h[(size_t)j * ma + i].x, h[(size_t)j * ma + i].y);
  return OVL_OK;
}

// Out_j = sum_i C[i][j] V_i (C host, mi x mo row-major)
int block_rotate(BlockOps &o, const double2 *V, int mi, const std::vector<cplx> &C, int mo,
                 double2 *Out) {
  std::vector<double2> h((size_t)mi * mo);
  for (size_t k = 0; k < h.size(); ++k) h[k] = make_double2(C[k].real(), C[k].imag());
  HIP_TRY(hipMemcpyAsync(o.gdev, h.data(), sizeof(double2) * h.size(), hipMemcpyHostToDevice, o.s));
  rotate_kernel<<<dim3((unsigned)((o.n + 255) / 256), (mo + kRotJ - 1) / kRotJ), 256, 0, o.s>>>(
      V, mi, o.n, o.gdev, mo, Out);
  HIP_TRY(hipGetLastError());
  // the staging of C must not be rewritten before the rotation has read it
  HIP_TRY(hipStreamSynchronize(o.s));
  return OVL_OK;
}

// r[j] = ||W_j - lam_j V_j|| (lam empty: ||W_j||) for j < m (synchronises the stream)
int block_resid(BlockOps &o, const double2 *W, const double2 *V, const std::vector<double> &lam,
                int m, std::vector<double> &r) {
  double *lam_dev = nullptr;
  if (!lam.empty()) {
    HIP_TRY(hipMemcpyAsync(o.gdev, lam.data(), sizeof(double) * m, hipMemcpyHostToDevice, o.s));
    lam_dev = (double *)o.gdev;
  }
  const int nb = (int)std::min<int64_t>(kResBlocks, (o.n + 255) / 256);
  resid_partial_kernel<<<dim3(nb, m), 256, 0, o.s>>>(W, V, lam_dev, o.n, o.rpart);
  HIP_TRY(hipGetLastError());
  std::vector<double> h((size_t)m * nb);
  HIP_TRY(hipMemcpyAsync(h.data(), o.rpart, sizeof(double) * h.size(), hipMemcpyDeviceToHost, o.s));
  HIP_TRY(hipStreamSynchronize(o.s));
  r.assign(m, 0.0);
  for (int j = 0; j < m; ++j) {
    double t = 0.0;
    for (int b = 0; b < nb; ++b) t += h[(size_t)j * nb + b];
    r[j] = std::sqrt(t);
  }
  return OVL_OK;
}

// out = c K in + a src + b w for a block of nrhs vectors (FP64), one fused launch
int block_k(const ovl_gauge *g, double2 *out, const double2 *in, double c, const double2 *src,
            double a, const double2 *w, double b, int nrhs, double m_W, hipStream_t s) {
  StepArgs<false> p = single_args(g, nrhs);
  p.item.psi = src;
  p.item.buf[0] = const_cast<double2 *>(in);
  p.item.buf[1] = const_cast<double2 *>(w);
  p.item.buf[2] = out;
  p.v_role = ROLE_B0;
  p.w_role = w ? ROLE_B1 : ROLE_NONE;
  p.out_role = ROLE_B2;
  p.y_g5 = 1;
  p.kd = c * (4.0 - m_W);
  p.kh = -0.5 * c;
  p.a = src ? a : 0.0;
  p.t = w ? b : 0.0;
  return dispatch_single(P_F64, p, s);
}

}  // namespace

extern "C" {

// Chebyshev-filtered subspace iteration on K for the n_ev eigenpairs of smallest |lambda|: the
// filter T_degree((2 K^2 - (cut^2 + lmax^2)) / (lmax^2 - cut^2)) grows fastest towards K = 0 and
// is bounded by 1 on cut <= |lambda| <= lmax; each iteration orthonormalises the block (scaled
// SVQB from its Gram matrix), applies Rayleigh-Ritz with K itself (so +lambda and -lambda
// separate), orders the Ritz pairs by ||K v||, checks the residuals and filters the block.
int ovl_low_modes(const ovl_gauge *g, int n_ev, int block, double lmax, double cut, int degree,
                  int max_iter, double tol, uint64_t seed, double m_W, void *phi_out,
                  double *lambda_out, double *resid_out, double *eps_next_out, int *iters_out,
                  void *stream) {
  g_err[0] = 0;
  if (!g || !phi_out || !lambda_out || !resid_out) return fail(OVL_EINVAL, "NULL argument");
  if (g->store_dt != OVL_F64) return fail(OVL_EDTYPE, "the eigen-solve needs FP64 link storage");
  const int m = block;
  if (n_ev < 1 || m <= n_ev || m > 256 || (int64_t)m > (int64_t)12 * g->g.V)
    return fail(OVL_EINVAL, "need 1 <= n_ev < block <= min(256, 12 V) (n_ev %d, block %d)", n_ev, m);
  if (!std::isfinite(lmax) || !std::isfinite(cut) || !std::isfinite(m_W) || !std::isfinite(tol))
    return fail(OVL_ENONFINITE, "non-finite parameter");
  if (!(cut > 0.0) || !(lmax > cut) || degree < 1 || degree > 10000 || max_iter < 1 || !(tol > 0.0))
    return fail(OVL_EINVAL, "need 0 < cut < lmax, degree in [1, 10000], max_iter >= 1, tol > 0");
  if (!fits_u32(12ull * g->g.V, OVL_F64)) return fail(OVL_EDIMS, "lattice too large");
  hipStream_t s = as_stream(stream);
  const int64_t n = (int64_t)12 * g->g.V;
  const size_t vb = (size_t)m * n * sizeof(double2);
  const size_t vbp = (vb + 255) / 256 * 256;
  const int64_t tiles = (int64_t)((m + kGramT - 1) / kGramT) * ((m + kGramT - 1) / kGramT);
  const size_t part_elems = (size_t)tiles * kGramT * kGramT * 512;
  Scratch sc;
  int rc = scratch_alloc(sc, 5 * vbp + part_elems * sizeof(double2) +
                                 (size_t)m * m * sizeof(double2) + (size_t)m * kResBlocks * 8 + 1024, s);
  if (rc) return rc;
  char *base = (char *)sc.p;
  double2 *buf[5];
  for (int k = 0; k < 5; ++k) buf[k] = (double2 *)(base + k * vbp);
  BlockOps o{s, n, (double2 *)(base + 5 * vbp), part_elems, nullptr, nullptr};
  o.gdev = (double2 *)((char *)o.partial + part_elems * sizeof(double2));
  o.rpart = (double *)((char *)o.gdev + (size_t)m * m * sizeof(double2));
  double2 *V = buf[0], *W = buf[1], *T0 = buf[2], *T1 = buf[3], *T2 = buf[4];
  uint64_t draws = 0;  // fresh draws of the seeded generator
  auto fill = [&](double2 *dst, int64_t count) -> int {
    gaussian_block_kernel<<<(unsigned)((count + 255) / 256), 256, 0, s>>>(dst, count, seed + draws++);
    HIP_TRY(hipGetLastError());
    return OVL_OK;
  };
  if ((rc = fill(V, (int64_t)m * n))) return rc;
  // The filter is K on a block of m right-hand sides, a problem of its own for the launch
  // configuration (on 16^3 x 32 with 128 vectors the tuned form runs 1.2x faster than the default
  // rule): without a configuration for it, measure the candidates once (as ovl_autotune does,
  // on the block itself and W as output).
  {
    StepItem probe;
    fill_item(probe, g, m);
    const TuneKey key = tune_key((int)P_F64, &probe, 1);
    bool known;
    {
      std::lock_guard<std::mutex> lk(g_tune_mu);
      known = g_tuned.count(key) > 0;
    }
    if (!known) {
      const ovl_batch_item it{g, V, W, m};
      if ((rc = ovl_autotune(&it, 1, nullptr, OVL_F64, nullptr, nullptr, stream))) return rc;
    }
  }
  std::vector<double> lam, res;
  const double bq = lmax * lmax, aq = cut * cut;
  const double c1 = 2.0 / (bq - aq), c0 = -(aq + bq) / (bq - aq);
  int it = 0;
  for (;; ++it) {
    // orthonormalise: G = V^+ V, D = diag(G)^-1/2, D G D = Q diag(l) Q^+, V <- (D Q l^-1/2)^T V;
    // directions with l below 1e-12 l_max are dropped and refilled from the generator
    for (int pass = 0, good = 0; good < 2; ++pass) {
      if (pass > 8) return fail(OVL_EDIVERGED, "block orthonormalisation failed");
      std::vector<cplx> G, Q;
      std::vector<double> l;
      if ((rc = block_gram(o, V, m, V, m, G))) return rc;
      std::vector<double> d(m);
      for (int i = 0; i < m; ++i) {
        const double gi = G[(size_t)i * m + i].real();
        if (!std::isfinite(gi)) return fail(OVL_ENONFINITE, "non-finite block vector");
        d[i] = gi > 0.0 ? 1.0 / std::sqrt(gi) : 0.0;
      }
      for (int i = 0; i < m; ++i)
        for (int j = 0; j < m; ++j) G[(size_t)i * m + j] *= d[i] * d[j];
      if (!hermitian_eigh(m, G, l, Q)) return fail(OVL_EDIVERGED, "Gram eigen-decomposition failed");
      int weak = 0;
      while (weak < m && !(l[weak] > 1e-12 * l[m - 1])) ++weak;
      const int keep = m - weak;
      std::vector<cplx> C((size_t)m * keep);
      for (int i = 0; i < m; ++i)
        for (int k = 0; k < keep; ++k)
          C[(size_t)i * keep + k] = d[i] * Q[(size_t)i * m + weak + k] / std::sqrt(l[weak + k]);
      if ((rc = block_rotate(o, V, m, C, keep, T0))) return rc;
      std::swap(V, T0);
      if (weak) {
        if ((rc = fill(V + (int64_t)keep * n, (int64_t)weak * n))) return rc;
        good = 0;
      } else {
        ++good;
      }
    }
    // Rayleigh-Ritz with K: H = V^+ K V, ordered by ||K v|| (directions that have not converged
    // mix +lambda and -lambda and have Rayleigh quotients near zero)
    if ((rc = block_k(g, W, V, 1.0, nullptr, 0.0, nullptr, 0.0, m, m_W, s))) return rc;
    std::vector<cplx> H, M, Y;
    if ((rc = block_gram(o, V, m, W, m, H))) return rc;
    if ((rc = block_gram(o, W, m, W, m, M))) return rc;
    for (int i = 0; i < m; ++i)
      for (int j = i; j < m; ++j) {
        const cplx h = 0.5 * (H[(size_t)i * m + j] + std::conj(H[(size_t)j * m + i]));
        H[(size_t)i * m + j] = h;
        H[(size_t)j * m + i] = std::conj(h);
      }
    std::vector<double> w;
    if (!hermitian_eigh(m, H, w, Y)) return fail(OVL_EDIVERGED, "Ritz eigen-decomposition failed");
    std::vector<double> kn(m, 0.0);
    for (int k = 0; k < m; ++k) {
      cplx t = 0.0;
      for (int i = 0; i < m; ++i) {
        cplx row = 0.0;
        for (int j = 0; j < m; ++j) row += M[(size_t)i * m + j] * Y[(size_t)j * m + k];
        t += std::conj(Y[(size_t)i * m + k]) * row;
      }
      kn[k] = t.real();
    }
    std::vector<int> order(m);
    for (int k = 0; k < m; ++k) order[k] = k;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return kn[a] < kn[b]; });
    std::vector<cplx> C((size_t)m * m);
    lam.assign(m, 0.0);
    for (int k = 0; k < m; ++k) {
      lam[k] = w[order[k]];
      for (int i = 0; i < m; ++i) C[(size_t)i * m + k] = Y[(size_t)i * m + order[k]];
    }
    if ((rc = block_rotate(o, V, m, C, m, T0))) return rc;
    std::swap(V, T0);
    if ((rc = block_rotate(o, W, m, C, m, T0))) return rc;
    std::swap(W, T0);
    if ((rc = block_resid(o, W, V, lam, m, res))) return rc;
    double worst = 0.0;
    for (int k = 0; k < n_ev; ++k) worst = std::max(worst, res[k]);
    if (worst < tol || it + 1 >= max_iter) break;
    // filter: t_0 = V, t_1 = Z V, t_{j+1} = 2 Z t_j - t_{j-1}, Z x = c1 K (K x) + c0 x
    if ((rc = block_k(g, T0, V, 1.0, nullptr, 0.0, nullptr, 0.0, m, m_W, s))) return rc;
    if ((rc = block_k(g, T1, T0, c1, V, c0, nullptr, 0.0, m, m_W, s))) return rc;
    double2 *tp = V, *tc = T1;
    double2 *spare = T2;
    for (int j = 2; j <= degree; ++j) {
      if ((rc = block_k(g, T0, tc, 1.0, nullptr, 0.0, nullptr, 0.0, m, m_W, s))) return rc;
      // t_{j} = 2 c1 K y + 2 c0 t_{j-1} - t_{j-2}, written over t_{j-2}
      if ((rc = block_k(g, tp, T0, 2.0 * c1, tc, 2.0 * c0, tp, -1.0, m, m_W, s))) return rc;
      std::swap(tp, tc);
    }
    // the filtered block becomes V; the other two buffers are work space again
    V = tc;
    T1 = tp;
    T2 = spare;
  }
  HIP_TRY(hipMemcpyAsync(phi_out, V, sizeof(double2) * (size_t)n_ev * n, hipMemcpyDeviceToDevice, s));
  HIP_TRY(hipStreamSynchronize(s));
  double worst = 0.0;
  for (int k = 0; k < n_ev; ++k) {
    lambda_out[k] = lam[k];
    resid_out[k] = res[k];
    worst = std::max(worst, res[k]);
  }
  if (eps_next_out) *eps_next_out = std::fabs(lam[n_ev]) / lmax;
  if (iters_out) *iters_out = it + 1;
  if (!(worst < tol))
    return fail(OVL_EDIVERGED, "residual %.3e above %.3e after %d iterations", worst, tol, it + 1);
  return OVL_OK;
}

// Hermitian eigen-decomposition of the eigen-solve, on host memory (no device involved)
int ovl_hermitian_eigh(int n, const double *a, double *w, double *q) {
  g_err[0] = 0;
  if (!a || !w || !q) return fail(OVL_EINVAL, "NULL argument");
  if (n < 1 || n > 4096) return fail(OVL_EINVAL, "n = %d out of range [1, 4096]", n);
  std::vector<cplx> A((size_t)n * n), Q;
  for (size_t k = 0; k < A.size(); ++k) A[k] = cplx(a[2 * k], a[2 * k + 1]);
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j)
      if (std::abs(A[(size_t)i * n + j] - std::conj(A[(size_t)j * n + i])) >
          1e-12 * (1.0 + std::abs(A[(size_t)i * n + j])))
        return fail(OVL_EINVAL, "matrix is not Hermitian at (%d, %d)", i, j);
  std::vector<double> wv;
  if (!hermitian_eigh(n, A, wv, Q)) return fail(OVL_EDIVERGED, "QL iteration did not converge");
  for (int i = 0; i < n; ++i) w[i] = wv[i];
  for (size_t k = 0; k < Q.size(); ++k) {
    q[2 * k] = Q[k].real();
    q[2 * k + 1] = Q[k].imag();
  }
  return OVL_OK;
}

// Times one plain Clenshaw step of the problem set (stencil input `in`, own-site reads of `in`
// as source and recurrence vector, output `out`: the memory streams of an odd-k step) in every
// candidate configuration and keeps the fastest for this problem set.
int ovl_autotune(const ovl_batch_item *items, int n_items, const ovl_poly *p, int spin_dt,
                 const char *cache_path, double *best_us, void *stream) {
  g_err[0] = 0;
  SignJob jobs[kMaxBatch];
  Prec prec;
  int rc = check_batch(items, n_items, spin_dt, jobs, prec);
  if (rc) return rc;
  hipStream_t s = as_stream(stream);
  const bool table = n_items > 1;
  const double lmax = p ? p->lmax : 6.5, m_W = p ? p->m_W : 1.5;
  StepItem its[kMaxBatch];
  int maxr = 1;
  int64_t work = 0;
  for (int i = 0; i < n_items; ++i) {
    fill_item(its[i], items[i].g, items[i].nrhs);
    its[i].psi = items[i].in;
    its[i].buf[0] = items[i].out;
    its[i].buf[1] = const_cast<void *>(items[i].in);
    maxr = std::max(maxr, items[i].nrhs);
    work += (int64_t)items[i].g->g.V * items[i].nrhs;
  }
  Scratch sc;
  if (table && (rc = scratch_alloc(sc, sizeof(StepItem) * n_items, s))) return rc;
  StepArgs<false> a1;
  StepArgs<true> at;
  clear_args(a1);
  clear_args(at);
  for (StepArgs<false> *q : {&a1}) {
    q->v_role = ROLE_PSI;
    q->w_role = ROLE_B1;
    q->out_role = ROLE_B0;
    q->y_g5 = 1;
    q->kd = 2.0 * (4.0 - m_W) / lmax;
    q->kh = -1.0 / lmax;
    q->a = 0.5;
    q->t = -1.0;
  }
  at.v_role = a1.v_role;
  at.w_role = a1.w_role;
  at.out_role = a1.out_role;
  at.y_g5 = 1;
  at.kd = a1.kd;
  at.kh = a1.kh;
  at.a = a1.a;
  at.t = a1.t;
  at.n_items = n_items;
  StepItem *table_dev = (StepItem *)sc.p;
  at.table = table_dev;
  at.r12 = 1;
  for (int i = 0; i < n_items; ++i) at.r12 = at.r12 && its[i].r12;
  const int sb = site_bytes_of(prec);
  const bool pairs = pairs_ok(prec, its, n_items);
  std::vector<LaunchCfg> cands;
  for (int spb : {128, 64, 16, 8})
    for (int tiles : {1, 0})
      for (int remap : {1, 0})
        for (int rb : {1, 2, 4}) {
          const LaunchCfg c{spb, tiles, remap, rb};
          if (spb == 128 && !pairs) continue;
          if (!rb_ok(c) || (rb > 1 && rb > maxr)) continue;
          if (tiles) {
            bool any = false;
            for (int i = 0; i < n_items; ++i) {
              int ty, tz;
              step_tile(its[i].g, spb, sb, ty, tz);
              any = any || ty > 0;
            }
            if (!any) continue;
          }
          cands.push_back(c);
        }
  if (march_ok(its, n_items)) cands.push_back(LaunchCfg{64, kMarch, 1, 1});
  if (!table)
    for (int spb : {64, 128, 192, 256})
      if (slab_ok(its[0].g, spb, prec))
        for (int remap : {1, 0}) cands.push_back(LaunchCfg{spb, 2, remap, 1});
  auto launch = [&](const LaunchCfg &cfg) -> int {
    if (!table) {
      a1.item = its[0];
      return dispatch_cfg(prec, a1, cfg, s);
    }
    return dispatch_step(prec, at, cfg, s);
  };
  hipEvent_t e0, e1;
  HIP_TRY(hipEventCreate(&e0));
  HIP_TRY(hipEventCreate(&e1));
  LaunchCfg best{0, 0, 0, 1};
  float best_ms = 1e30f;
  std::vector<float> times(cands.size(), 1e30f);
  for (size_t ci = 0; ci < cands.size(); ++ci) {
    const LaunchCfg &cfg = cands[ci];
    if (table) {
      plan_launch(at, its, n_items, cfg, prec);
      for (int i = 0; i < n_items && rc == OVL_OK; ++i) {
        write_item_kernel<<<1, 64, 0, s>>>(its[i], table_dev + i);
        if (hipGetLastError() != hipSuccess) rc = fail(OVL_EHIP, "item table write");
      }
    }
    for (int w = 0; w < 2 && rc == OVL_OK; ++w) rc = launch(cfg);
    if (rc == OVL_OK && hipEventRecord(e0, s) != hipSuccess) rc = fail(OVL_EHIP, "event record");
    for (int w = 0; w < 10 && rc == OVL_OK; ++w) rc = launch(cfg);
    if (rc == OVL_OK && hipEventRecord(e1, s) != hipSuccess) rc = fail(OVL_EHIP, "event record");
    float ms = 0.f;
    if (rc == OVL_OK && (hipEventSynchronize(e1) != hipSuccess ||
                         hipEventElapsedTime(&ms, e0, e1) != hipSuccess))
      rc = fail(OVL_EHIP, "event timing");
    if (rc) break;
    times[ci] = ms;
    if (ms < best_ms) {
      best_ms = ms;
      best = cfg;
    }
  }
  // Within 3% (run-to-run noise) the XCD-contiguous remap of the same form wins: it moves fewer
  // bytes across the XCDs' L2 caches (measured on the headline batch: 1.52x against 1.93x the
  // algorithmic bytes) at the same speed, and the choice stays stable from run to run.
  if (rc == OVL_OK && best.remap == 0)
    for (size_t ci = 0; ci < cands.size(); ++ci) {
      const LaunchCfg &c = cands[ci];
      if (c.remap == 1 && c.spb == best.spb && c.tiles == best.tiles && c.rb == best.rb &&
          times[ci] <= 1.03f * best_ms) {
        best = c;
        best_ms = times[ci];
      }
    }
  // Within 2% the t-streaming tile order of the same form wins over memory order: it re-reads
  // fewer t neighbours from HBM at the same speed (the headline batch: 1.22x against 1.41x the
  // algorithmic bytes, 196.6 against 197.1 us per step, counters on one machine).
  if (rc == OVL_OK && best.tiles == 0)
    for (size_t ci = 0; ci < cands.size(); ++ci) {
      const LaunchCfg &c = cands[ci];
      if (c.tiles == 1 && c.spb == best.spb && c.remap == best.remap && c.rb == best.rb &&
          times[ci] <= 1.02f * best_ms) {
        best = c;
        best_ms = times[ci];
      }
    }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc == OVL_OK && hipStreamSynchronize(s) != hipSuccess) rc = fail(OVL_EHIP, "synchronise");
  if (rc) return rc;
  const TuneKey key = tune_key((int)prec, its, n_items);
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tuned[key] = best;
  }
  (void)work;
  const double us = 1e3 * best_ms / 10.0;
  if (best_us) *best_us = us;
  if (cache_path) {
    FILE *f = std::fopen(cache_path, "a");
    if (!f) return fail(OVL_EINVAL, "cannot open tuning cache %s", cache_path);
    std::fprintf(f, "B %d %d %d", (int)prec, key.r12, n_items);
    for (const auto &it : key.items)
      std::fprintf(f, " %d %d %d %d %d", it[0], it[1], it[2], it[3], it[4]);
    std::fprintf(f, " %d %d %d %d %.3f\n", best.spb, best.tiles, best.remap, best.rb, us);
    std::fclose(f);
  }
  return OVL_OK;
}

int ovl_autotune_load(const char *cache_path) {
  g_err[0] = 0;
  if (!cache_path) return fail(OVL_EINVAL, "NULL path");
  return load_tune_cache(cache_path);
}

int ovl_launch_config(const ovl_gauge *g, int nrhs, int spin_dt, int cfg_out[3]) {
  if (!g || !cfg_out) return fail(OVL_EINVAL, "NULL argument");
  const Prec prec = precision(spin_dt, g->store_dt);
  if (prec == P_BAD) return fail(OVL_EDTYPE, "spinor dtype %d with link storage %d", spin_dt, g->store_dt);
  // vectors are taken as 16-byte aligned (torch allocations are)
  const int64_t work = (int64_t)g->g.V * nrhs;
  const bool pairs = prec != P_F64 && g->g.L[0] % 2 == 0;
  StepItem it;
  fill_item(it, g, nrhs);
  const LaunchCfg c = fit_slab(fit_cfg(lookup_cfg((int)prec, &it, 1, work, 3), pairs), it, prec, work, pairs);
  cfg_out[0] = c.spb;
  cfg_out[1] = c.tiles;
  cfg_out[2] = c.remap;
  return OVL_OK;
}

int ovl_batch_launch_config(const ovl_batch_item *items, int n_items, int spin_dt,
                            int cfg_out[4]) {
  g_err[0] = 0;
  if (!cfg_out) return fail(OVL_EINVAL, "NULL argument");
  SignJob jobs[kMaxBatch];
  Prec prec;
  int rc = check_batch(items, n_items, spin_dt, jobs, prec);
  if (rc) return rc;
  const LaunchCfg c = n_items > 1 ? sign_cfg<true>(jobs, n_items, prec)
                                  : sign_cfg<false>(jobs, n_items, prec);
  cfg_out[0] = c.spb;
  cfg_out[1] = c.tiles;
  cfg_out[2] = c.remap;
  cfg_out[3] = c.rb;
  return OVL_OK;
}

int ovl_status_flags(const ovl_gauge *g, uint32_t *flags, int clear) {
  if (!g || !flags) return fail(OVL_EINVAL, "NULL argument");
  HIP_TRY(hipDeviceSynchronize());
  HIP_TRY(hipMemcpy(flags, g->flags, sizeof(uint32_t), hipMemcpyDeviceToHost));
  if (clear) HIP_TRY(hipMemset(g->flags, 0, sizeof(uint32_t)));
  return OVL_OK;
}

int ovl_memory_release(void) {
  g_err[0] = 0;
  HIP_TRY(hipDeviceSynchronize());
  block_cache().release();
  return OVL_OK;
}

int ovl_graph_enable(int on) {
  g_graphs.store(on ? 1 : 0);
  return OVL_OK;
}

int ovl_timing_enable(int on) {
  g_timing.store(on ? 1 : 0);
  return OVL_OK;
}

int ovl_timing_read(int kind, double *total_ms, int64_t *launches) {
  if (!total_ms || !launches) return fail(OVL_EINVAL, "NULL argument");
  if (kind < 0 || kind >= TK_COUNT) return fail(OVL_EINVAL, "timing kind %d", kind);
  std::lock_guard<std::mutex> lk(g_timing_mu);
  double tot = 0.0;
  int64_t n = 0;
  std::vector<TimedRun> keep;
  for (auto &run : g_timing_events) {
    if (run.kind != kind) {
      keep.push_back(run);
      continue;
    }
    HIP_TRY(hipEventSynchronize(run.e1));
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, run.e0, run.e1));
    tot += ms;
    n += run.n;
    g_event_pool.push_back(run.e0);
    g_event_pool.push_back(run.e1);
  }
  *launches = n;
  *total_ms = tot;
  g_timing_events.swap(keep);
  return OVL_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------------------------
// Stout smearing of the links (Sec. 2: 3 steps of over-improved stout smearing, rho = 0.1,
// eps = -0.25) and its chain rule for the HMC force (Sec. 1).  FP64 links and derivatives in the
// caller layout; the staple weights are rho (5 - 2 eps)/3 (plaquettes) and -rho (1 - eps)/12
// (rectangles).
namespace {

bool spans_overlap(const void *a, const void *b, size_t n) {
  const char *x = (const char *)a, *y = (const char *)b;
  return x < y + n && y < x + n;
}

int check_stout(const int32_t dims[4], double rho, double eps, int steps, Geom &geo) {
  int rc = check_dims(dims, geo);
  if (rc) return rc;
  // the path kernels address a link field through 32-bit buffer offsets
  if (!fits_u32(36ull * geo.V, OVL_F64))
    return fail(OVL_EDIMS, "a link field of %d sites spans 4 GiB or more", geo.V);
  if (!std::isfinite(rho) || !std::isfinite(eps)) return fail(OVL_ENONFINITE, "non-finite rho or eps");
  if (steps < 0 || steps > 64) return fail(OVL_EINVAL, "steps = %d out of range [0, 64]", steps);
  return OVL_OK;
}

// t-streaming tile of the path kernels: the smallest whose slice is whole 256-site workgroups (none:
// memory order)
StoutOrder stout_order(const Geom &g) {
  StoutOrder best{0, 0};
  for (int ty = 2; ty <= 8; ty *= 2)
    for (int tz = 2; tz <= 8; tz *= 2) {
      if (g.L[1] % ty || g.L[2] % tz || (int64_t)g.L[0] * ty * tz % 256) continue;
      if (!best.ty || ty * tz < best.ty * best.tz) best = StoutOrder{ty, tz};
    }
  return best;
}
int stout_staples(const double2 *U, double2 *C, double wp, double wr, const Geom &geo, hipStream_t s) {
  stout_staple_kernel<<<4u * (unsigned)((geo.V + 255) / 256), 256, 0, s>>>(U, C, wp, wr, geo,
                                                                           stout_order(geo));
  HIP_TRY(hipGetLastError());
  return OVL_OK;
}

void stout_weights(double rho, double eps, double &wp, double &wr) {
  wp = rho * (5.0 - 2.0 * eps) / 3.0;
  wr = -rho * (1.0 - eps) / 12.0;
}

}  // namespace

extern "C" {

int ovl_stout_smear(const int32_t dims[4], void *U_out, const void *U_in, double rho, double eps,
                    int steps, void *stream) {
  g_err[0] = 0;
  if (!U_out || !U_in) return fail(OVL_EINVAL, "NULL argument");
  Geom geo;
  int rc = check_stout(dims, rho, eps, steps, geo);
  if (rc) return rc;
  const size_t bytes = (size_t)36 * geo.V * sizeof(double2);
  if (spans_overlap(U_out, U_in, bytes)) return fail(OVL_EALIAS, "U_out overlaps U_in");
  hipStream_t s = as_stream(stream);
  if (steps == 0) {
    HIP_TRY(hipMemcpyAsync(U_out, U_in, bytes, hipMemcpyDeviceToDevice, s));
    return OVL_OK;
  }
  double wp, wr;
  stout_weights(rho, eps, wp, wr);
  // levels ping-pong through two work fields, the last step writes U_out; a step's staple sums form in
  // its output
  Scratch sc;
  const size_t fb = (bytes + 255) / 256 * 256;
  if (steps > 1 && (rc = scratch_alloc(sc, 2 * fb, s))) return rc;
  const dim3 grid((unsigned)((geo.V + 255) / 256), 4);
  const double2 *cur = (const double2 *)U_in;
  for (int k = 0; k < steps; ++k) {
    double2 *dst = k == steps - 1 ? (double2 *)U_out : (double2 *)((char *)sc.p + (k % 2) * fb);
    if ((rc = stout_staples(cur, dst, wp, wr, geo, s))) return rc;
    stout_exp_kernel<<<grid, 256, 0, s>>>(cur, dst, dst, geo.V);
    HIP_TRY(hipGetLastError());
    cur = dst;
  }
  return OVL_OK;
}

int ovl_stout_backward(const int32_t dims[4], void *G_thin, const void *G_smeared,
                       const void *U_thin, double rho, double eps, int steps, void *stream) {
  g_err[0] = 0;
  if (!G_thin || !G_smeared || !U_thin) return fail(OVL_EINVAL, "NULL argument");
  Geom geo;
  int rc = check_stout(dims, rho, eps, steps, geo);
  if (rc) return rc;
  const size_t bytes = (size_t)36 * geo.V * sizeof(double2);
  if (spans_overlap(G_thin, G_smeared, bytes) || spans_overlap(G_thin, U_thin, bytes) ||
      spans_overlap(G_smeared, U_thin, bytes))
    return fail(OVL_EALIAS, "G_thin, G_smeared and U_thin must not overlap");
  hipStream_t s = as_stream(stream);
  if (steps == 0) {
    HIP_TRY(hipMemcpyAsync(G_thin, G_smeared, bytes, hipMemcpyDeviceToDevice, s));
    return OVL_OK;
  }
  double wp, wr;
  stout_weights(rho, eps, wp, wr);
  // work fields: levels 1 .. steps-1 of the forward smearing and the staple sums of every level (both
  // from the regenerating forward pass), Gamma, the direct part and two derivative fields between the
  // steps; the last level's staple sums form in the field that later takes the first derivative
  const size_t fb = (bytes + 255) / 256 * 256;
  const int nlev = steps - 1;
  const int nder = steps >= 3 ? 2 : 1;
  Scratch sc;
  if ((rc = scratch_alloc(sc, (size_t)(2 * nlev + 2 + nder) * fb, s))) return rc;
  char *base = (char *)sc.p;
  auto field = [&](int i) { return (double2 *)(base + (size_t)i * fb); };
  double2 *gam = field(2 * nlev), *dir = field(2 * nlev + 1);
  const dim3 grid((unsigned)((geo.V + 255) / 256), 4);
  const StoutOrder order = stout_order(geo);
  auto der = [&](int k) { return field(2 * nlev + 2 + (nder == 2 ? 1 - (k & 1) : 0)); };
  std::vector<const double2 *> lev(steps), stap(steps);
  lev[0] = (const double2 *)U_thin;
  for (int k = 0; k < steps; ++k) {
    double2 *c = k < nlev ? field(nlev + k) : der(k);
    if ((rc = stout_staples(lev[k], c, wp, wr, geo, s))) return rc;
    stap[k] = c;
    if (k == nlev) break;
    stout_exp_kernel<<<grid, 256, 0, s>>>(lev[k], c, field(k), geo.V);
    HIP_TRY(hipGetLastError());
    lev[k + 1] = field(k);
  }
  const double2 *gin = (const double2 *)G_smeared;
  for (int k = steps - 1; k >= 0; --k) {
    double2 *gout = k == 0 ? (double2 *)G_thin : der(k);
    stout_back_local_kernel<<<grid, 256, 0, s>>>(lev[k], stap[k], gin, gam, dir, geo.V);
    HIP_TRY(hipGetLastError());
    stout_back_gather_kernel<<<4u * grid.x, 256, 0, s>>>(lev[k], gam, dir, gout, wp, wr, geo, order);
    HIP_TRY(hipGetLastError());
    gin = gout;
  }
  return OVL_OK;
}

}  // extern "C"
