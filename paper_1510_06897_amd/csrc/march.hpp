// t-marching form of the fused Clenshaw step (plain recurrence steps, one site per thread), for
// launches whose vectors do not fit the 256 MB last-level cache.
//
// A workgroup owns a tile of whole x lines, Lx x ty x tz (up to 256) sites of one (x, y, z)
// cross-section, and marches it through a chunk of consecutive t.  The tile's input spinors of the
// current t, with the faces y0 + ty, y0 - 1, z0 + tz, z0 - 1 (periodic; up to 256 face sites, of which
// there may be more than tile sites), sit in LDS: the x, y and z neighbours and the own value are read
// from there.  The t + 1 slice is read into registers during
// the step (the forward t neighbour of this slice, the LDS contents of the next), and the backward
// t hop is carried as the half-spinor U_t^+ h(t), formed with the link the forward t hop reads.
//
// Why: the direction-split kernels read every spinor eight times and every link twice through L1 and
// L2.  With vectors beyond the last-level cache the re-reads that miss L2 are what they wait for: K and
// the fused K step on 64 FP64 vectors of 16^3 x 32 read 5.4 and 9.5 GB from beyond L2 (their inputs: 1.7
// and 4.9), 4.3 and 7.5 GB here, and take 2.74 ms together instead of 3.65.  Bound by HBM: the 18 right-hand sides of
// 12 x 16^3 x 32 + 4 x 8^3 x 16 + 2 x 12^3 x 24 in FP32 with two-row links move 861 MB in 163 us (5.3
// TB/s; a plain copy: 4.9), the direction-split pair kernel 813 MB in 184 us: in this case the gain is
// the rate, not fewer bytes; the degree-299 sign function takes 49.4 instead of 56.0 ms.
// The registers (FP32 232 to 250, FP64 440 to 476 of 512) leave two FP32 waves or one FP64 wave per
// SIMD, so the loads of a step are issued in a few groups well ahead of their use instead of relying
// on other waves: with each hop waiting for its own link loads the FP64 launches took 1.3x longer.
#pragma once

#include "kernels.hpp"

namespace ovl {

// half-spinor of (1 - SG gamma_MU) on raw (u, d), s5 = -1 applying gamma5
template <int MU, int SG, class C>
__device__ __forceinline__ void half_project(const cx<C> u[2][3], const cx<C> d[2][3], C s5,
                                             cx<C> h[2][3]) {
  using K = DirK<MU>;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const cx<C> dA = K::p ? d[1][c] : d[0][c];
    const cx<C> dB = K::p ? d[0][c] : d[1][c];
    h[0][c] = add_szx<SG * K::z0r, SG * K::z0i>(u[0][c], s5, dA);
    h[1][c] = add_szx<SG * K::z1r, SG * K::z1i>(u[1][c], s5, dB);
  }
}
// r = M h or M^+ h
template <bool DAG, class C>
__device__ __forceinline__ void half_mul(const cx<C> m[3][3], const cx<C> h[2][3], cx<C> r[2][3]) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    r[0][a] = mk<C>(0, 0);
    r[1][a] = mk<C>(0, 0);
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      if (DAG) {
        r[0][a] = cjmadd(r[0][a], m[b][a], h[0][b]);
        r[1][a] = cjmadd(r[1][a], m[b][a], h[1][b]);
      } else {
        r[0][a] = cmadd(r[0][a], m[a][b], h[0][b]);
        r[1][a] = cmadd(r[1][a], m[a][b], h[1][b]);
      }
    }
  }
}
// acc += the 4-spinor of (1 - SG gamma_MU) rebuilt from its half-spinor r
template <int MU, int SG, class C>
__device__ __forceinline__ void half_add(cx<C> acc[12], const cx<C> r[2][3]) {
  using K = DirK<MU>;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    acc[c] = acc[c] + r[0][c];
    acc[3 + c] = acc[3 + c] + r[1][c];
    const cx<C> rA = K::p ? r[1][c] : r[0][c];
    const cx<C> rB = K::p ? r[0][c] : r[1][c];
    acc[6 + c] = acc[6 + c] + zc<SG * K::w0r, SG * K::w0i>(rA);
    acc[9 + c] = acc[9 + c] + zc<SG * K::w1r, SG * K::w1i>(rB);
  }
}

// link at per-lane byte offset voff, scalar byte offset soff; component stride ls bytes
template <class C, class LE, bool R12>
__device__ __forceinline__ void load_link_off(rsrc_t U, uint32_t ls, uint32_t voff, uint32_t soff,
                                              cx<C> m[3][3]) {
#pragma unroll
  for (int a = 0; a < (R12 ? 2 : 3); ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) m[a][b] = bio<LE, C>::ld(U, voff, soff + (a * 3 + b) * ls);
}

constexpr int kMarchThreads = 256;  // most sites of a tile, and most face sites

// Tile of the t-marching form for a lattice: whole x lines, ty x tz in (y, z) dividing the extents,
// n = Lx ty tz sites in whole waves, at most kMarchThreads, and no more face sites than that (a thread
// stages at most one tile site and one face site; the faces may outnumber the tile's sites, as for
// 32 x 2 x 2 with 128 and 256); the links' t slices must be whole 64-site blocks.  Among the tiles the
// one with the fewest face sites per site wins.  Returns n (0: none fits).
inline int march_tile(const Geom &g, int &ty, int &tz) {
  ty = tz = 0;
  if ((int64_t)g.L[0] * g.L[1] * g.L[2] % 64 || g.L[0] > kMarchThreads) return 0;
  int64_t best = 0, bh = 0;
  for (int a = 1; a <= g.L[1] && g.L[0] * a <= kMarchThreads; ++a)
    for (int b = 1; b <= g.L[2] && g.L[0] * a * b <= kMarchThreads; ++b) {
      const int64_t n = (int64_t)g.L[0] * a * b;
      if (g.L[1] % a || g.L[2] % b || n % 64) continue;
      const int64_t h = (a < g.L[1] ? 2 * g.L[0] * b : 0) + (b < g.L[2] ? 2 * g.L[0] * a : 0);
      if (h > kMarchThreads || (best && h * best >= bh * n)) continue;
      best = n;
      bh = h;
      ty = a;
      tz = b;
    }
  return (int)best;
}

// Least t slices of a chunk for a launch of `slices` tile slices: the longest of 4, 8, 16, 32 that
// leaves 2048 workgroups (a chunk re-reads the slices before and after it, so longer is less
// traffic: 64 FP64 vectors of 16^3 x 32 2.91, 2.78, 2.73 ms at 8, 16, 32; but a launch of few
// workgroups ends in a nearly empty round: 12 vectors 263, 273, 288 us at 4, 8, 16).
inline int march_chunk(int64_t slices) {
  int ct = 4;
  while (ct < 32 && slices / (2 * ct) >= 2048) ct *= 2;
  return ct;
}
// chunks of Lt slices: the lengths are ct or more, up to 2 ct - 1 (an extent of 5, 6 or 7 is one chunk: 16^3 x 7,
// 28 FP64 vectors 136 us, in two chunks 175; 16^3 x 6, 32 vectors 124 and 134)
inline int march_chunks(int lt, int ct) { return lt / ct > 1 ? lt / ct : 1; }
// Plans the items of a launch (all of them have a tile); returns its workgroups.
inline int march_plan(StepItem *items, int n) {
  int64_t slices = 0;
  for (int i = 0; i < n; ++i) {
    StepItem &it = items[i];
    slices += (int64_t)it.g.V / march_tile(it.g, it.mty, it.mtz) * it.nrhs;
  }
  const int ct = march_chunk(slices);
  int blocks = 0;
  for (int i = 0; i < n; ++i) {
    StepItem &it = items[i];
    const int tiles = it.g.L[1] / it.mty * (it.g.L[2] / it.mtz);
    it.nt = march_chunks(it.g.L[3], ct);
    // the tiles of about 32 workgroups (an XCD's compute units) run side by side, so that faces are
    // read from its L2
    it.mgroup = tiles < 32 ? 32 / tiles : 1;
    it.mblk0 = blocks;
    blocks += it.nrhs * tiles * it.nt;
  }
  return blocks;
}

// LDS bytes of a workgroup: 12 components of the tile and its faces
template <class C>
__host__ __device__ constexpr int march_lds_bytes() {
  return 12 * 2 * kMarchThreads * (int)sizeof(cx<C>);
}

// A workgroup's share of an item and a thread's place in it.
struct MarchPlace {
  int r, tile, t0, t1;          // right-hand side, tile, chunk [t0, t1)
  int n, nh;                    // tile sites, face sites
  int y0, z0;                   // corner of the tile
  int hy, hz;                   // sites of one y face, one z face (0: the tile wraps there)
  // thread tid stages (and computes) tile site tid, and stages face site tid: each by its own bound,
  // as either count may be the larger
  __host__ __device__ bool tile_lane(int tid) const { return tid < n; }
  __host__ __device__ bool face_lane(int tid) const { return tid < nh; }
};
__host__ __device__ __forceinline__ MarchPlace march_place(const StepItem &I, const Ext4 &ex, int lb) {
  MarchPlace p;
  const int ty = I.mty, tz = I.mtz, nrhs = I.nrhs;
  const int nty = ex.ly / ty, ntile = nty * (ex.lz / tz);
  // workgroup order: right-hand sides of a group, tiles, groups, t chunks
  const int per = nrhs * ntile;
  const int chunk = lb / per;
  lb -= chunk * per;
  const int gs = min(I.mgroup, nrhs);
  const int full = nrhs / gs, span = gs * ntile;
  const int gi = min(lb / span, full);
  const int gl = gi < full ? gs : nrhs - full * gs;
  const int within = lb - gi * span;
  p.r = gi * gs + within % gl;
  p.tile = within / gl;
  // chunk lengths differ by at most one; which chunks are the long ones varies with the tile and the
  // right-hand side, as an XCD's range of workgroups holds few chunks (16^3 x 33, FP32, 8 chunks, the long
  // one always last / varying: 11 vectors 163 / 150 us, 21 vectors 296 / 271)
  const int turn = (p.r + p.tile) % I.nt;
  p.t0 = (chunk * ex.lt + turn) / I.nt;
  p.t1 = ((chunk + 1) * ex.lt + turn) / I.nt;
  p.n = ex.lx * ty * tz;
  p.y0 = (p.tile % nty) * ty;
  p.z0 = (p.tile / nty) * tz;
  p.hy = ty < ex.ly ? ex.lx * tz : 0;
  p.hz = tz < ex.lz ? ex.lx * ty : 0;
  p.nh = 2 * p.hy + 2 * p.hz;
  return p;
}
// (x, y, z) site index of staged site j: the tile's sites, then the faces y + ty, y - 1, z + tz, z - 1
__host__ __device__ __forceinline__ int march_staged(const MarchPlace &p, const StepItem &I, const Ext4 &ex,
                                            int j) {
  int xx, yy, zz;
  if (j < p.n) {
    xx = j % ex.lx;
    const int row = j / ex.lx;
    yy = p.y0 + row % I.mty;
    zz = p.z0 + row / I.mty;
  } else if (j < p.n + 2 * p.hy) {
    int f = j - p.n;
    const bool lo = f >= p.hy;
    f -= lo ? p.hy : 0;
    xx = f % ex.lx;
    zz = p.z0 + f / ex.lx;
    yy = lo ? (p.y0 == 0 ? ex.ly - 1 : p.y0 - 1) : (p.y0 + I.mty == ex.ly ? 0 : p.y0 + I.mty);
  } else {
    int f = j - p.n - 2 * p.hy;
    const bool lo = f >= p.hz;
    f -= lo ? p.hz : 0;
    xx = f % ex.lx;
    yy = p.y0 + f / ex.lx;
    zz = lo ? (p.z0 == 0 ? ex.lz - 1 : p.z0 - 1) : (p.z0 + I.mtz == ex.lz ? 0 : p.z0 + I.mtz);
  }
  return xx + ex.sy * yy + ex.sz * zz;
}
// staged indices of a tile site's six neighbours and the sites behind it (whose links it reads)
struct MarchSite {
  int s3, xm3, ym3, zm3;
  int jxp, jxm, jyp, jym, jzp, jzm;
};
__host__ __device__ __forceinline__ MarchSite march_site(const MarchPlace &p, const StepItem &I,
                                                const Ext4 &ex, int sj) {
  MarchSite m;
  const int ty = I.mty, tz = I.mtz, n = p.n;
  const int x = sj % ex.lx, row = sj / ex.lx;
  const int yl = row % ty, zl = row / ty;
  const int y = p.y0 + yl, z = p.z0 + zl;
  m.s3 = x + ex.sy * y + ex.sz * z;
  m.xm3 = x == 0 ? m.s3 + ex.lx - 1 : m.s3 - 1;
  m.ym3 = y == 0 ? m.s3 + (ex.ly - 1) * ex.sy : m.s3 - ex.sy;
  m.zm3 = z == 0 ? m.s3 + (ex.lz - 1) * ex.sz : m.s3 - ex.sz;
  const int fy = x + ex.lx * zl, fz = x + ex.lx * yl;
  const int wy = (ty - 1) * ex.lx, wz = (tz - 1) * ex.lx * ty;
  m.jxp = x + 1 == ex.lx ? sj + 1 - ex.lx : sj + 1;
  m.jxm = x == 0 ? sj + ex.lx - 1 : sj - 1;
  m.jyp = yl + 1 < ty ? sj + ex.lx : (p.hy ? n + fy : sj - wy);
  m.jym = yl > 0 ? sj - ex.lx : (p.hy ? n + p.hy + fy : sj + wy);
  m.jzp = zl + 1 < tz ? sj + ex.lx * ty : (p.hz ? n + 2 * p.hy + fz : sj - wz);
  m.jzm = zl > 0 ? sj - ex.lx * ty : (p.hz ? n + 2 * p.hy + p.hz + fz : sj + wz);
  return m;
}

template <class C, class SE, class LE, bool TABLE, bool R12>
__global__ void __launch_bounds__(kMarchThreads, sizeof(C) == 4 ? 2 : 1)
    march_kernel(StepArgs<TABLE> p) {
  constexpr int NS = 2 * kMarchThreads;
  extern __shared__ __align__(16) unsigned char march_smem[];
  cx<C> *stage = reinterpret_cast<cx<C> *>(march_smem);  // [12][NS]
  const int gb = xcd_block(blockIdx.x, gridDim.x, p.remap);
  int it = 0;
  if (TABLE)
    for (int i = 1; i < p.n_items; ++i)
      if (p.table[i].mblk0 <= gb) it = i;
  const StepItem &I = TABLE ? p.table[it] : p.item;
  const Ext4 ex = ext_of(I.g);
  const MarchPlace mp = march_place(I, ex, gb - I.mblk0);
  const int r = mp.r, t0 = mp.t0, t1 = mp.t1, n = mp.n, V3 = ex.st;
  const int tid = threadIdx.x;
  // (a tile is whole waves: one answer per wave, and scalar branches on it)
  const bool active = __builtin_amdgcn_readfirstlane(mp.tile_lane(tid)) != 0, hactive = mp.face_lane(tid);
  const int sj = active ? tid : 0;
  const MarchSite ms = march_site(mp, I, ex, sj);
  const int jxp = ms.jxp, jxm = ms.jxm, jyp = ms.jyp, jym = ms.jym, jzp = ms.jzp, jzm = ms.jzm;
  const int hs3 = hactive ? march_staged(mp, I, ex, n + tid) : 0;
  constexpr uint32_t SB = elem_traits<SE>::bytes, LB = elem_traits<LE>::bytes;
  const uint32_t cs = (uint32_t)ex.V * SB, vb = 12u * cs;
  const uint32_t ts = (uint32_t)V3 * SB;                       // bytes per t slice of a component
  const uint32_t ls = (uint32_t)I.lstride * LB;                // bytes between link components
  const uint32_t lt = (uint32_t)(V3 >> 6) * 36u * ls;          // bytes per t slice of the links
  const uint32_t vo = (uint32_t)ms.s3 * SB, vh = (uint32_t)hs3 * SB;
  const uint32_t lo = link_lane(ms.s3) * LB, lx = link_lane(ms.xm3) * LB,
                 ly = link_lane(ms.ym3) * LB, lz = link_lane(ms.zm3) * LB;
  const rsrc_t v = make_rsrc(role_vec<SE>(I, p.v_role, r, ex.V), vb);
  const rsrc_t U = make_rsrc(I.U, link_bytes(ex.V, ls));
  const rsrc_t o = make_rsrc(role_vec<SE>(I, p.out_role, r, ex.V), vb);
  const double pa = role_a(I, p.a, r);
  // absent operands read as zero (an empty range), so the loads need no branch
  const bool has_src = pa != 0.0, has_w = p.w_role != ROLE_NONE;
  const rsrc_t sr = make_rsrc(role_vec<SE>(I, has_src ? ROLE_PSI : p.v_role, r, ex.V), has_src ? vb : 0u);
  const rsrc_t w = make_rsrc(role_vec<SE>(I, has_w ? p.w_role : p.v_role, r, ex.V), has_w ? vb : 0u);
  // gamma5 on the input, the output (y_g5) and psi (src_g5): signs of the lower spin pair
  const C s5 = p.v_g5 ? C(-1) : C(1);
  const C sy = p.y_g5 ? C(-1) : C(1);
  const C al = C(pa), ah = p.src_g5 ? C(-pa) : C(pa), tw = C(p.t);
  const C kd = C(p.kd), kh = C(p.kh);

  cx<C> pu[2][3], pd[2][3], hu[2][3], hd[2][3];  // t + 1 slice: own and face site
  cx<C> bt[2][3];                                // U_t^+(t - 1) h(t - 1)
  auto load12 = [&](uint32_t voff, int t, cx<C> u[2][3], cx<C> d[2][3]) {
    const uint32_t so = (uint32_t)t * ts;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        u[s][c] = bio<SE, C>::ld(v, voff, so + (s * 3 + c) * cs);
        d[s][c] = bio<SE, C>::ld(v, voff, so + ((s + 2) * 3 + c) * cs);
      }
  };
  auto put12 = [&](int j, const cx<C> u[2][3], const cx<C> d[2][3]) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        stage[(s * 3 + c) * NS + j] = u[s][c];
        stage[((s + 2) * 3 + c) * NS + j] = d[s][c];
      }
  };
  auto get12 = [&](int j, cx<C> u[2][3], cx<C> d[2][3]) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        u[s][c] = stage[(s * 3 + c) * NS + j];
        d[s][c] = stage[((s + 2) * 3 + c) * NS + j];
      }
  };
  auto link = [&](uint32_t voff, int mu, int t, cx<C> m[3][3]) {
    load_link_off<C, LE, R12>(U, ls, voff, (uint32_t)t * lt + (uint32_t)mu * 9u * ls, m);
  };
  cx<C> k0[3][3], k1[3][3], k2[3][3], k3[3][3];  // links in flight
  auto links4 = [&](int t) {
    link(lo, 0, t, k0);
    link(lx, 0, t, k1);
    link(lo, 1, t, k2);
    link(ly, 1, t, k3);
  };
  if (!active) {  // a wave beside the tile: its share of the faces, and the barriers of the others
    for (int t = t0; t < t1; ++t) {
      if (hactive) load12(vh, t, hu, hd);
      if (t > t0) __syncthreads();
      if (hactive) put12(n + tid, hu, hd);
      __syncthreads();
    }
    return;
  }
  {
    const int tm = t0 == 0 ? ex.lt - 1 : t0 - 1;
    cx<C> h[2][3];
    load12(vo, t0, pu, pd);
    if (hactive) load12(vh, t0, hu, hd);
    link(lo, 3, tm, k0);
    put12(sj, pu, pd);
    if (hactive) put12(n + tid, hu, hd);
    load12(vo, tm, pu, pd);
    if (R12) su3_row2(k0);
    half_project<3, -1>(pu, pd, s5, h);
    half_mul<true>(k0, h, bt);
    links4(t0);
  }
  __syncthreads();
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using M1 = std::integral_constant<int, -1>;
  // Loads complete in issue order, so each group is issued after everything that is waited for
  // before it: x and y links (issued before the barrier), the z links, the t + 1 slice, the t link,
  // psi and w.
  for (int t = t0; t < t1; ++t) {
    const uint32_t so = (uint32_t)t * ts;
    cx<C> acc[12], dir[12], wv[12], sv[12];  // hopping sum, one direction's part, w and psi
    auto settle = [&](cx<C> *q) {
#pragma unroll
      for (int i = 0; i < 12; ++i) pin(q[i]);
      __builtin_amdgcn_sched_barrier(0);
    };
    auto hop = [&](auto mu_, auto sg_, int j, cx<C> m[3][3]) {
      constexpr int MU = decltype(mu_)::value, SG = decltype(sg_)::value;
      cx<C> u[2][3], d[2][3], h[2][3], rr[2][3];
      if (SG > 0) {
#pragma unroll
        for (int i = 0; i < 12; ++i) dir[i] = mk<C>(0, 0);
      }
      get12(j, u, d);
      half_project<MU, SG>(u, d, s5, h);
      if (R12) su3_row2(m);
      half_mul<(SG < 0)>(m, h, rr);
      half_add<MU, SG>(dir, rr);
      settle(dir);
    };
    // the directions' parts are added in the order of the direction-split kernels, ((x + y) + z) + t
    // with forward before backward, so that every launch form gives the same bits
    auto add_dir = [&]() {
#pragma unroll
      for (int i = 0; i < 12; ++i) acc[i] = acc[i] + dir[i];
    };
    hop(I0{}, I1{}, jxp, k0);
    hop(I0{}, M1{}, jxm, k1);
#pragma unroll
    for (int i = 0; i < 12; ++i) acc[i] = dir[i];
    settle(acc);
    link(lo, 2, t, k0);
    link(lz, 2, t, k1);
    __builtin_amdgcn_sched_barrier(0);
    hop(I1{}, I1{}, jyp, k2);
    hop(I1{}, M1{}, jym, k3);
    add_dir();
    settle(acc);
    const int tn = t + 1 == ex.lt ? 0 : t + 1;
    load12(vo, tn, pu, pd);
    if (hactive && t + 1 < t1) load12(vh, tn, hu, hd);
    __builtin_amdgcn_sched_barrier(0);
    hop(I2{}, I1{}, jzp, k0);
    hop(I2{}, M1{}, jzm, k1);
    add_dir();
    settle(acc);
    link(lo, 3, t, k2);
#pragma unroll
    for (int i = 0; i < 12; ++i) sv[i] = bio<SE, C>::ld(sr, vo, so + i * cs);
#pragma unroll
    for (int i = 0; i < 12; ++i) wv[i] = bio<SE, C>::ld(w, vo, so + i * cs);
    __builtin_amdgcn_sched_barrier(0);
    // t forward with the t + 1 slice, t backward with the carried half-spinor, and the one carried on
    cx<C> u[2][3], d[2][3], h[2][3], rr[2][3];
#pragma unroll
    for (int i = 0; i < 12; ++i) dir[i] = mk<C>(0, 0);
    half_project<3, 1>(pu, pd, s5, h);
    if (R12) su3_row2(k2);
    half_mul<false>(k2, h, rr);
    half_add<3, 1>(dir, rr);
    half_add<3, -1>(dir, bt);
    add_dir();
    settle(acc);
    get12(sj, u, d);
    half_project<3, -1>(u, d, s5, h);
    half_mul<true>(k2, h, bt);
#pragma unroll
    for (int i = 0; i < 12; ++i) {
      const cx<C> v0 = i < 6 ? u[i / 3][i % 3] : d[i / 3 - 2][i % 3];
      const cx<C> xv = i < 6 ? v0 : mk<C>(s5 * v0.re, s5 * v0.im);
      // the roundings of the direction-split kernels, spelled out
      cx<C> yv = mk<C>(fma(kd, xv.re, kh * acc[i].re), fma(kd, xv.im, kh * acc[i].im));
      if (i >= 6) yv = mk<C>(sy * yv.re, sy * yv.im);
      const C ai = i < 6 ? al : ah;
      yv = mk<C>(fma(ai, sv[i].re, yv.re), fma(ai, sv[i].im, yv.im));
      acc[i] = mk<C>(fma(tw, wv[i].re, yv.re), fma(tw, wv[i].im, yv.im));
    }
#pragma unroll
    for (int i = 0; i < 12; ++i) bio<SE, C>::st(o, vo, so + i * cs, acc[i]);
    if (t + 1 < t1) {
      __syncthreads();
      links4(t + 1);
      put12(sj, pu, pd);
      if (hactive) put12(n + tid, hu, hd);
      __syncthreads();
    }
  }
}

}  // namespace ovl
