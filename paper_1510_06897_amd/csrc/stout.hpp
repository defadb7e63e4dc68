// Stout smearing of the gauge links on the device and its chain-rule derivative (FP64).
//
// The links entering K are smoothed by three steps of over-improved stout smearing with
// rho = 0.1 and eps = -0.25 (Sec. 2).  One step replaces every link at once by
//   U'_mu(x) = exp(M) U_mu(x),   M = TA(Omega) = (Omega - Omega^+)/2 - tr(Omega - Omega^+)/6,
//   Omega = C_mu(x) U_mu(x)^+,
// where C_mu(x) sums the paths from x to x + mu that close a loop with the link: the three-link
// plaquette staples with weight rho c_p and the five-link staples of the 2 x 1 rectangles with
// weight rho c_r, c_p = (5 - 2 eps)/3, c_r = -(1 - eps)/12 (the over-improved gauge action; eps = 1
// leaves the plaquette alone: plain stout smearing).
//
// Links are read and written in the caller layout U[mu][a][b][site] (complex double), so one
// wave reads one matrix element of 64 consecutive sites per load; the path factors are read
// through raw buffer resources (lane offset site * 16 bytes, element offset in a scalar register),
// so a field must span less than 4 GiB.  A thread owns one link
// (site, mu); the workgroup's 256 threads share mu, so the path loops below are uniform over a
// wave.  exp(M) and its Frechet derivative: m3.hpp.
#pragma once

#include "m3.hpp"

namespace ovl {

// element (a, b) of link `dir` at `site`: U[dir][a][b][site]
__device__ __forceinline__ M3 load_m3(const double2 *__restrict__ U, int dir, int site, int V) {
  M3 r;
  const double2 *p = U + (int64_t)dir * 9 * V + site;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const double2 v = p[(int64_t)(3 * i + j) * V];
      r.e[i][j] = mk<double>(v.x, v.y);
    }
  return r;
}
__device__ __forceinline__ void store_m3(double2 *__restrict__ U, int dir, int site, int V,
                                         const M3 &m) {
  double2 *p = U + (int64_t)dir * 9 * V + site;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) p[(int64_t)(3 * i + j) * V] = make_double2(m.e[i][j].re, m.e[i][j].im);
}

// ---------------------------------------------------------------------------------------------
// Staple paths.  For a link along mu, a plane mu-nu (nu != mu) and an orientation s = +1 or -1 of
// nu, four paths lead from x to x + mu:
//   shape 0  plaquette            (nu,s)  (mu,+)  (nu,-s)
//   shape 1  2 x 1, link first    (nu,s)  (mu,+)  (mu,+)  (nu,-s) (mu,-)
//   shape 2  2 x 1, link second   (mu,-)  (nu,s)  (mu,+)  (mu,+)  (nu,-s)
//   shape 3  1 x 2                (nu,s)  (nu,s)  (mu,+)  (nu,-s) (nu,-s)
// A step (d,+) from position z takes the factor U_d(x + z) and moves to z + e_d; a step (d,-)
// moves to z - e_d and takes U_d(x + z - e_d)^+.  Together with the link these are the 6
// plaquettes and 18 rectangles that contain it.
__device__ __forceinline__ int path_len(int shape) { return shape == 0 ? 3 : 5; }

__device__ __forceinline__ void path_step(int mu, int nu, int s, int shape, int k, int &dir,
                                          int &sgn) {
  // (direction selector, sign) per position: 0 = mu, 1 = nu; sign in units of s for nu
  int sel, sg;
  switch (shape) {
    case 0: sel = (k == 1) ? 0 : 1; sg = (k == 0) ? 1 : (k == 1 ? 1 : -1); break;
    case 1: sel = (k == 1 || k == 2 || k == 4) ? 0 : 1; sg = (k == 3 || k == 4) ? -1 : 1; break;
    case 2: sel = (k == 1 || k == 4) ? 1 : 0; sg = (k == 0 || k == 4) ? -1 : 1; break;
    default: sel = (k == 2) ? 0 : 1; sg = (k >= 3) ? -1 : 1; break;
  }
  dir = sel == 0 ? mu : nu;
  sgn = sel == 0 ? sg : sg * s;
}

struct SiteCoord {
  int c[4];
};
__device__ __forceinline__ SiteCoord site_coord(int site, const Geom &g) {
  SiteCoord r;
  int v = site;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    r.c[d] = v % g.L[d];
    v /= g.L[d];
  }
  return r;
}

// Positions on the paths of link (x, mu) in the plane (mu, nu): a path moves along mu and nu only,
// so a position is x + a e_mu + b e_nu (|a|, |b| <= 2) and its site index takes two periodic wraps.
struct PlaneAddr {
  int rest;    // site index of x without its mu and nu parts
  int xm, xn;  // coordinates of x along mu and nu
  int lm, ln;  // extents along mu and nu
  int sm, sn;  // strides along mu and nu
};
__device__ __forceinline__ PlaneAddr plane_addr(const SiteCoord &x, int site, int mu, int nu,
                                                const Geom &g) {
  PlaneAddr p;
  p.xm = x.c[mu];
  p.xn = x.c[nu];
  p.lm = g.L[mu];
  p.ln = g.L[nu];
  p.sm = g.stride[mu];
  p.sn = g.stride[nu];
  p.rest = site - p.xm * p.sm - p.xn * p.sn;
  return p;
}
// v mod L for -2 L <= v < 3 L (two conditional steps each way also cover extent 1)
__device__ __forceinline__ int wrap2(int v, int L) {
  v += v < 0 ? L : 0;
  v += v < 0 ? L : 0;
  v -= v >= L ? L : 0;
  v -= v >= L ? L : 0;
  return v;
}
__device__ __forceinline__ int plane_site(const PlaneAddr &p, int a, int b) {
  return p.rest + wrap2(p.xm + a, p.lm) * p.sm + wrap2(p.xn + b, p.ln) * p.sn;
}

// link field U[dir][a][b][site] read through a buffer resource
__device__ __forceinline__ M3 load_m3r(rsrc_t r, int dir, int site, int V) {
  M3 m;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      m.e[i][j] = bld<double, double2>(r, (uint32_t)((dir * 9 + 3 * i + j) * V) * 16u, site);
  return m;
}

// Path step k of (shape, s): along mu (along = 0) or nu (1), forward (fwd) or backward, from
// the path_step table.  A forward step at position (a, b) takes U_dir(x + a e_mu + b e_nu) and
// moves on; a backward step moves first and takes the link there, daggered.
__device__ __forceinline__ void path_move(int shape, int k, int s, int &along, bool &fwd) {
  int dir, sgn;
  path_step(0, 1, s, shape, k, dir, sgn);
  along = dir;
  fwd = sgn > 0;
}
__device__ __forceinline__ M3 path_factor(rsrc_t U, const PlaneAddr &pa, int &a, int &b,
                                          int along, bool fwd, int mu, int nu, int V) {
  const int dir = along == 0 ? mu : nu;
  int &z = along == 0 ? a : b;
  if (fwd) {
    const M3 f = load_m3r(U, dir, plane_site(pa, a, b), V);
    z += 1;
    return f;
  }
  z -= 1;
  return m3_dag(load_m3r(U, dir, plane_site(pa, a, b), V));
}

// C_mu(x) = sum over the paths of their products, plaquette paths weighted wp, rectangles wr
__device__ inline M3 staple_sum(rsrc_t U, const SiteCoord &x, int site, int mu, double wp,
                                double wr, const Geom &g) {
  M3 c = m3_zero();
  for (int nu = 0; nu < 4; ++nu) {
    if (nu == mu) continue;
    const PlaneAddr pa = plane_addr(x, site, mu, nu, g);
    for (int s = 1; s >= -1; s -= 2) {
      // shapes 0 and 1 share their first two factors (nu,s)(mu,+): the plaquette closes from
      // there, the rectangle goes on from the same product and position
      int a = 0, b = 0, along;
      bool fwd;
      path_move(0, 0, s, along, fwd);
      M3 p = path_factor(U, pa, a, b, along, fwd, mu, nu, g.V);
      path_move(0, 1, s, along, fwd);
      p = m3_mul(p, path_factor(U, pa, a, b, along, fwd, mu, nu, g.V));
      if (wp != 0.0) {
        int a0 = a, b0 = b;
        path_move(0, 2, s, along, fwd);
        c = m3_axpy(c, wp, m3_mul(p, path_factor(U, pa, a0, b0, along, fwd, mu, nu, g.V)));
      }
      if (wr == 0.0) continue;
      for (int k = 2; k < path_len(1); ++k) {
        path_move(1, k, s, along, fwd);
        p = m3_mul(p, path_factor(U, pa, a, b, along, fwd, mu, nu, g.V));
      }
      c = m3_axpy(c, wr, p);
      for (int shape = 2; shape < 4; ++shape) {
        a = b = 0;
        path_move(shape, 0, s, along, fwd);
        p = path_factor(U, pa, a, b, along, fwd, mu, nu, g.V);
        for (int k = 1; k < path_len(shape); ++k) {
          path_move(shape, k, s, along, fwd);
          p = m3_mul(p, path_factor(U, pa, a, b, along, fwd, mu, nu, g.V));
        }
        c = m3_axpy(c, wr, p);
      }
    }
  }
  return c;
}

// Workgroup order of the path kernels: a launch of 4 ceil(V / 256) workgroups, XCD-contiguous ranges,
// the four directions of 256 sites side by side; the sites in memory order, or (ty > 0) in t-streaming
// tiles -- whole x lines, ty x tz in (y, z), consecutive workgroups walking t.  The paths of the four
// directions run over the same links, so what one workgroup reads its neighbours on the XCD find in
// L2.  (With the directions one after the other over the whole lattice and workgroups dealt round
// robin to the XCDs the kernels waited for L2 misses: three steps of 24^3 x 48 take 6.1 ms forward and
// 20.3 ms backward instead of 13.2 and 41.2, of 16^3 x 32 1.39 and 4.20 instead of 2.1 and 7.8.)
struct StoutOrder {
  int ty, tz;
};
__device__ __forceinline__ int stout_site(const Geom &g, StoutOrder o, int &mu) {
  const int gb = xcd_block(blockIdx.x, gridDim.x, 1);
  mu = gb & 3;
  if (o.ty <= 0) return (gb >> 2) * 256 + threadIdx.x;
  const int slice = g.L[0] * o.ty * o.tz, nsub = slice / 256;
  const int tb = (gb >> 2) / nsub;
  const int local = ((gb >> 2) - tb * nsub) * 256 + threadIdx.x;
  const int t = tb % g.L[3], tile = tb / g.L[3], nty = g.L[1] / o.ty;
  const int x = local % g.L[0], row = local / g.L[0];
  const int y = (tile % nty) * o.ty + row % o.ty, z = (tile / nty) * o.tz + row / o.ty;
  return x + g.stride[1] * y + g.stride[2] * z + g.stride[3] * t;
}

// C_mu(x) of every link.  146 registers, three waves per SIMD (bounded to 128 for four: 373 -> 415 us
// at 16^3 x 32).
__global__ void __launch_bounds__(256)
    stout_staple_kernel(const double2 *__restrict__ U, double2 *__restrict__ C, double wp, double wr,
                        Geom g, StoutOrder order) {
  int mu;
  const int site = stout_site(g, order, mu);
  if (site >= g.V) return;
  store_m3(C, mu, site, g.V,
           staple_sum(make_rsrc(U, 576u * (uint32_t)g.V), site_coord(site, g), site, mu, wp, wr, g));
}

// One smearing step from the staple sums: out_mu(x) = exp(TA(C_mu(x) U_mu(x)^+)) U_mu(x).  out may be C.
// Grid (ceil(V / 256), 4).  Apart from the staple kernel, which then needs fewer registers.
__global__ void __launch_bounds__(256)
    stout_exp_kernel(const double2 *U, const double2 *C, double2 *out, int V) {
  const int site = blockIdx.x * 256 + threadIdx.x;
  const int mu = blockIdx.y;
  if (site >= V) return;
  const M3 c = load_m3(C, mu, site, V), u = load_m3(U, mu, site, V);
  store_m3(out, mu, site, V, m3_axpy(u, 1.0, m3_mul(m3_expm1(m3_ta(m3_muld(c, u))), u)));
}

// Backward of one step, the part local to each link.  With G' = dL/dRe U' + i dL/dIm U' of the
// step's output (same convention throughout):
//   dL/dE = G' U^+,  dL/dM = L(M^+, dL/dE)  (the adjoint of the Frechet derivative of exp at M),
//   dL/dOmega = (g - g^+)/2 - (i/3) Im tr(g) for g = dL/dM  (M = TA(Omega)),
//   Gamma = dL/dC = dL/dOmega U,   direct = E^+ G' + (dL/dOmega)^+ C.
// Writes Gamma and the direct part of dL/dU; C: the level's staple sums.  Grid (ceil(V / 256), 4).
__global__ void __launch_bounds__(256)
    stout_back_local_kernel(const double2 *__restrict__ U, const double2 *__restrict__ C,
                            const double2 *__restrict__ gout, double2 *__restrict__ gamma,
                            double2 *__restrict__ direct, int V) {
  const int site = blockIdx.x * 256 + threadIdx.x;
  const int mu = blockIdx.y;
  if (site >= V) return;
  const M3 c = load_m3(C, mu, site, V);
  const M3 u = load_m3(U, mu, site, V);
  const M3 m = m3_ta(m3_muld(c, u));
  const M3 gp = load_m3(gout, mu, site, V);
  // exp(M^+) = exp(-M) = E^+ (M is anti-Hermitian), and dL/dM = L(M^+, G' U^+)
  M3 ed, gm;  // E^+ - 1
  m3_expm1_frechet(m3_scale(m, -1.0), m3_muld(gp, u), &ed, &gm);
  const M3 go = m3_ta(gm);
  store_m3(gamma, mu, site, V, m3_mul(go, u));
  store_m3(direct, mu, site, V, m3_axpy(gp, 1.0, m3_muladd(m3_dmul(go, c), ed, gp)));
}

// Backward of one step, the staple part.  Link (y, d) receives w A^+ Gamma_nu(x) B^+ (its adjoint
// for a backward step) from every staple path of every link (x, nu) that runs through it, A and B
// the path's products before and after it.  Summed over the paths through (y, d), this equals the
// derivative of (y, d)'s own staple sum C_d(y) in the direction Gamma: every factor of each of its
// staple paths replaced in turn by the Gamma matrix of the same link, daggered like the factor
// (the staple sum is the gradient of the gauge action, whose second derivative is symmetric).  So
// each link walks its own 24 paths once, carrying the product X and its derivative T:
//   X <- X F,  T <- T F + X Gamma(F).
// out = direct + sum_paths w T: dL/dU of the step's input.
// factor of path step (dir, sgn) at `pos` of U and the same link of Gamma (both daggered for a
// backward step); pos is advanced
__device__ __forceinline__ void path_factor2(rsrc_t U, rsrc_t Gm, const PlaneAddr &pa, int &a,
                                             int &b, int along, bool fwd, int mu, int nu, int V,
                                             M3 &f, M3 &gf) {
  const int dir = along == 0 ? mu : nu;
  int &z = along == 0 ? a : b;
  if (fwd) {
    const int site = plane_site(pa, a, b);
    f = load_m3r(U, dir, site, V);
    gf = load_m3r(Gm, dir, site, V);
    z += 1;
  } else {
    z -= 1;
    const int site = plane_site(pa, a, b);
    f = m3_dag(load_m3r(U, dir, site, V));
    gf = m3_dag(load_m3r(Gm, dir, site, V));
  }
}

__global__ void __launch_bounds__(256)
    stout_back_gather_kernel(const double2 *__restrict__ U, const double2 *__restrict__ gamma,
                             const double2 *__restrict__ direct, double2 *__restrict__ out,
                             double wp, double wr, Geom g, StoutOrder order) {
  int d;
  const int site = stout_site(g, order, d);
  if (site >= g.V) return;
  const SiteCoord y = site_coord(site, g);
  const rsrc_t ru = make_rsrc(U, 576u * (uint32_t)g.V);
  const rsrc_t rg = make_rsrc(gamma, 576u * (uint32_t)g.V);
  M3 acc = load_m3(direct, d, site, g.V);
  for (int nu = 0; nu < 4; ++nu) {
    if (nu == d) continue;
    const PlaneAddr pa = plane_addr(y, site, d, nu, g);
    for (int s = 1; s >= -1; s -= 2) {
      // shapes 0 and 1 share their first two factors (nu,s)(mu,+): the plaquette closes from
      // there, the rectangle goes on from the same (X, T) and position
      int a = 0, b = 0, along;
      bool fwd;
      M3 x, t, f, gf;
      path_move(0, 0, s, along, fwd);
      path_factor2(ru, rg, pa, a, b, along, fwd, d, nu, g.V, x, t);
      path_move(0, 1, s, along, fwd);
      path_factor2(ru, rg, pa, a, b, along, fwd, d, nu, g.V, f, gf);
      t = m3_axpy(m3_mul(t, f), 1.0, m3_mul(x, gf));
      x = m3_mul(x, f);
      if (wp != 0.0) {
        int a0 = a, b0 = b;
        path_move(0, 2, s, along, fwd);
        path_factor2(ru, rg, pa, a0, b0, along, fwd, d, nu, g.V, f, gf);
        acc = m3_axpy(acc, wp, m3_axpy(m3_mul(t, f), 1.0, m3_mul(x, gf)));
      }
      if (wr == 0.0) continue;
      for (int k = 2; k < path_len(1); ++k) {
        path_move(1, k, s, along, fwd);
        path_factor2(ru, rg, pa, a, b, along, fwd, d, nu, g.V, f, gf);
        t = m3_axpy(m3_mul(t, f), 1.0, m3_mul(x, gf));
        if (k + 1 < path_len(1)) x = m3_mul(x, f);
      }
      acc = m3_axpy(acc, wr, t);
      for (int shape = 2; shape < 4; ++shape) {
        a = b = 0;
        path_move(shape, 0, s, along, fwd);
        path_factor2(ru, rg, pa, a, b, along, fwd, d, nu, g.V, x, t);
        const int len = path_len(shape);
        for (int k = 1; k < len; ++k) {
          path_move(shape, k, s, along, fwd);
          path_factor2(ru, rg, pa, a, b, along, fwd, d, nu, g.V, f, gf);
          t = m3_axpy(m3_mul(t, f), 1.0, m3_mul(x, gf));
          if (k + 1 < len) x = m3_mul(x, f);
        }
        acc = m3_axpy(acc, wr, t);
      }
    }
  }
  store_m3(out, d, site, g.V, acc);
}

}  // namespace ovl
