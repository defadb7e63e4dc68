// 3 x 3 complex FP64 matrices in registers, the exponential of a traceless one and its derivative.
#pragma once

#include "common.hpp"

namespace ovl {

struct M3 {
  cx<double> e[3][3];
};

__host__ __device__ __forceinline__ M3 m3_zero() {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) r.e[i][j] = mk<double>(0.0, 0.0);
  return r;
}
// R + A B
__host__ __device__ __forceinline__ M3 m3_muladd(const M3 &r, const M3 &a, const M3 &b) {
  M3 o;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      cx<double> s = r.e[i][j];
#pragma unroll
      for (int k = 0; k < 3; ++k) s = cmadd(s, a.e[i][k], b.e[k][j]);
      o.e[i][j] = s;
    }
  return o;
}
// A B
__host__ __device__ __forceinline__ M3 m3_mul(const M3 &a, const M3 &b) { return m3_muladd(m3_zero(), a, b); }
// A^+ B
__host__ __device__ __forceinline__ M3 m3_dmul(const M3 &a, const M3 &b) {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      cx<double> s = mk<double>(0.0, 0.0);
#pragma unroll
      for (int k = 0; k < 3; ++k) s = cjmadd(s, a.e[k][i], b.e[k][j]);
      r.e[i][j] = s;
    }
  return r;
}
// A B^+
__host__ __device__ __forceinline__ M3 m3_muld(const M3 &a, const M3 &b) {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      cx<double> s = mk<double>(0.0, 0.0);
#pragma unroll
      for (int k = 0; k < 3; ++k) s = cjmadd(s, b.e[j][k], a.e[i][k]);
      r.e[i][j] = s;
    }
  return r;
}
__host__ __device__ __forceinline__ M3 m3_dag(const M3 &a) {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) r.e[i][j] = mk<double>(a.e[j][i].re, -a.e[j][i].im);
  return r;
}
// a + s b
__host__ __device__ __forceinline__ M3 m3_axpy(const M3 &a, double s, const M3 &b) {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      r.e[i][j] = mk<double>(fma(s, b.e[i][j].re, a.e[i][j].re), fma(s, b.e[i][j].im, a.e[i][j].im));
  return r;
}
__host__ __device__ __forceinline__ M3 m3_scale(const M3 &a, double s) {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) r.e[i][j] = scale(a.e[i][j], s);
  return r;
}
__host__ __device__ __forceinline__ double m3_frob(const M3 &a) {
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) s += a.e[i][j].re * a.e[i][j].re + a.e[i][j].im * a.e[i][j].im;
  return sqrt(s);
}

// traceless anti-Hermitian part: (W - W^+)/2 - tr(W - W^+)/6
__host__ __device__ __forceinline__ M3 m3_ta(const M3 &w) {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      r.e[i][j] = mk<double>(0.5 * (w.e[i][j].re - w.e[j][i].re), 0.5 * (w.e[i][j].im + w.e[j][i].im));
  const double tr_im = (r.e[0][0].im + r.e[1][1].im + r.e[2][2].im) / 3.0;
#pragma unroll
  for (int i = 0; i < 3; ++i) r.e[i][i].im -= tr_im;
  return r;
}

// ---------------------------------------------------------------------------------------------
// D(A) = exp(A) - 1 and the Frechet derivative L(A, F) = d/dt exp(A + t F) at t = 0 for traceless A.
//   Scale: X = A / 2^s with ||X||_F <= 1/2.  Series: a traceless 3 x 3 matrix obeys (Cayley-Hamilton)
//   X^3 = p X + q, p = tr(X^2) / 2, q = det X, so a polynomial in X is a + b X + c X^2, and a step of
//   Horner's rule, 1 + X (a + b X + c X^2) / k, gives a' = 1 + c q / k, b' = (a + c p) / k, c' = b / k:
//   the series runs on three complex numbers and exp(X) = f0 + f1 X + f2 X^2 takes one matrix product.
//   The derivative along a traceless G changes p by tr(X G) and q by tr(X^2 G):
//     L(X, G) = f1 G + f2 (X G + G X) + df0 + df1 X + df2 X^2,  df = f_p tr(X G) + f_q tr(X^2 G),
//   with the p and q derivatives of a, b, c carried along; a trace of F adds (tr F / 3) exp(X).
//   Double: D(2Y) = 2 D + D D and L(2Y, 2G) = 2 L + L D + D L for D, L at Y.
// 18 terms leave a remainder below 0.5^19 / 19! (1e-23) of the scaled series.  (The same series as
// matrix powers takes 18 products for exp and 54 for the derivative.)
// Precision: Horner's rule adds the smallest terms first, and the ones of exp and of f1 are left out of
// every sum and product (f0 - 1 and f1 - 1 are kept, X and F are added last), so the roundings are
// relative to D and to L - F.  Error against extended precision, relative in the Frobenius norm, for
// random anti-Hermitian matrices of norm 0.3 / 1.7 / 9 and random F, in 1e-16:
//   exp         here 0.34 / 0.87 / 5.1, matrix powers 0.78 / 3.7 / 20, the same three numbers summed
//               forwards with the ones in them 0.84 / 3.9 / 25
//   derivative  here 0.51 / 1.1 / 4.6,  matrix powers 1.6 / 3.1 / 20,  forwards 1.7 / 3.3 / 24
constexpr int kExpTerms = 18;

__host__ __device__ __forceinline__ int exp_scaling(const M3 &a) {
  double n = m3_frob(a);
  int s = 0;
  while (n > 0.5 && s < 40) {
    n *= 0.5;
    ++s;
  }
  return s;
}

using cxd = cx<double>;
__host__ __device__ __forceinline__ cxd cmul(cxd a, cxd b) { return cmadd(mk<double>(0.0, 0.0), a, b); }
// tr(A B)
__host__ __device__ __forceinline__ cxd m3_trmul(const M3 &a, const M3 &b) {
  cxd t = mk<double>(0.0, 0.0);
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int k = 0; k < 3; ++k) t = cmadd(t, a.e[i][k], b.e[k][i]);
  return t;
}
__host__ __device__ __forceinline__ cxd m3_det(const M3 &a) {
  cxd d = mk<double>(0.0, 0.0);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int j = (i + 1) % 3, k = (i + 2) % 3;
    const cxd m = cmadd(cmul(a.e[1][j], a.e[2][k]), -a.e[1][k], a.e[2][j]);
    d = cmadd(d, a.e[0][i], m);
  }
  return d;
}
// r += s A, s complex
__host__ __device__ __forceinline__ void m3_cacc(M3 &r, cxd s, const M3 &a) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) r.e[i][j] = cmadd(r.e[i][j], s, a.e[i][j]);
}

// Horner's rule on a + b X + c X^2 (a without its 1), from the last term to the first
struct ExpSeries {
  cxd p, q, a, b, c;
  __host__ __device__ __forceinline__ ExpSeries(cxd p_, cxd q_) : p(p_), q(q_) {
    a = b = c = mk<double>(0.0, 0.0);
  }
  // 1 + X (1 + a + b X + c X^2) / k without its 1; last (k = 1): b without its 1 too
  __host__ __device__ __forceinline__ void step(double r, bool last) {
    const cxd an = scale(cmul(c, q), r);
    cxd bn = cmadd(a, c, p);
    if (!last) bn = scale(mk<double>(1.0 + bn.re, bn.im), r);
    const cxd cn = scale(b, r);
    a = an;
    b = bn;
    c = cn;
  }
};

// D = exp(M) - 1
__host__ __device__ inline M3 m3_expm1(const M3 &m) {
  const int s = exp_scaling(m);
  const M3 x = m3_scale(m, ldexp(1.0, -s));
  const M3 x2 = m3_mul(x, x);
  ExpSeries f(scale(x2.e[0][0] + x2.e[1][1] + x2.e[2][2], 0.5), m3_det(x));
#pragma unroll
  for (int k = kExpTerms; k >= 1; --k) f.step(1.0 / k, k == 1);
  M3 d = m3_zero();  // f0 - 1 + (f1 - 1) X + f2 X^2, then X
#pragma unroll
  for (int i = 0; i < 3; ++i) d.e[i][i] = f.a;
  m3_cacc(d, f.c, x2);
  m3_cacc(d, f.b, x);
  d = m3_axpy(x, 1.0, d);
  for (int i = 0; i < s; ++i) d = m3_axpy(m3_mul(d, d), 2.0, d);
  return d;
}

// exp(M) - 1 into *d_out and L(M, F) into *l_out
__host__ __device__ inline void m3_expm1_frechet(const M3 &m, const M3 &f, M3 *d_out, M3 *l_out) {
  const int s = exp_scaling(m);
  const double sc = ldexp(1.0, -s);
  const M3 x = m3_scale(m, sc), fs = m3_scale(f, sc);
  const cxd tr = scale(fs.e[0][0] + fs.e[1][1] + fs.e[2][2], 1.0 / 3.0);
  M3 g = fs;
#pragma unroll
  for (int i = 0; i < 3; ++i) g.e[i][i] = g.e[i][i] - tr;
  const M3 x2 = m3_mul(x, x);
  ExpSeries v(scale(x2.e[0][0] + x2.e[1][1] + x2.e[2][2], 0.5), m3_det(x));
  const cxd dp = m3_trmul(x, g), dq = m3_trmul(x2, g);
  cxd ad = mk<double>(0.0, 0.0), bd = ad, cd = ad;  // derivatives of a, b, c along (dp, dq)
#pragma unroll
  for (int k = kExpTerms; k >= 1; --k) {
    const double r = 1.0 / k;
    const cxd an = scale(cmadd(cmul(cd, v.q), v.c, dq), r);
    const cxd bn = scale(cmadd(cmadd(ad, cd, v.p), v.c, dp), r), cn = scale(bd, r);
    ad = an;
    bd = bn;
    cd = cn;
    v.step(r, k == 1);
  }
  M3 d = m3_zero();
#pragma unroll
  for (int i = 0; i < 3; ++i) d.e[i][i] = v.a;
  m3_cacc(d, v.c, x2);
  m3_cacc(d, v.b, x);
  d = m3_axpy(x, 1.0, d);
  M3 l = m3_zero();  // L - F
#pragma unroll
  for (int i = 0; i < 3; ++i) l.e[i][i] = ad;
  m3_cacc(l, cd, x2);
  m3_cacc(l, bd, x);
  m3_cacc(l, v.b, g);
  m3_cacc(l, v.c, m3_muladd(m3_mul(x, g), g, x));
  m3_cacc(l, tr, d);
  l = m3_axpy(fs, 1.0, l);
  for (int i = 0; i < s; ++i) {
    l = m3_axpy(m3_muladd(m3_mul(l, d), d, l), 2.0, l);
    d = m3_axpy(m3_mul(d, d), 2.0, d);
  }
  *d_out = d;
  *l_out = l;
}

}  // namespace ovl
