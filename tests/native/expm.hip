// Precision of exp and its Frechet derivative (csrc/m3.hpp) on the CPU: against extended precision they are
// no further off than the sum of matrix powers in double, for random traceless anti-Hermitian matrices from
// small norms to ones that take several doublings.
#include <cmath>
#include <cstdio>
#include <random>

#include "../../paper_1510_06897_amd/csrc/m3.hpp"

using namespace ovl;

template <class T>
struct Mat {
  T re[3][3], im[3][3];
};
template <class T>
static Mat<T> zero() {
  Mat<T> r{};
  return r;
}
template <class T>
static Mat<T> unit() {
  Mat<T> r{};
  for (int i = 0; i < 3; ++i) r.re[i][i] = 1;
  return r;
}
static double madd(double a, double b, double c) { return std::fma(a, b, c); }  // as on the device
static long double madd(long double a, long double b, long double c) { return a * b + c; }
template <class T>
static Mat<T> mul(const Mat<T> &a, const Mat<T> &b) {
  Mat<T> r{};
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) {
      T x = 0, y = 0;
      for (int k = 0; k < 3; ++k) {
        x = madd(a.re[i][k], b.re[k][j], x);
        x = madd(-a.im[i][k], b.im[k][j], x);
        y = madd(a.re[i][k], b.im[k][j], y);
        y = madd(a.im[i][k], b.re[k][j], y);
      }
      r.re[i][j] = x;
      r.im[i][j] = y;
    }
  return r;
}
template <class T>
static Mat<T> axpy(const Mat<T> &a, T s, const Mat<T> &b) {
  Mat<T> r;
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) {
      r.re[i][j] = madd(s, b.re[i][j], a.re[i][j]);
      r.im[i][j] = madd(s, b.im[i][j], a.im[i][j]);
    }
  return r;
}
template <class T>
static Mat<T> times(const Mat<T> &a, T s) {
  return axpy(zero<T>(), s, a);
}
template <class T>
static T norm(const Mat<T> &a) {
  T s = 0;
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) s += a.re[i][j] * a.re[i][j] + a.im[i][j] * a.im[i][j];
  return std::sqrt(s);
}
// exp and derivative as sums of matrix powers, scaled to norm 1/2 (`terms` of them) and squared
template <class T>
static void powers(const Mat<T> &a, const Mat<T> &f, int terms, Mat<T> &e, Mat<T> &l) {
  int s = 0;
  for (T n = norm(a); n > T(0.5) && s < 40; n /= 2) ++s;
  const Mat<T> x = times(a, std::ldexp(T(1), -s)), g = times(f, std::ldexp(T(1), -s));
  Mat<T> t = unit<T>(), d = zero<T>();
  e = unit<T>();
  l = zero<T>();
  for (int k = 1; k <= terms; ++k) {
    const Mat<T> dn = times(axpy(mul(g, t), T(1), mul(x, d)), T(1) / k);
    t = times(mul(x, t), T(1) / k);
    d = dn;
    e = axpy(e, T(1), t);
    l = axpy(l, T(1), d);
  }
  for (int i = 0; i < s; ++i) {
    l = axpy(mul(l, e), T(1), mul(e, l));
    e = mul(e, e);
  }
}
template <class A, class B>
static Mat<B> cast(const Mat<A> &a) {
  Mat<B> r;
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) r.re[i][j] = (B)a.re[i][j], r.im[i][j] = (B)a.im[i][j];
  return r;
}
static Mat<double> from(const M3 &m) {
  Mat<double> r;
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) r.re[i][j] = m.e[i][j].re, r.im[i][j] = m.e[i][j].im;
  return r;
}
static double off(const Mat<double> &a, const Mat<long double> &b) {
  return (double)(norm(axpy(cast<double, long double>(a), -1.0L, b)) / norm(b));
}

int main() {
  using LD = long double;
  std::mt19937_64 rng(12);
  std::normal_distribution<double> gauss;
  int worse = 0;
  std::printf("norm      exp(here powers) U'(here powers) derivative(here powers), rms of 1e-16\n");
  for (double size : {1e-3, 0.05, 0.3, 0.49, 0.51, 0.9, 1.7, 3.0, 9.0, 40.0}) {
    const int n = 2000;
    double sum[6] = {};
    for (int it = 0; it < n; ++it) {
      M3 h, f, u;
      for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
          h.e[i][j] = mk<double>(gauss(rng), gauss(rng));
          f.e[i][j] = mk<double>(gauss(rng), gauss(rng));
          u.e[i][j] = mk<double>(gauss(rng), gauss(rng));
        }
      M3 m = m3_ta(h);
      m = m3_scale(m, size / m3_frob(m));
      Mat<LD> e, l;
      powers<LD>(cast<double, LD>(from(m)), cast<double, LD>(from(f)), 24, e, l);
      Mat<double> pe, pl;
      powers<double>(from(m), from(f), kExpTerms, pe, pl);
      const M3 d1 = m3_expm1(m);
      M3 d2, l2;
      m3_expm1_frechet(m, f, &d2, &l2);
      const Mat<double> e1 = axpy(unit<double>(), 1.0, from(d1)), e2 = axpy(unit<double>(), 1.0, from(d2));
      const Mat<LD> ue = mul(e, cast<double, LD>(from(u)));
      auto add = [&](int k, double v) { sum[k] += v * v; };
      add(0, std::fmax(off(e1, e), off(e2, e)));
      add(1, off(pe, e));
      add(2, off(from(m3_axpy(u, 1.0, m3_mul(d1, u))), ue));  // what a smearing step stores
      add(3, off(mul(pe, from(u)), ue));
      add(4, off(from(l2), l));
      add(5, off(pl, l));
    }
    std::printf("%-9g", size);
    for (int k = 0; k < 6; k += 2) {
      const double here = std::sqrt(sum[k] / n), there = std::sqrt(sum[k + 1] / n);
      std::printf("   %6.2f %6.2f", 1e16 * here, 1e16 * there);
      worse += here > there;
    }
    std::printf("\n");
  }
  std::printf("%d worse than the powers\n", worse);
  return worse != 0;
}
