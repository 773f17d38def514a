// Host program over the solver's scalar steps and element updates (tp_bicg.h): an ordinary
// iteration against the textbook formulas in std::complex<double>, and iterations that break down.
#include <stdio.h>

#include <complex>
#include <limits>

#include "tp_bicg.h"

typedef std::complex<double> zc;
static zc z(cx<double> a) { return zc(a.re, a.im); }
static cx<double> c(zc a) { return cx<double>{a.real(), a.imag()}; }
static int failed = 0;
static void check(bool ok, const char* what) {
  if (!ok) {
    printf("FAILED: %s\n", what);
    failed = 1;
  }
}
static bool finite(cx<double> a) { return std::isfinite(a.re) && std::isfinite(a.im); }
static bool near(zc a, zc b) { return std::abs(a - b) <= 1e-14 * std::abs(b); }

// One iteration's second half: the scalars from <rhat,v> and the four inner products, then the updates.
struct It {
  double st[BS_COUNT] = {};
  cx<double> x[2], p[2], r[2], v[2], s[2], t[2];
  It() {
    st[BS_RHO] = 0.7;
    st[BS_RHO + 1] = -0.2;
    for (int k = 0; k < 2; ++k) {
      x[k] = {1.0 + k, 0.5};
      p[k] = {0.3, 0.2 - k};
      r[k] = {-0.4, 0.6 + k};
      v[k] = {0.9 - k, 0.1};
      t[k] = {0.2, -0.3 * k};
    }
  }
  void run(bool rounded, zc rv, zc ts, double tt, zc rs, zc rt) {
    const double a[2] = {rv.real(), rv.imag()};
    bicg_post(rounded ? BP_ALPHA_ROUNDED : BP_ALPHA, a, st);
    for (int k = 0; k < 2; ++k) s[k] = r[k];
    bicg_half<2>(cx<double>{st[BS_AXPY], st[BS_AXPY + 1]}, v, s);
    const double b[7] = {ts.real(), ts.imag(), tt, rs.real(), rs.imag(), rt.real(), rt.imag()};
    bicg_post(rounded ? BP_OMEGA_ROUNDED : BP_OMEGA, b, st);
    const double* f = st + BS_FUSED;
    for (int k = 0; k < 2; ++k) r[k] = s[k];
    bicg_full<2>(cx<double>{f[0], f[1]}, cx<double>{f[2], f[3]}, cx<double>{f[4], f[5]}, x, p, r, t, v);
  }
};

int main() {
  const double inf = std::numeric_limits<double>::infinity(), nan = std::numeric_limits<double>::quiet_NaN();
  const zc rv(0.4, 0.3), ts(0.5, -0.1), rs(0.2, 0.2), rt(-0.3, 0.6);
  const double tt = 0.8;
  for (int rounded = 0; rounded < 2; ++rounded) {
    {
      It o, n;
      n.run(rounded, rv, ts, tt, rs, rt);
      const zc rho(0.7, -0.2), al = rho / rv, om = ts / tt, rn = rs - om * rt, be = rn / rho * al / om;
      check(n.st[BS_BREAK] == 0.0, "ordinary iteration flagged");
      check(near(zc(n.st[BS_RHO], n.st[BS_RHO + 1]), rn), "rho");
      for (int k = 0; k < 2; ++k) {
        const zc s = z(o.r[k]) - al * z(o.v[k]), r = s - om * z(o.t[k]);
        check(near(z(n.x[k]), z(o.x[k]) + al * z(o.p[k]) + om * s), "x");
        check(near(z(n.r[k]), r), "r");
        check(near(z(n.p[k]), r + be * (z(o.p[k]) - om * z(o.v[k]))), "p");
      }
    }
    // <rhat, v> vanishes, overflows in its square, is infinite or NaN; v finite or not: x and r stay
    for (zc d : {zc(0, 0), zc(1e-170, 0), zc(1e170, 1e170), zc(inf, 0), zc(nan, nan)})
      for (double vv : {0.9, inf, nan}) {
        It o, n;
        n.v[1].im = vv;
        n.run(rounded, d, ts, tt, rs, rt);
        check(n.st[BS_BREAK] != 0.0, "breakdown of alpha not flagged");
        for (int k = 0; k < 2; ++k) {
          check(z(n.x[k]) == z(o.x[k]), "x moved without alpha");
          check(z(n.r[k]) == z(o.r[k]), "r moved without alpha");
        }
      }
    // no usable omega: the half step, also where t is not finite
    struct { zc ts; double tt, t; } cases[] = {{ts, 0.0, 0.2}, {zc(0, 0), tt, 0.2}, {zc(inf, 0), inf, inf},
                                               {zc(nan, nan), nan, nan}, {ts, inf, inf}};
    for (auto& q : cases) {
      It o, n;
      n.t[0].re = q.t;
      n.run(rounded, rv, q.ts, q.tt, rs, zc(q.t, q.t));
      check(n.st[BS_BREAK] != 0.0, "breakdown of omega not flagged");
      const zc al = zc(0.7, -0.2) / rv;
      for (int k = 0; k < 2; ++k) {
        check(finite(n.x[k]) && near(z(n.x[k]), z(o.x[k]) + al * z(o.p[k])), "x of the half step");
        check(finite(n.r[k]) && near(z(n.r[k]), z(o.r[k]) - al * z(o.v[k])), "r of the half step");
      }
    }
    // s not finite either: x keeps the half step
    {
      It o, n;
      n.v[0].re = inf;
      n.run(rounded, rv, zc(nan, 0), nan, zc(inf, 0), zc(nan, 0));
      for (int k = 0; k < 2; ++k) check(finite(n.x[k]), "x where s is not finite");
    }
  }
  if (!failed) printf("bicg steps ok\n");
  return failed;
}
