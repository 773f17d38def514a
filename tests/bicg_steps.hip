// Host program over the solver's scalar steps (tp_bicg.h): an ordinary iteration against the formulas
// in std::complex<double>, and inner products that end one.
#include <stdio.h>

#include <complex>
#include <limits>

#include "tp_bicg.h"

typedef std::complex<double> zc;
static int failed = 0;
static void check(bool ok, const char* what) {
  if (!ok) {
    printf("FAILED: %s\n", what);
    failed = 1;
  }
}
static bool near(zc a, zc b) { return std::abs(a - b) <= 1e-14 * std::abs(b); }

// The scalar steps of one iteration from its inner products.
struct It {
  double st[BS_COUNT] = {};
  It(bool rounded, zc rho, zc rv, zc ts, double tt, zc rs, zc rt) {
    st[BS_RHO] = rho.real();
    st[BS_RHO + 1] = rho.imag();
    st[BS_BREAK] = BRK_OMEGA;  // of an earlier solve
    const double a[2] = {rv.real(), rv.imag()};
    bicg_post(rounded ? BP_ALPHA_ROUNDED : BP_ALPHA, a, st);
    const double b[7] = {ts.real(), ts.imag(), tt, rs.real(), rs.imag(), rt.real(), rt.imag()};
    bicg_post(rounded ? BP_OMEGA_ROUNDED : BP_OMEGA, b, st);
  }
  zc at(int k) const { return zc(st[k], st[k + 1]); }
  bool ended(double why) const { return st[BS_BREAK] == why && st[BS_FUSED + 6] != 0.0 && st[BS_AXPY + 6] == 0.0; }
};

int main() {
  const double inf = std::numeric_limits<double>::infinity(), nan = std::numeric_limits<double>::quiet_NaN();
  const zc rho(0.7, -0.2), rv(0.4, 0.3), ts(0.5, -0.1), rs(0.2, 0.2), rt(-0.3, 0.6);
  const double tt = 0.8;
  for (int rounded = 0; rounded < 2; ++rounded) {
    const It n(rounded, rho, rv, ts, tt, rs, rt);
    const zc al = rho / rv, om = ts / tt, rn = rs - om * rt, be = rn / rho * al / om;
    check(n.st[BS_BREAK] == BRK_NONE && n.st[BS_FUSED + 6] == 0.0, "ordinary iteration ended");
    check(near(n.at(BS_RHO), rn) && near(n.at(BS_ALPHA), al) && near(n.at(BS_AXPY), -al), "rho, alpha");
    check(near(n.at(BS_FUSED), al) && near(n.at(BS_FUSED + 2), om) && near(n.at(BS_FUSED + 4), be), "update");
    // <rhat, v> vanishes, leaves the range in its square, is infinite or NaN, whatever follows
    for (zc d : {zc(0, 0), zc(1e-170, 0), zc(1e170, 1e170), zc(inf, 0), zc(nan, nan)})
      for (double t2 : {tt, 0.0, nan}) {
        const It b(rounded, rho, d, ts, t2, rs, rt);
        check(b.ended(BRK_ALPHA), "<rhat, v>");
      }
    // no usable omega: the half step is alpha's
    const struct { zc rho, ts; double tt; } cases[] = {{rho, ts, 0.0}, {rho, zc(0, 0), tt}, {rho, zc(inf, 0), inf},
                                                       {rho, zc(nan, nan), nan}, {rho, ts, inf}, {zc(0, 0), ts, tt}};
    for (const auto& q : cases) {
      const It b(rounded, q.rho, rv, q.ts, q.tt, rs, rt);
      check(b.ended(BRK_OMEGA), "omega");
      check(b.at(BS_ALPHA) == b.at(BS_FUSED) && std::abs(b.at(BS_ALPHA) - q.rho / rv) <= 1e-14, "alpha of the half step");
    }
  }
  if (!failed) printf("bicg steps ok\n");
  return failed;
}
