// BiCGStab's scalar steps on the device (single right-hand side), from the reduced values v of the op
// just finished.  An iteration runs to its end whatever they find; one that breaks down is flagged
// (BS_BREAK) and skips its update of x, r and p, so that the host can end it from what they were.
#pragma once
#include "tp_internal.h"

// alpha = rho / <rhat, v>, unless <rhat, v> vanishes or is not finite (BRK_ALPHA).
#define TP_BICG_ALPHA                                                                          \
  const double den = v[0] * v[0] + v[1] * v[1];                                                \
  const bool bad = den == 0.0 || !__builtin_isfinite(den);                                     \
  const double rr = st[BS_RHO], ri = st[BS_RHO + 1];                                           \
  const double ar = bad ? 0.0 : (rr * v[0] + ri * v[1]) / den;                                 \
  const double ai = bad ? 0.0 : (ri * v[0] - rr * v[1]) / den;                                 \
  st[BS_BREAK] = bad ? BRK_ALPHA : BRK_NONE;                                                   \
  st[BS_ALPHA] = ar;                                                                           \
  st[BS_ALPHA + 1] = ai;                                                                       \
  st[BS_AXPY] = -ar;                                                                           \
  st[BS_AXPY + 1] = -ai;                                                                       \
  for (int q = 2; q < 7; ++q) st[BS_AXPY + q] = 0.0;
// v = <t, s>, |t|^2, <rhat, s>, <rhat, t>: omega = <t, s> / |t|^2, rho_new = <rhat, s - omega t>,
// beta = (rho_new / rho) (alpha / omega), unless there is no usable omega (BRK_OMEGA).
#define TP_BICG_OMEGA                                                                          \
  const double om_r = v[0] / v[2], om_i = v[1] / v[2];                                         \
  const double rn_r = v[3] - (om_r * v[5] - om_i * v[6]);                                      \
  const double rn_i = v[4] - (om_r * v[6] + om_i * v[5]);                                      \
  const double rho_r = st[BS_RHO], rho_i = st[BS_RHO + 1];                                     \
  const double al_r = st[BS_ALPHA], al_i = st[BS_ALPHA + 1];                                   \
  const double rr = rho_r * rho_r + rho_i * rho_i, oo = om_r * om_r + om_i * om_i;             \
  const double q_r = (rn_r * rho_r + rn_i * rho_i) / rr, q_i = (rn_i * rho_r - rn_r * rho_i) / rr; \
  const double w_r = (al_r * om_r + al_i * om_i) / oo, w_i = (al_i * om_r - al_r * om_i) / oo; \
  const double be_r = q_r * w_r - q_i * w_i, be_i = q_r * w_i + q_i * w_r;                     \
  const bool bad = v[2] == 0.0 || !__builtin_isfinite(oo) || oo == 0.0 || rr == 0.0;           \
  if (bad && st[BS_BREAK] == BRK_NONE) st[BS_BREAK] = BRK_OMEGA;                               \
  st[BS_FUSED] = al_r;                                                                         \
  st[BS_FUSED + 1] = al_i;                                                                     \
  st[BS_FUSED + 2] = om_r;                                                                     \
  st[BS_FUSED + 3] = om_i;                                                                     \
  st[BS_FUSED + 4] = be_r;                                                                     \
  st[BS_FUSED + 5] = be_i;                                                                     \
  st[BS_FUSED + 6] = st[BS_BREAK];                                                             \
  st[BS_RHO] = rn_r;                                                                           \
  st[BS_RHO + 1] = rn_i;

// The FP64 solver's scalars round every product, as the host arithmetic that formed them before
// did (its iterates stay what they were bit for bit); the mixed solver's may fuse.
TP_HD void bicg_alpha_rounded(const double* v, double* st) {
#pragma clang fp contract(off)
  TP_BICG_ALPHA
}
TP_HD void bicg_omega_rounded(const double* v, double* st) {
#pragma clang fp contract(off)
  TP_BICG_OMEGA
}
TP_HD void bicg_post(int post, const double* v, double* st) {
  if (post == BP_RHO) {
    st[BS_RHO] = v[0];
    st[BS_RHO + 1] = v[1];
  } else if (post == BP_ALPHA) {
    TP_BICG_ALPHA
  } else if (post == BP_ALPHA_ROUNDED) {
    bicg_alpha_rounded(v, st);
  } else if (post == BP_S2) {
    st[BS_S2] = v[0];
  } else if (post == BP_OMEGA) {
    TP_BICG_OMEGA
  } else if (post == BP_OMEGA_ROUNDED) {
    bicg_omega_rounded(v, st);
  } else if (post == BP_R2) {
    st[BS_R2] = v[0];
  }
}
#undef TP_BICG_ALPHA
#undef TP_BICG_OMEGA
