// Link gradient: the hopping part and the SW term's link dependence.
//
// With x and lambda (dL = -Re <lambda, dM x>) the hopping terms give, per link U_mu(s),
//   K = Y + Z^dag,  Y_ca = sum_a [P-^mu x(s+mu)]_c conj(lambda(s)_a),
//                   Z_ca = sum_a [P+^mu x(s)]_c conj(lambda(s+mu)_a),   raw gradient k b K^dag,
// and the SW term (Sec. II), with the corner fields of plane p
//   Yh_p = (c_p/2)(Z - Z^dag),  Z = W/8 - tr(W)/24,  W_p = sum_{s s'} sigma_p[s][s'] x_s' lambda_s^dag,
// adds from each plaquette that contains the link the product of its other three links with Yh
// inserted at every corner.  Grouped by the sides of the plaquette (Yh^dag = -Yh), with
//   E_nu(P) = Yh(P) U_nu(P) + U_nu(P) Yh(P + nu),
// the plaquettes at x (up) and x - nu (down) add to the gradient of U_mu(x), with sign + for
// mu < nu and - otherwise (the plane's orientation),
//   up:    U_nu(P) U_mu(P+nu) E_nu(P+mu)^dag - E_nu(P) U_mu(P+nu) U_nu(P+mu)^dag,       P = x,
//   down:  U_nu(P)^dag U_mu(P) E_nu(P+mu) - E_nu(P)^dag U_mu(P) U_nu(P+mu),             P = x - nu.
#include "tp_internal.h"
#include "tp_links.h"

namespace {

struct SigmaTab {
  double2 s[6][4][4];  // sigma_{mu nu} = [gamma_mu, gamma_nu]/2, planes (03 13 23 01 02 12)
};

// Corner fields: an anti-hermitian traceless matrix per plane and site as nine real planes (the
// imaginary diagonal, then the entries (1,0), (2,0), (2,1)), two lattice planes per buffer, in
// p4 order [plane][2 parity][9][V2].
struct CornerF {
  double* p[3];
  TP_DEV double* at(const Geom& g, int pl, int par) const {
    double* b = pl < 2 ? p[0] : (pl < 4 ? p[1] : p[2]);
    return b + (int64_t)((pl & 1) * 2 + par) * 9 * g.V2;
  }
};

TP_DEV int plane_index(int a, int b) {  // a < b
  return b == 3 ? a : (a == 0 ? (b == 1 ? 3 : 4) : 5);
}

// Canonical x and lambda into p4 planes, and the corner fields of every site.  One thread per
// site: bound by the bytes it streams (384 read, 384 written, 432 for the corner fields).
template <bool CLOV>
__global__ void __launch_bounds__(64) k_force_fields(const double2* __restrict__ xc, const double2* __restrict__ lc,
                                                     SpinorF<double2> x0, SpinorF<double2> x1,
                                                     SpinorF<double2> l0, SpinorF<double2> l1, CornerF Y, Geom g,
                                                     SigmaTab sig, double c_s, double c_t) {
  const SubSite q = sub_site(g, threadIdx.x);
  if (!q.ok) return;
  const C3 c = p3_coords(g, q.p, q.s);
  const int64_t n = c.x + (int64_t)g.Lx * (c.y + (int64_t)g.Ly * (c.z + (int64_t)g.Lz * q.t));
  const int par = q.p ^ (q.t & 1);
  const int64_t i = q.s + (int64_t)g.Vs2 * q.t;
  cx<double> xs[12], ls[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    const double2 a = xc[n * 12 + k], b = lc[n * 12 + k];
    xs[k] = cx<double>{a.x, a.y};
    ls[k] = cx<double>{b.x, b.y};
  }
  const SpinorF<double2> xo = par ? x1 : x0, lo = par ? l1 : l0;
  store_half<double2>(xo, 0, i, xs);
  store_half<double2>(xo, 1, i, xs + 6);
  store_half<double2>(lo, 0, i, ls);
  store_half<double2>(lo, 1, i, ls + 6);
  if constexpr (!CLOV) return;
  // W_ba = sum_s v_sb conj(lambda_sa) with v_sb = sum_s' sigma_ss' x_s'b; every loop is
  // unrolled so that the spinor components and the table are read at constant indices (arrays
  // indexed by a loop variable would live in scratch memory)
#pragma unroll
  for (int pl = 0; pl < 6; ++pl) {
    cx<double> W[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) W[k] = czero<double>();
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      cx<double> v[3] = {czero<double>(), czero<double>(), czero<double>()};
#pragma unroll
      for (int sp = 0; sp < 4; ++sp) {
        const cx<double> sg = cx<double>{sig.s[pl][s][sp].x, sig.s[pl][s][sp].y};
#pragma unroll
        for (int b = 0; b < 3; ++b) v[b] += cmul(sg, xs[3 * sp + b]);
      }
#pragma unroll
      for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int a = 0; a < 3; ++a) W[3 * b + a] += cmul(v[b], conj(ls[3 * s + a]));
    }
    const double cc = 0.5 * (pl < 3 ? c_t : c_s);
    const cx<double> tr = (1.0 / 3.0) * (W[0] + W[4] + W[8]);
    double* o = Y.at(g, pl, par) + i;
    // (cc/8)(W - W^dag) without its trace: 2i Im on the diagonal
#pragma unroll
    for (int r = 0; r < 3; ++r) o[(int64_t)r * g.V2] = (cc / 4.0) * (W[4 * r].im - tr.im);
    const int lr[3] = {1, 2, 2}, lq[3] = {0, 0, 1};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const cx<double> v = (cc / 8.0) * (W[3 * lr[k] + lq[k]] - conj(W[3 * lq[k] + lr[k]]));
      o[(int64_t)(3 + 2 * k) * g.V2] = v.re;
      o[(int64_t)(4 + 2 * k) * g.V2] = v.im;
    }
  }
}

// A lattice point: coordinates (wrapped), p4 parity and index.
struct Pt {
  int x, y, z, t, par;
  int64_t i;
};
TP_DEV Pt point(const Geom& g, int x, int y, int z, int t) {
  Pt q;
  q.x = x < 0 ? x + g.Lx : (x >= g.Lx ? x - g.Lx : x);
  q.y = y < 0 ? y + g.Ly : (y >= g.Ly ? y - g.Ly : y);
  q.z = z < 0 ? z + g.Lz : (z >= g.Lz ? z - g.Lz : z);
  q.t = t < 0 ? t + g.Lt : (t >= g.Lt ? t - g.Lt : t);
  q.par = (q.x + q.y + q.z + q.t) & 1;
  q.i = p3_index(g, q.x, q.y, q.z) + (int64_t)g.Vs2 * q.t;
  return q;
}
TP_DEV Pt step(const Geom& g, const Pt& q, int mu, int d) {
  return point(g, q.x + (mu == 0 ? d : 0), q.y + (mu == 1 ? d : 0), q.z + (mu == 2 ? d : 0), q.t + (mu == 3 ? d : 0));
}

TP_DEV void ld_link(const double2* __restrict__ u4, const Geom& g, int mu, const Pt& q, cx<double>* m) {
  const double2* src = u4 + (int64_t)(mu * 2 + q.par) * 9 * g.V2 + q.i;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const double2 e = src[(int64_t)k * g.V2];
    m[k] = cx<double>{e.x, e.y};
  }
}
TP_DEV void ld_corner(const CornerF& Y, const Geom& g, int pl, const Pt& q, cx<double>* m) {
  const double* src = Y.at(g, pl, q.par) + q.i;
  double v[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) v[k] = src[(int64_t)k * g.V2];
#pragma unroll
  for (int r = 0; r < 3; ++r) m[4 * r] = cx<double>{0.0, v[r]};
  m[3] = cx<double>{v[3], v[4]};
  m[6] = cx<double>{v[5], v[6]};
  m[7] = cx<double>{v[7], v[8]};
  m[1] = cx<double>{-v[3], v[4]};
  m[2] = cx<double>{-v[5], v[6]};
  m[5] = cx<double>{-v[7], v[8]};
}

// acc += a b and acc += conj(a) b, each in four multiply-adds: the FP64 products are what bounds
// k_force, and a complex product formed first costs six instructions.
TP_DEV void cmac(cx<double>& acc, cx<double> a, cx<double> b) {
  acc.re = fma(-a.im, b.im, fma(a.re, b.re, acc.re));
  acc.im = fma(a.im, b.re, fma(a.re, b.im, acc.im));
}
TP_DEV void cmacc(cx<double>& acc, cx<double> a, cx<double> b) {
  acc.re = fma(a.im, b.im, fma(a.re, b.re, acc.re));
  acc.im = fma(-a.im, b.re, fma(a.re, b.im, acc.im));
}
// acc += a b (DA: a^dag, DB: b^dag)
template <bool DA, bool DB>
TP_DEV void mma(const cx<double>* a, const cx<double>* b, cx<double>* acc) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const cx<double> x = a[DA ? 3 * k + i : 3 * i + k], y = b[DB ? 3 * j + k : 3 * k + j];
        if constexpr (DA && DB) cmac(acc[3 * i + j], conj(x), conj(y));
        else if constexpr (DA) cmacc(acc[3 * i + j], x, y);
        else if constexpr (DB) cmacc(acc[3 * i + j], y, x);
        else cmac(acc[3 * i + j], x, y);
      }
}
template <bool DA, bool DB>
TP_DEV void mul(const cx<double>* a, const cx<double>* b, cx<double>* c) {
#pragma unroll
  for (int k = 0; k < 9; ++k) c[k] = czero<double>();
  mma<DA, DB>(a, b, c);
}

// E_nu(P) for the links u = U_nu(P)
TP_DEV void side(const CornerF& Y, const Geom& g, int pl, int nu, const Pt& q, const cx<double>* u, cx<double>* E) {
  cx<double> m[9];
  ld_corner(Y, g, pl, q, m);
  mul<false, false>(m, u, E);
  ld_corner(Y, g, pl, step(g, q, nu, 1), m);
  mma<false, false>(u, m, E);
}

// Projected half spinors of a hop in direction MU: (1 -+ gamma_MU) psi, two spins (time: the
// kept spins, times sqrt(2) folded into the caller's factor).
template <int MU, bool MINUS>
TP_DEV void half_of(const SpinorF<double2>& f, int64_t i, cx<double>* h) {
  if constexpr (MU == 3) {
    load_half<double2>(f, MINUS ? 1 : 0, i, h);
  } else {
    cx<double> psi[12];
    load_half<double2>(f, 0, i, psi);
    load_half<double2>(f, 1, i, psi + 6);
    if constexpr (MINUS) proj_minus<MU, double>(psi, h);
    else proj_plus<MU, double>(psi, h);
  }
}
// G += f (K_part)^dag for the product of half spinors: K_ca = sum_s hx[s c] conj(hl[s a]), or its
// dagger when DAG.
template <bool DAG>
TP_DEV void add_outer(const cx<double>* hx, const cx<double>* hl, double f, cx<double>* G) {
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      cx<double> k = cmulc(hl[a], hx[c]);
      k += cmulc(hl[3 + a], hx[3 + c]);
      if constexpr (DAG) G[3 * c + a] += f * k;          // ((Z^dag)^dag)_ca = Z_ca
      else G[3 * a + c] += f * conj(k);                  // (Y^dag)_ac = conj(Y_ca)
    }
}
template <int MU>
TP_DEV void hop_part(const SpinorF<double2>* x, const SpinorF<double2>* l, const Pt& q, const Pt& n, double f,
                     cx<double>* G) {
  // <lambda, P x> over four spins is the product of the two projected half spinors, over two
  // (space: P = P^2 and each half spinor carries a factor 2, so 1/2; time: P keeps two spins)
  const double w = MU == 3 ? f : 0.5 * f;
  cx<double> hx[6], hl[6];
  half_of<MU, true>(n.par ? x[1] : x[0], n.i, hx);
  half_of<MU, true>(q.par ? l[1] : l[0], q.i, hl);
  add_outer<false>(hx, hl, w, G);
  half_of<MU, false>(q.par ? x[1] : x[0], q.i, hx);
  half_of<MU, false>(n.par ? l[1] : l[0], n.i, hl);
  add_outer<true>(hx, hl, w, G);
}

struct ForceArgs {
  SpinorF<double2> x[2], l[2];
  CornerF Y;
  const double2* u4;
  double2* grad;
  Geom g;
  int64_t V;
  double inv_gf, b;
  int projected;
};

// The gradient of every link: a workgroup handles 64 sites, wavefront mu the links of direction
// mu.  Bound by the latency of what it reads around each link (six plaquettes of three links and
// four corner fields, from L2) at two wavefronts per SIMD, and by its FP64 products (8 per
// plaquette): everything comes from planes whose adjacent lanes are adjacent, in sub-blocks whose
// neighbours share an L2 (1.9 GB fetched per launch at 16^3x128), and E is formed twice per
// plaquette rather than stored (12 per site, 1.7 KB).  Each plaquette is summed before it joins G, and
// the hopping part comes last: with all products accumulated in G, which starts from the hopping
// part, the rounding error is 4.2e-16 instead of 2.4e-16 of the norm (16^3x128), for 27 us less.  At
// 16^3x128 a whole gradient takes 1.15 ms; it took 1.84 ms with canonical links and corner fields
// (one cache line per lane and load), nine products per plaquette and the hopping part in a pass of
// its own.
template <bool CLOV>
__global__ void __launch_bounds__(256) k_force(ForceArgs a) {
  const Geom& g = a.g;
  const int lane = threadIdx.x & 63, mu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const SubSite ss = sub_site(g, lane);
  if (!ss.ok) return;
  const C3 c0 = p3_coords(g, ss.p, ss.s);
  const Pt q = point(g, c0.x, c0.y, c0.z, ss.t);
  const double wrap = (mu == 3 && q.t == g.Lt - 1) ? a.b : 1.0;
  cx<double> G[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) G[k] = czero<double>();
  if constexpr (CLOV) {
#pragma unroll 1
    for (int k = 0; k < 6; ++k) {
      const int nu = (mu + 1 + (k >> 1)) & 3;
      const bool down = k & 1;
      const int pl = mu < nu ? plane_index(mu, nu) : plane_index(nu, mu);
      const double sg = mu < nu ? wrap : -wrap;  // the stored time links of the last slice carry b
      const Pt P = down ? step(g, q, nu, -1) : q;
      const Pt Pm = step(g, P, mu, 1);
      cx<double> T1[9], T2[9];
      {
        cx<double> B[9], M[9], E1[9];
        ld_link(a.u4, g, nu, Pm, B);
        ld_link(a.u4, g, mu, down ? P : step(g, P, nu, 1), M);
#pragma unroll
        for (int r = 0; r < 9; ++r) M[r] = sg * M[r];
        if (down) mul<false, false>(M, B, T2);
        else mul<false, true>(M, B, T2);
        side(a.Y, g, pl, nu, Pm, B, E1);
        if (down) mul<false, false>(M, E1, T1);
        else mul<false, true>(M, E1, T1);
      }
      cx<double> A[9], E0[9], S[9];
      ld_link(a.u4, g, nu, P, A);
      if (down) mul<true, false>(A, T1, S);
      else mul<false, false>(A, T1, S);
      side(a.Y, g, pl, nu, P, A, E0);
#pragma unroll
      for (int r = 0; r < 9; ++r) T2[r] = -T2[r];
      if (down) mma<true, false>(E0, T2, S);
      else mma<false, false>(E0, T2, S);
#pragma unroll
      for (int r = 0; r < 9; ++r) G[r] += S[r];
    }
  }
  {
    const Pt n = step(g, q, mu, 1);
    const double f = (mu == 3 ? 1.0 : a.inv_gf) * wrap;
    cx<double> H[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) H[k] = czero<double>();
    switch (mu) {
      case 0: hop_part<0>(a.x, a.l, q, n, f, H); break;
      case 1: hop_part<1>(a.x, a.l, q, n, f, H); break;
      case 2: hop_part<2>(a.x, a.l, q, n, f, H); break;
      default: hop_part<3>(a.x, a.l, q, n, f, H); break;
    }
#pragma unroll
    for (int k = 0; k < 9; ++k) G[k] += H[k];
  }
  const int64_t n = q.x + (int64_t)g.Lx * (q.y + (int64_t)g.Ly * (q.z + (int64_t)g.Lz * q.t));
  double2* out = a.grad + ((int64_t)mu * a.V + n) * 9;
  if (!a.projected) {
#pragma unroll
    for (int k = 0; k < 9; ++k) out[k] = make_double2(G[k].re, G[k].im);
    return;
  }
  // su(3) projection TH[i U G^dag]
  cx<double> U[9], M[9];
  ld_link(a.u4, g, mu, q, U);
  mul<false, true>(U, G, M);
#pragma unroll
  for (int k = 0; k < 9; ++k) M[k] = wrap * ti(M[k]);
  const double tr = (M[0].re + M[4].re + M[8].re) / 3.0;
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      cx<double> h = 0.5 * (M[3 * r + k] + conj(M[3 * k + r]));
      if (r == k) h.re -= tr;
      out[3 * r + k] = make_double2(h.re, h.im);
    }
}

}  // namespace

void launch_force(tp_op op, const double2* x, const double2* lam, double2* grad, bool projected, bool clover,
                  const double sig[6][4][4][2]) {
  tp_ctx ctx = op->g->ctx;
  const Lattice& L = ctx->lat;
  ForceArgs a{};
  Field& xf = ws_get_n(op, TP_F64, W_TMP, 1);
  Field& lf = ws_get_n(op, TP_F64, W_TMP + 1, 1);
  for (int p = 0; p < 2; ++p) {
    a.x[p] = xf.par<double2>(p);
    a.l[p] = lf.par<double2>(p);
  }
  SigmaTab t{};
  if (clover) {
    // two planes of corner fields (36 V/2 doubles) per work field (48 V/2)
    const int slots[3] = {W_ETA, W_SOL, W_R64};
    for (int k = 0; k < 3; ++k) a.Y.p[k] = static_cast<double*>(ws_get_n(op, TP_F64, slots[k], 1).data);
    for (int p = 0; p < 6; ++p)
      for (int r = 0; r < 4; ++r)
        for (int q = 0; q < 4; ++q) t.s[p][r][q] = make_double2(sig[p][r][q][0], sig[p][r][q][1]);
  }
  a.u4 = op->g->u4_d;
  a.grad = grad;
  a.g = L.g;
  a.V = L.V;
  a.inv_gf = 1.0 / op->gf;
  a.b = double(ctx->bc);
  a.projected = projected ? 1 : 0;
  ProfScope ps(ctx, KID_FORCE, double(L.V) * (2 * 192 * 2 + 576 * (clover || projected ? 2 : 1) + (clover ? 2 * 432 : 0)));
  const dim3 grid(sub_blocks(L));
  if (clover) {
    hipLaunchKernelGGL(k_force_fields<true>, grid, dim3(64), 0, ctx->stream, x, lam, a.x[0], a.x[1], a.l[0], a.l[1],
                       a.Y, L.g, t, op->c->cs, op->c->ct);
    LAUNCH_CHECK();
    hipLaunchKernelGGL(k_force<true>, grid, dim3(256), 0, ctx->stream, a);
  } else {
    hipLaunchKernelGGL(k_force_fields<false>, grid, dim3(64), 0, ctx->stream, x, lam, a.x[0], a.x[1], a.l[0], a.l[1],
                       a.Y, L.g, t, 0.0, 0.0);
    LAUNCH_CHECK();
    hipLaunchKernelGGL(k_force<false>, grid, dim3(256), 0, ctx->stream, a);
  }
  LAUNCH_CHECK();
}
