// One-off and layout kernels: canonical <-> internal spinor layouts, link
// packing, the per-time-line products W(t) and the FP64 closure of T^-1,
// the clover term in its chiral block form and (A + mu)^-1.
#include "tp_internal.h"
#include "tp_links.h"

namespace {

constexpr int kBlock = 256;

// internal (parity, index) of a site for the p3 or p4 layout
TP_DEV void site_pi(const Geom& g, bool l4, int x, int y, int z, int t, int& p, int64_t& i) {
  int64_t f3 = (int64_t)(x + g.Lx * (y + g.Ly * z));
  if (l4) {
    p = (x + y + z + t) & 1;
    i = (f3 + (int64_t)g.Lx * g.Ly * g.Lz * t) >> 1;
  } else {
    p = (x + y + z) & 1;
    i = p3_idx(g, t, int(f3 >> 1));
  }
}

// psi(colour) <- W^dag psi (to_axial) or W psi (from the axial frame), all four spins, FP64.
TP_DEV void rotate_spinor(const double2* __restrict__ w, int p, int64_t i, int64_t V2, bool dag,
                          cx<double>* v) {
  const double2* b = w + (int64_t)p * 9 * V2 + i;
  su3<double> W;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    double2 e = b[(int64_t)k * V2];
    W.e[k] = cx<double>{e.x, e.y};
  }
#pragma unroll
  for (int sp = 0; sp < 4; ++sp) {
    cx<double> o[3];
    if (dag) mvd(W, v + 3 * sp, o);
    else mv(W, v + 3 * sp, o);
#pragma unroll
    for (int c = 0; c < 3; ++c) v[3 * sp + c] = o[c];
  }
}

// Canonical spinors <-> an internal layout, with the rotation into and out of the axial frame (w) and
// gamma5.  Bound by bytes (F64, p3: 528 per site).  A workgroup's two wavefronts handle the two
// parities of a sub-block: 64 sites each, runs of 256 bytes in the planes and W, and together 32
// consecutive canonical sites (spatial indices 2 s and 2 s + 1) per slice.  The canonical field is
// written through LDS, so that a wavefront stores whole lines instead of 16 bytes of 64 sites.
// In canonical order (runs of 64 bytes) pack and unpack took 228 and 255 us at 24^3x128 (F64), 187
// and 176 us now (5.0 and 5.3 TB/s); unpack without LDS 253 us.  Which order pack takes: see
// pack_order.
struct PackSite {
  int64_t n, i;  // canonical site; index in the layout
  int p;         // parity in the layout
  int64_t iw;    // p3 index (of W), parity pw
  int pw;
  int s0, t0;    // first spatial index and slice of the sub-block
  bool ok;
};
constexpr int kPack = 128;
TP_DEV PackSite pack_site(const Geom& g, bool l4) {
  const uint32_t blk = xcd_block(blockIdx.x, gridDim.x), nsb = uint32_t(g.Vs2 + 15) / 16;
  const SubSite q = sub_site_at(g, blk * 2 + (threadIdx.x >> 6), threadIdx.x & 63);
  const C3 c = p3_coords(g, q.p, q.s);
  PackSite r;
  r.n = c.x + (int64_t)g.Lx * (c.y + (int64_t)g.Ly * (c.z + (int64_t)g.Lz * q.t));
  r.iw = p3_idx(g, q.t, q.s);
  r.pw = q.p;
  r.p = l4 ? (q.p ^ (q.t & 1)) : q.p;
  r.i = l4 ? q.s + (int64_t)g.Vs2 * q.t : r.iw;
  r.s0 = int(blk % nsb) * 16;
  r.t0 = int(blk / nsb) * 4;
  r.ok = q.ok;
  return r;
}

// The same for a thread per site in canonical order (parts: of which each XCD takes a contiguous part).
constexpr int kPackCanon = 256;
TP_DEV PackSite pack_site_canon(const Geom& g, bool l4, bool parts) {
  PackSite r;
  r.n = (int64_t)(parts ? xcd_block(blockIdx.x, gridDim.x) : blockIdx.x) * kPackCanon + threadIdx.x;
  r.ok = r.n < 2 * g.V2;
  const int x = int(r.n % g.Lx);
  int64_t q = r.n / g.Lx;
  const int y = int(q % g.Ly);
  q /= g.Ly;
  const int z = int(q % g.Lz), t = int(q / g.Lz);
  r.pw = (x + y + z) & 1;
  r.iw = p3_idx(g, t, p3_index(g, x, y, z));
  r.p = l4 ? (r.pw ^ (t & 1)) : r.pw;
  r.i = l4 ? r.n >> 1 : r.iw;
  r.s0 = r.t0 = 0;
  return r;
}

template <typename S, bool CANON>
__global__ void __launch_bounds__(CANON ? kPackCanon : kPack) k_pack(const double2* __restrict__ canon, SpinorF<S> f0, SpinorF<S> f1,
                                                 Geom g, bool l4, bool g5,
                                                 const double2* __restrict__ w, bool parts) {
  using R = typename Prec<S>::R;
  const PackSite q = CANON ? pack_site_canon(g, l4, parts) : pack_site(g, l4);
  if (!q.ok) return;
  cx<double> d[12];
  const double2* src = canon + q.n * 12;
#pragma unroll
  for (int c = 0; c < 12; ++c) d[c] = cx<double>{src[c].x, src[c].y};
  if (w) rotate_spinor(w, q.pw, q.iw, g.V2, true, d);
  cx<R> v[12];
#pragma unroll
  for (int c = 0; c < 12; ++c) v[c] = cx<R>{R(d[c].re), R(d[c].im)};
  if (g5) {  // gamma5 = [[0,-1],[-1,0]] in the Dirac-Pauli basis
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      cx<R> a = v[c];
      v[c] = -v[6 + c];
      v[6 + c] = -a;
    }
  }
  const SpinorF<S> f = q.p ? f1 : f0;
  store_half<S, R>(f, 0, q.i, v);
  store_half<S, R>(f, 1, q.i, v + 6);
}

template <typename S>
__global__ void __launch_bounds__(kPack) k_unpack(double2* __restrict__ canon, SpinorF<S> f0, SpinorF<S> f1, Geom g,
                                                   bool l4, bool g5, const double2* __restrict__ w) {
  using R = typename Prec<S>::R;
  constexpr int kPad = 13;  // double2 per site in LDS: 16 lanes' 16-byte accesses meet every bank once
  __shared__ double2 out[128 * kPad];
  const PackSite q = pack_site(g, l4);
  cx<R> v[12];
  const SpinorF<S> f = q.p ? f1 : f0;
  load_half<S, R>(f, 0, q.i, v);
  load_half<S, R>(f, 1, q.i, v + 6);
  if (g5) {
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      cx<R> a = v[c];
      v[c] = -v[6 + c];
      v[6 + c] = -a;
    }
  }
  cx<double> d[12];
#pragma unroll
  for (int c = 0; c < 12; ++c) d[c] = cx<double>{double(v[c].re), double(v[c].im)};
  if (w) rotate_spinor(w, q.pw, q.iw, g.V2, false, d);
  // site of the 4 x 32: slice, then canonical order (n is even or odd with the site's parity)
  const int lane = threadIdx.x & 63;
  double2* o = out + ((lane >> 4) * 32 + (lane & 15) * 2 + int(q.n & 1)) * kPad;
  if (q.ok) {
#pragma unroll
    for (int c = 0; c < 12; ++c) o[c] = make_double2(d[c].re, d[c].im);
  }
  __syncthreads();
  const int sites = 2 * (g.Vs2 - q.s0 < 16 ? g.Vs2 - q.s0 : 16);  // per slice
  for (int r = 0; r < 4 && q.t0 + r < g.Lt; ++r) {
    double2* dst = canon + (2 * (q.s0 + (int64_t)g.Vs2 * (q.t0 + r))) * 12;
    for (int k = threadIdx.x; k < sites * 12; k += kPack) dst[k] = out[(r * 32 + k / 12) * kPad + k % 12];
  }
}

// W(t) = U'(t) U'(t+1) ... U'(Lt-1) per time line, U' the time links with the phase b
// folded into U'(Lt-1).  One thread per line: an Lt-step product, run once per gauge field.
// Bound by the latency of the links' loads, which do not depend on the product: they are issued
// kAhead slices ahead (24^3x128: 0.17 ms with none ahead).
constexpr int kAhead = 4;
__global__ void __launch_bounds__(64) k_wline(const double2* __restrict__ canon, double2* wd, double2* poly, Geom g,
                                              int64_t V, double b) {
  int s = blockIdx.x * blockDim.x + threadIdx.x;
  int p = blockIdx.y;
  if (s >= g.Vs2) return;
  int64_t V2 = g.V2;
  C3 q = p3_coords(g, p, s);
  int64_t f3 = (int64_t)q.x + (int64_t)g.Lx * (q.y + (int64_t)g.Ly * q.z);
  int64_t Vs = (int64_t)g.Lx * g.Ly * g.Lz;
  double2* w = wd + (int64_t)p * 9 * V2;
  const double2* line = canon + ((int64_t)3 * V + f3) * 9;
  double2 buf[kAhead][9];
#pragma unroll
  for (int a = 0; a < kAhead; ++a)
#pragma unroll
    for (int k = 0; k < 9; ++k) buf[a][k] = line[Vs * (g.Lt - 1 - a > 0 ? g.Lt - 1 - a : 0) * 9 + k];
  cx<double> acc[9], u[9], nw[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) acc[k] = cx<double>{(k % 4 == 0) ? 1.0 : 0.0, 0.0};
  for (int t0 = g.Lt - 1; t0 >= 0; t0 -= kAhead) {
#pragma unroll
    for (int a = 0; a < kAhead; ++a) {
      const int t = t0 - a;
      if (t < 0) break;
      const int64_t i = p3_idx(g, t, s);
      const double ph = t == g.Lt - 1 ? b : 1.0;
      const int tn = t - kAhead > 0 ? t - kAhead : 0;
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        u[k] = cx<double>{ph * buf[a][k].x, ph * buf[a][k].y};
        buf[a][k] = line[Vs * tn * 9 + k];
      }
      mm3(u, acc, nw);
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        acc[k] = nw[k];
        w[(int64_t)k * V2 + i] = make_double2(nw[k].re, nw[k].im);
      }
    }
  }
  double2* pl = poly + (int64_t)p * 9 * g.Vs2;
#pragma unroll
  for (int k = 0; k < 9; ++k) pl[(int64_t)k * g.Vs2 + s] = make_double2(acc[k].re, acc[k].im);
}

// The links' layouts, from one read of the canonical links: p4 planes (F64, F32; the 4D even-odd
// operator) with the phase b folded into U_t(Lt-1), and p3 planes (F64, F32, F16) of the
// axial-gauge links U^ax_mu(x) = W(x)^dag U'_mu(x) W(x+mu) with Omega = W^dag (Sec. II.C, App. C):
// every time link becomes the identity except U^ax_t(Lt-1) = W(0) = P.  A workgroup handles the
// 64 sites of a sub-block, wavefront mu one direction, so that planes and W are runs of 256 bytes;
// the caller's links are nine loads whose lanes lie 144 bytes apart.  At 24^3x128 1.58 ms, 2.75 TB/s of
// the 2448 bytes per site that it cannot do without (1872 of them written); 2.9 ms in three kernels
// in canonical order, whose planes took 16 and 64 bytes at a time.
__global__ void __launch_bounds__(256) k_links(const double2* __restrict__ canon, const double2* __restrict__ wd,
                                               double2* u3d, float2* u3f, __half2* u3h, double2* u4d, float2* u4f,
                                               Geom g, int64_t V, double b, int* flags) {
  const int lane = threadIdx.x & 63, mu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const SubSite q = sub_site(g, lane);
  if (!q.ok) return;
  const C3 c = p3_coords(g, q.p, q.s);
  const int t = q.t, pa = q.p;
  const int xn = mu == 0 ? (c.x + 1 == g.Lx ? 0 : c.x + 1) : c.x;
  const int yn = mu == 1 ? (c.y + 1 == g.Ly ? 0 : c.y + 1) : c.y;
  const int zn = mu == 2 ? (c.z + 1 == g.Lz ? 0 : c.z + 1) : c.z;
  const int tn = mu == 3 ? (t + 1 == g.Lt ? 0 : t + 1) : t;
  const int64_t n = c.x + (int64_t)g.Lx * (c.y + (int64_t)g.Ly * (c.z + (int64_t)g.Lz * t));
  const int64_t ia = p3_idx(g, t, q.s), V2 = g.V2;
  int pb;
  int64_t ib;
  site_pi(g, false, xn, yn, zn, tn, pb, ib);
  cx<double> U[9], Wa[9], Wb[9], T1[9], T2[9];
  const double ph = (mu == 3 && t == g.Lt - 1) ? b : 1.0;
  const double2* src = canon + ((int64_t)mu * V + n) * 9;
  bool finite = true;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const double2 e = src[k];
    finite = finite && isfinite(e.x) && isfinite(e.y);
    U[k] = cx<double>{ph * e.x, ph * e.y};
    const double2 ea = wd[((int64_t)pa * 9 + k) * V2 + ia];
    const double2 eb = wd[((int64_t)pb * 9 + k) * V2 + ib];
    Wa[k] = cx<double>{ea.x, -ea.y};  // conj, transposed below
    Wb[k] = cx<double>{eb.x, eb.y};
  }
  {
    const int p4 = pa ^ (t & 1);
    const int64_t i4 = q.s + (int64_t)g.Vs2 * t, off = (int64_t)(mu * 2 + p4) * 9 * V2;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      u4d[off + (int64_t)k * V2 + i4] = make_double2(U[k].re, U[k].im);
      u4f[off + comp_off<float2>(k, 9, V2, i4)] = make_float2(float(U[k].re), float(U[k].im));
    }
  }
  cx<double> Wad[9];
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int k = 0; k < 3; ++k) Wad[3 * r + k] = Wa[3 * k + r];
  mm3(Wad, U, T1);
  mm3(T1, Wb, T2);
  const int64_t off = (int64_t)(mu * 2 + pa) * 9 * V2;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const float2 f = make_float2(float(T2[k].re), float(T2[k].im));
    u3d[off + (int64_t)k * V2 + ia] = make_double2(T2[k].re, T2[k].im);
    u3f[off + comp_off<float2>(k, 9, V2, ia)] = f;
    u3h[off + comp_off<__half2>(k, 9, V2, ia)] = __float22half2_rn(f);
  }
  // spatial links: deviation of the axial-frame link from SU(3); time links: deviation of
  // the input link from unitarity (the axial frame is a gauge rotation only for unitary W)
  cx<double> m[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) m[k] = mu < 3 ? T2[k] : U[k];
  double dev = 0;
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      cx<double> e = cx<double>{r == k ? -1.0 : 0.0, 0.0};
#pragma unroll
      for (int j = 0; j < 3; ++j) e += cmul(m[3 * r + j], conj(m[3 * k + j]));
      dev = fmax(dev, sqrt(norm2(e)));
    }
  if (mu < 3) {
    cx<double> c0 = cmul(m[4], m[8]) - cmul(m[5], m[7]);
    cx<double> c1 = cmul(m[5], m[6]) - cmul(m[3], m[8]);
    cx<double> c2 = cmul(m[3], m[7]) - cmul(m[4], m[6]);
    cx<double> det = cmul(m[0], c0) + cmul(m[1], c1) + cmul(m[2], c2);
    dev = fmax(dev, sqrt(norm2(det - cx<double>{1.0, 0.0})));
    if (!(dev <= 1e-9)) flags[0] = 1;
    if (!(dev <= 1e-13)) flags[3] = 1;
  } else if (!(dev <= 1e-10)) {
    flags[1] = 1;
  }
  if (!finite) flags[2] = 1;
}

TP_DEV bool inv3(const cx<double>* m, cx<double>* r) {
  // adjugate / determinant
  cx<double> c00 = cmul(m[4], m[8]) - cmul(m[5], m[7]);
  cx<double> c01 = cmul(m[5], m[6]) - cmul(m[3], m[8]);
  cx<double> c02 = cmul(m[3], m[7]) - cmul(m[4], m[6]);
  cx<double> det = cmul(m[0], c00) + cmul(m[1], c01) + cmul(m[2], c02);
  double dn = norm2(det);
  if (!(dn > 0.0)) return false;
  cx<double> id = cx<double>{det.re / dn, -det.im / dn};
  r[0] = cmul(c00, id);
  r[3] = cmul(c01, id);
  r[6] = cmul(c02, id);
  r[1] = cmul(cmul(m[2], m[7]) - cmul(m[1], m[8]), id);
  r[4] = cmul(cmul(m[0], m[8]) - cmul(m[2], m[6]), id);
  r[7] = cmul(cmul(m[1], m[6]) - cmul(m[0], m[7]), id);
  r[2] = cmul(cmul(m[1], m[5]) - cmul(m[2], m[4]), id);
  r[5] = cmul(cmul(m[2], m[3]) - cmul(m[0], m[5]), id);
  r[8] = cmul(cmul(m[0], m[4]) - cmul(m[1], m[3]), id);
  return true;
}

TP_DEV double norm1(const cx<double>* m) {
  double best = 0;
  for (int j = 0; j < 3; ++j) {
    double s = 0;
    for (int i = 0; i < 3; ++i) s += sqrt(norm2(m[3 * i + j]));
    best = fmax(best, s);
  }
  return best;
}

// Closure of the temporal inverse per line: K = (I - mu^-Lt P)^-1 and G = K P / mu,
// so that delta = G sigma(0) for T^-1 and delta' = G^dagger rho(Lt-1) for T^dagger^-1.
__global__ void k_closure(const double2* __restrict__ poly, double2* gclos, float2* gclos_f,
                          double* cond, Geom g, double mu, double mu_mlt) {
  int s = blockIdx.x * blockDim.x + threadIdx.x;
  int p = blockIdx.y;
  if (s >= g.Vs2) return;
  const double2* pl = poly + (int64_t)p * 9 * g.Vs2;
  cx<double> P[9], A[9], K[9], G[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    double2 e = pl[(int64_t)k * g.Vs2 + s];
    P[k] = cx<double>{e.x, e.y};
    A[k] = cx<double>{(k % 4 == 0 ? 1.0 : 0.0) - mu_mlt * e.x, -mu_mlt * e.y};
  }
  double c;
  if (inv3(A, K)) {
    c = norm1(A) * norm1(K);
    mm3(K, P, G);
  } else {
    c = INFINITY;
    for (int k = 0; k < 9; ++k) G[k] = cx<double>{0, 0};
  }
  if (!isfinite(c)) c = INFINITY;
  cond[(int64_t)p * g.Vs2 + s] = c;
  double2* go = gclos + (int64_t)p * 9 * g.Vs2;
  float2* gf = gclos_f + (int64_t)p * 9 * g.Vs2;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    go[(int64_t)k * g.Vs2 + s] = make_double2(G[k].re / mu, G[k].im / mu);
    gf[(int64_t)k * g.Vs2 + s] = make_float2(float(G[k].re / mu), float(G[k].im / mu));
  }
}

// ---- clover ------------------------------------------------------------------------------
struct SigTab {
  double2 s[6][2][2][2];  // plane, chirality, row, col:  coef_p * V_chi^dag sigma_p V_chi / 2
};

TP_DEV void chain4(const cx<double>* a, const cx<double>* b, const cx<double>* c,
                   const cx<double>* d, cx<double>* out) {
  cx<double> t1[9], t2[9];
  mm3(a, b, t1);
  mm3(t1, c, t2);
  mm3(t2, d, out);
}

// F_{mu nu}(x) = (Q - Q^dag)/8 - tr/3 with Q the four leaves, all oriented mu -> nu: exactly
// anti-hermitian as computed (each entry is the rounded negative conjugate of its mirror).
template <bool AX>
TP_DEV void field_strength(const double2* __restrict__ u, const Geom& g, int mu, int nu, int x, int y, int z,
                           int t, cx<double>* F) {
  // U_d(x + am*mu + an*nu); the offsets are formed arithmetically (a direction table indexed
  // by mu and nu would live in scratch memory)
  auto L = [&](int d, int am, int an, cx<double>* m) {
    load_soa<AX>(u, g, d, x + am * (mu == 0) + an * (nu == 0), y + am * (mu == 1) + an * (nu == 1),
            z + am * (mu == 2) + an * (nu == 2), t + am * (mu == 3) + an * (nu == 3), m);
  };
  cx<double> a[9], b[9], c[9], d[9], cd[9], dd[9], leaf[9], Q[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) Q[k] = cx<double>{0, 0};
  // leaf 1: U_mu(x) U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag
  L(mu, 0, 0, a); L(nu, 1, 0, b); L(mu, 0, 1, c); L(nu, 0, 0, d);
  dag3(c, cd); dag3(d, dd); chain4(a, b, cd, dd, leaf);
#pragma unroll
  for (int k = 0; k < 9; ++k) Q[k] += leaf[k];
  // leaf 2: U_nu(x) U_mu(x-mu+nu)^dag U_nu(x-mu)^dag U_mu(x-mu)
  L(nu, 0, 0, a); L(mu, -1, 1, b); L(nu, -1, 0, c); L(mu, -1, 0, d);
  { cx<double> bd[9]; dag3(b, bd); dag3(c, cd); chain4(a, bd, cd, d, leaf); }
#pragma unroll
  for (int k = 0; k < 9; ++k) Q[k] += leaf[k];
  // leaf 3: U_mu(x-mu)^dag U_nu(x-mu-nu)^dag U_mu(x-mu-nu) U_nu(x-nu)
  L(mu, -1, 0, a); L(nu, -1, -1, b); L(mu, -1, -1, c); L(nu, 0, -1, d);
  { cx<double> ad[9], bd[9]; dag3(a, ad); dag3(b, bd); chain4(ad, bd, c, d, leaf); }
#pragma unroll
  for (int k = 0; k < 9; ++k) Q[k] += leaf[k];
  // leaf 4: U_nu(x-nu)^dag U_mu(x-nu) U_nu(x+mu-nu) U_mu(x)^dag
  L(nu, 0, -1, a); L(mu, 0, -1, b); L(nu, 1, -1, c); L(mu, 0, 0, d);
  { cx<double> ad[9]; dag3(a, ad); dag3(d, dd); chain4(ad, b, c, dd, leaf); }
#pragma unroll
  for (int k = 0; k < 9; ++k) Q[k] += leaf[k];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) F[3 * i + j] = 0.125 * (Q[3 * i + j] - conj(Q[3 * j + i]));
  cx<double> tr = (1.0 / 3.0) * (F[0] + F[4] + F[8]);
  F[0] -= tr; F[4] -= tr; F[8] -= tr;
}

// An anti-hermitian 3x3 matrix in LDS as nine reals per site: the imaginary diagonal, then the
// entries (1,0), (2,0), (2,1); consecutive lanes are adjacent.
struct AntiH {
  double* p;
  int lane;
  TP_DEV double& at(int k) const { return p[k * kSub + lane]; }
  TP_DEV void put(const cx<double>* F) const {
    at(0) = F[0].im; at(1) = F[4].im; at(2) = F[8].im;
    at(3) = F[3].re; at(4) = F[3].im;
    at(5) = F[6].re; at(6) = F[6].im;
    at(7) = F[7].re; at(8) = F[7].im;
  }
  TP_DEV cx<double> low(int a, int b) const {  // a > b
    const int k = a == 1 ? 3 : (b == 0 ? 5 : 7);
    return cx<double>{at(k), at(k + 1)};
  }
  TP_DEV cx<double> get(int a, int b) const {
    if (a == b) return cx<double>{0.0, at(a)};
    if (a > b) return low(a, b);
    const cx<double> v = low(b, a);
    return cx<double>{-v.re, v.im};
  }
};

// The stored entries (6 real diagonal, 15 complex below it) of chiral block C: the sum over the
// planes of the sigma-table coefficients times F, all at compile-time indices.
template <int C>
TP_DEV void chiral_block(double* fs, int lane, const SigTab& sig, double* dg, cx<double>* lo) {
#pragma unroll
  for (int k = 0; k < 6; ++k) dg[k] = 0.0;
#pragma unroll
  for (int k = 0; k < 15; ++k) lo[k] = cx<double>{0, 0};
#pragma unroll
  for (int pl = 0; pl < 6; ++pl) {
    const AntiH F{fs + pl * 9 * kSub, lane};
    const double2 w00 = sig.s[pl][C][0][0], w10 = sig.s[pl][C][1][0], w11 = sig.s[pl][C][1][1];
#pragma unroll
    for (int r = 0; r < 6; ++r)
#pragma unroll
      for (int q = 0; q <= r; ++q) {
        const int sr = r / 3, sq = q / 3;
        const double2 wv = sr == 0 ? w00 : (sq == 0 ? w10 : w11);
        const cx<double> v = cmul(cx<double>{wv.x, wv.y}, F.get(r % 3, q % 3));
        if (r == q) dg[r] += v.re;
        else lo[r * (r - 1) / 2 + q] += v;
      }
  }
}

// The clover term in one frame: p3 blocks from the axial-frame links (AX; every p3 operator),
// p4 blocks from the original links (the 4D even-odd operator).  One workgroup handles 64 sites;
// its wavefronts form F of two planes each, then, through LDS, two of them one chiral block each.
//
// Bound by the fabric: 72 link matrices (10 KB) per site and frame, few of which a cache still
// holds.  F is formed once per site, not once per chirality; the links come from planes in which
// adjacent lanes are adjacent (canonical links, 144 bytes a lane, cost one cache line per lane and
// load), and the sub-block order keeps a neighbour's links in the XCD's L2.  Both frames at
// 24^3x128: 6.5 ms with a thread per site, chirality and frame on canonical links; 6.4 ms in
// blocks dealt to the XCDs in turn (20.9 GB fetched per launch); 3.6 ms so (2, 3 and 6 wavefronts
// per workgroup: 3.7, 3.6 and 4.2 ms).
constexpr int kClovWaves = 3;
template <bool AX, int NW>
__global__ void __launch_bounds__(64 * NW) k_clover_build(const double2* __restrict__ u, double2* ad, float2* af,
                                                      __half2* ah, Geom g, SigTab sig, uint32_t planes) {
  __shared__ double fs[6 * 9 * kSub];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const SubSite q = sub_site(g, lane);
  const C3 c = p3_coords(g, q.p, q.s);
#pragma unroll 1
  for (int pl = (6 / NW) * wave; pl < (6 / NW) * (wave + 1); ++pl) {  // planes 03 13 23 | 01 02 12
    const int mu = pl < 3 ? pl : (pl == 5 ? 1 : 0), nu = pl < 3 ? 3 : (pl == 3 ? 1 : 2);
    cx<double> F[9];
    if ((planes >> pl) & 1u) {
      field_strength<AX>(u, g, mu, nu, c.x, c.y, c.z, q.t, F);
    } else {
#pragma unroll
      for (int k = 0; k < 9; ++k) F[k] = cx<double>{0, 0};
    }
    AntiH{fs + pl * 9 * kSub, lane}.put(F);
  }
  __syncthreads();
  if (!q.ok || wave >= 2) return;
  const int C = wave;
  double dg[6];
  cx<double> lo[15];
  if (C == 0) chiral_block<0>(fs, lane, sig, dg, lo);
  else chiral_block<1>(fs, lane, sig, dg, lo);
  const int p = AX ? q.p : (q.p ^ (q.t & 1));
  const int64_t off = ((int64_t)p * 36 + 18 * C) * g.V2;
  const int64_t i = AX ? p3_idx(g, q.t, q.s) : q.s + (int64_t)g.Vs2 * q.t;
  // slots 0..2: diagonal pairs, 3..17: lower triangle row-major (the layout of store_herm6_parts)
#pragma unroll
  for (int slot = 0; slot < 18; ++slot) {
    const double2 v = slot < 3 ? make_double2(dg[2 * slot], dg[2 * slot + 1])
                               : make_double2(lo[slot - 3].re, lo[slot - 3].im);
    const float2 vf = make_float2(float(v.x), float(v.y));
    ad[off + (int64_t)slot * g.V2 + i] = v;
    af[off + comp_off<float2>(slot, 18, g.V2, i)] = vf;
    if constexpr (AX) ah[off + comp_off<__half2>(slot, 18, g.V2, i)] = __float22half2_rn(vf);
  }
}

// Inverse of a hermitian 6x6 block from its stored form (real diagonal dg, lower triangle lo
// row-major), by H = L D L^dag with L unit lower triangular and D real: H^-1 = L^-dag D^-1 L^-1.
// Every loop has fixed bounds, so all entries stay in registers.  Returns false when a pivot
// falls below 1e-13 of the largest diagonal entry (the block is then reported singular).
TP_DEV bool inv_herm6(const double* dg, const cx<double>* lo, double* idg, cx<double>* ilo) {
  auto T = [](int r, int c) { return r * (r - 1) / 2 + c; };  // lower-triangle index, r > c
  double scale = 0;
#pragma unroll
  for (int k = 0; k < 6; ++k) scale = fmax(scale, fabs(dg[k]));
  double d[6];
  cx<double> L[15];
  bool ok = true;
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    double dj = dg[j];
#pragma unroll
    for (int k = 0; k < j; ++k) dj -= norm2(L[T(j, k)]) * d[k];
    d[j] = dj;
    if (!(fabs(dj) > 1e-13 * scale)) ok = false;
    const double id = 1.0 / dj;
#pragma unroll
    for (int i = j + 1; i < 6; ++i) {
      cx<double> v = lo[T(i, j)];
#pragma unroll
      for (int k = 0; k < j; ++k) v -= d[k] * cmul(L[T(i, k)], conj(L[T(j, k)]));
      L[T(i, j)] = id * v;
    }
  }
  // M = L^-1 (unit lower triangular), by forward substitution
  cx<double> M[15];
#pragma unroll
  for (int i = 1; i < 6; ++i)
#pragma unroll
    for (int j = 0; j < i; ++j) {
      cx<double> v = -L[T(i, j)];
#pragma unroll
      for (int k = j + 1; k < i; ++k) v -= cmul(L[T(i, k)], M[T(k, j)]);
      M[T(i, j)] = v;
    }
  // H^-1[i][j] = sum_{k >= i} conj(M[k][i]) M[k][j] / d[k]  (i >= j; M[k][k] = 1)
  double id[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) id[k] = 1.0 / d[k];
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    double v = id[i];
#pragma unroll
    for (int k = i + 1; k < 6; ++k) v += norm2(M[T(k, i)]) * id[k];
    idg[i] = v;
  }
#pragma unroll
  for (int i = 1; i < 6; ++i)
#pragma unroll
    for (int j = 0; j < i; ++j) {
      cx<double> v = id[i] * M[T(i, j)];
#pragma unroll
      for (int k = i + 1; k < 6; ++k) v += id[k] * cmul(conj(M[T(k, i)]), M[T(k, j)]);
      ilo[T(i, j)] = v;
    }
  return ok;
}

// Stored form of a hermitian block: slots 0..2 diagonal pairs, 3..17 the lower triangle
// row-major.  The clover kernels read this form (clover_apply, herm6_from_slots).
TP_DEV void load_herm6_parts(const double2* base, int64_t st, int64_t i, double* dg, cx<double>* lo) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double2 v = base[(int64_t)k * st + i];
    dg[2 * k] = v.x;
    dg[2 * k + 1] = v.y;
  }
#pragma unroll
  for (int k = 0; k < 15; ++k) {
    const double2 v = base[(int64_t)(3 + k) * st + i];
    lo[k] = cx<double>{v.x, v.y};
  }
}
TP_DEV void store_herm6_parts(const double* dg, const cx<double>* lo, double2* d, float2* f, __half2* h,
                              int64_t st, int64_t i) {
#pragma unroll
  for (int slot = 0; slot < 18; ++slot) {
    const double2 v = slot < 3 ? make_double2(dg[2 * slot], dg[2 * slot + 1])
                               : make_double2(lo[slot - 3].re, lo[slot - 3].im);
    d[(int64_t)slot * st + i] = v;
    const float2 vf = make_float2(float(v.x), float(v.y));
    f[comp_off<float2>(slot, 18, st, i)] = vf;
    if (h) h[comp_off<__half2>(slot, 18, st, i)] = __float22half2_rn(vf);
  }
}

// From the stored A/2 blocks (layout p3 or p4), write (A+mu)/2 and (A+mu)^-1/2 blocks (the FP16
// copies of the p3 layout as well).
__global__ void __launch_bounds__(64) k_clover_derived(const double2* __restrict__ a, double2* amu,
                                                       double2* ainv, float2* amu_f, float2* ainv_f,
                                                       __half2* amu_h, __half2* ainv_h,
                                                       int64_t V2, double mu, int* bad) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int p = blockIdx.y;
  if (i >= V2) return;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int64_t off = ((int64_t)p * 36 + 18 * c) * V2;
    double dg[6], idg[6];
    cx<double> lo[15], ilo[15];
    if (a) {
      load_herm6_parts(a + off, V2, i, dg, lo);
    } else {
#pragma unroll
      for (int k = 0; k < 6; ++k) dg[k] = 0.0;
#pragma unroll
      for (int k = 0; k < 15; ++k) lo[k] = cx<double>{0, 0};
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) dg[k] += 0.5 * mu;  // (A + mu)/2
    store_herm6_parts(dg, lo, amu + off, amu_f + off, amu_h ? amu_h + off : nullptr, V2, i);
    // (A+mu)^-1/2 = [(A+mu)/2]^-1 / 4
    if (!inv_herm6(dg, lo, idg, ilo)) {
      bad[0] = 1;
#pragma unroll
      for (int k = 0; k < 6; ++k) idg[k] = 0.0;
#pragma unroll
      for (int k = 0; k < 15; ++k) ilo[k] = cx<double>{0, 0};
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) idg[k] *= 0.25;
#pragma unroll
    for (int k = 0; k < 15; ++k) ilo[k] = 0.25 * ilo[k];
    store_herm6_parts(idg, ilo, ainv + off, ainv_f + off, ainv_h ? ainv_h + off : nullptr, V2, i);
  }
}

// Plaquette averages (1/3 Re tr) over spatial and temporal planes: a workgroup handles the 64
// sites of a sub-block, each of its three wavefronts two planes, and writes one partial pair;
// Re tr(U_mu(x) U_nu(x+mu) [U_nu(x) U_mu(x+nu)]^dag) needs two products and a sum.  Bound by the
// links' reads (24^3x128: 2.1 ms from canonical links, one cache line per lane and load).
__global__ void __launch_bounds__(192) k_plaquette(const double2* __restrict__ u4, Geom g, double* part) {
  __shared__ double sh[3][2];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const SubSite q = sub_site(g, lane);
  const C3 c = p3_coords(g, q.p, q.s);
  double ps = 0, pt = 0;
  // planes 01 02 | 12 03 | 13 23; offsets formed arithmetically, not from a table indexed by
  // the plane (which would live in scratch memory)
#pragma unroll 1
  for (int pl = 2 * wave; pl < 2 * wave + 2; ++pl) {
    const int mu = pl == 2 || pl == 4 ? 1 : (pl == 5 ? 2 : 0);
    const int nu = pl < 3 ? (pl == 0 ? 1 : 2) : 3;
    cx<double> a[9], b[9], m[9], n[9];
    load_soa<false>(u4, g, mu, c.x, c.y, c.z, q.t, a);
    load_soa<false>(u4, g, nu, c.x + (mu == 0), c.y + (mu == 1), c.z + (mu == 2), q.t, b);
    mm3(a, b, m);
    load_soa<false>(u4, g, nu, c.x, c.y, c.z, q.t, a);
    load_soa<false>(u4, g, mu, c.x, c.y + (nu == 1), c.z + (nu == 2), q.t + (nu == 3), b);
    mm3(a, b, n);
    double re = 0;
#pragma unroll
    for (int k = 0; k < 9; ++k) re += m[k].re * n[k].re + m[k].im * n[k].im;
    re /= 3.0;
    if (!q.ok) re = 0;
    if (pl < 3) ps += re; else pt += re;
  }
  for (int off = 32; off > 0; off >>= 1) {
    ps += __shfl_xor(ps, off);
    pt += __shfl_xor(pt, off);
  }
  if (lane == 0) {
    sh[wave][0] = ps;
    sh[wave][1] = pt;
  }
  __syncthreads();
  if (threadIdx.x < 2) part[2 * (int64_t)blockIdx.x + threadIdx.x] = sh[0][threadIdx.x] + sh[1][threadIdx.x] + sh[2][threadIdx.x];
}
// Sums the n partial pairs into the pair behind them.
__global__ void __launch_bounds__(kBlock) k_plaquette_sum(double* part, int64_t n) {
  __shared__ double sh[2][kBlock];
  double v[2] = {0, 0};
  for (int64_t k = threadIdx.x; k < n; k += kBlock) {
    v[0] += part[2 * k];
    v[1] += part[2 * k + 1];
  }
  sh[0][threadIdx.x] = v[0];
  sh[1][threadIdx.x] = v[1];
  __syncthreads();
  for (int w = kBlock / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      sh[0][threadIdx.x] += sh[0][threadIdx.x + w];
      sh[1][threadIdx.x] += sh[1][threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x < 2) part[2 * n + threadIdx.x] = sh[threadIdx.x][0];
}

inline unsigned nblk(int64_t n, int64_t b = kBlock) { return (unsigned)((n + b - 1) / b); }

// Up to 65536 sites sub-blocks always: they leave a site in the L2 of the XCD whose next kernel reads
// it (a 4D even-odd apply at 8^3x32, F64: 30.4 us, 31.7 with canonical order, 30.9 with its parts).
// Beyond, into p4, where canonical order is that of the planes and sub-blocks only shorten the runs (in
// us: sub-blocks, canonical order, its parts):
//   parts up to 2^20 sites, for the same reason (F64 16^3x128 31.4, 35.4, 30.7 and the apply 380, 383, 378;
//     32^3x32 82.8, 81.5, 78.5 and 875, 884, 868), plain beyond (32^3x128 321, 295, 306 and 3062, 3045, 3055; F32
//     40^3x48 188, 160, 167).
// Into p3 sub-blocks pay (F64 24^3x128 186 and 247 us, 32^3x4 11.0 and 11.7) but for
//   lines of 5 to 27 slices that are no multiple of four, whose last slices leave sub-blocks part
//     empty: 32^3x5 20.2 and 16.3, 32^3x14 41.8 and 38.3, F32 32^3x18 41.9 and 39.8 (but F64 32^3x26 93
//     and 99; 32^3x3 8.7 and 9.6, 32^3x33 138 and 145; parts 32^3x5 18.1, 32^3x14 47.0);
//   odd lines of 64 slices or more in a field that outgrows the last-level cache (256 MB): their runs
//     start in the middle of a cache line, whose halves are then written to memory apart: 24^3x107
//     203 and 195 us (24^3x106: 159 and 191), F32 32^3x65 228 and 212, but 16^3x255 123 and 159.
enum PackOrder { kPackSub, kPackPlain, kPackParts };
PackOrder pack_order(const Lattice& L, bool l4) {
  const int Lt = L.L[3];
  if (L.V <= (1 << 16)) return kPackSub;
  if (l4) return L.V <= (1 << 20) ? kPackParts : kPackPlain;
  if (Lt > 4 && Lt < 28 && Lt % 4) return kPackPlain;
  return Lt % 2 && Lt >= 64 && double(L.V) * 192.0 > 256e6 ? kPackPlain : kPackSub;
}
template <typename S>
void pack_t(tp_ctx ctx, const double2* canon, Field& dst, bool l4, bool g5, const double2* w) {
  const Lattice& L = ctx->lat;
  const SpinorF<S> f0 = dst.template par<S>(0), f1 = dst.template par<S>(1);
  const PackOrder o = pack_order(L, l4);
  if (o == kPackSub)
    hipLaunchKernelGGL((k_pack<S, false>), dim3(sub_blocks(L) / 2), dim3(kPack), 0, ctx->stream, canon, f0, f1, L.g,
                       l4, g5, w, false);
  else
    hipLaunchKernelGGL((k_pack<S, true>), dim3(nblk(L.V, kPackCanon)), dim3(kPackCanon), 0, ctx->stream, canon, f0, f1,
                       L.g, l4, g5, w, o == kPackParts);
  LAUNCH_CHECK();
}
template <typename S>
void unpack_t(tp_ctx ctx, const Field& src, double2* canon, bool l4, bool g5, const double2* w) {
  const Lattice& L = ctx->lat;
  hipLaunchKernelGGL(k_unpack<S>, dim3(sub_blocks(L) / 2), dim3(kPack), 0, ctx->stream, canon,
                     src.template par<S>(0), src.template par<S>(1), L.g, l4, g5, w);
  LAUNCH_CHECK();
}


}  // namespace

void launch_pack(tp_ctx ctx, const double2* canon, Field& dst, bool l4, bool g5, const double2* w) {
  ProfScope ps(ctx, KID_PACK, double(ctx->lat.V) * (192 + 2 * Field::half_bytes(dst.prec) + (w ? 144 : 0)));
  switch (dst.prec) {
    case TP_F64: pack_t<double2>(ctx, canon, dst, l4, g5, w); break;
    case TP_F32: pack_t<float2>(ctx, canon, dst, l4, g5, w); break;
    default: pack_t<__half2>(ctx, canon, dst, l4, g5, w); break;
  }
}

void launch_unpack(tp_ctx ctx, const Field& src, double2* canon, bool l4, bool g5, const double2* w) {
  ProfScope ps(ctx, KID_PACK, double(ctx->lat.V) * (192 + 2 * Field::half_bytes(src.prec) + (w ? 144 : 0)));
  switch (src.prec) {
    case TP_F64: unpack_t<double2>(ctx, src, canon, l4, g5, w); break;
    case TP_F32: unpack_t<float2>(ctx, src, canon, l4, g5, w); break;
    default: unpack_t<__half2>(ctx, src, canon, l4, g5, w); break;
  }
}

void launch_wline(tp_ctx ctx, tp_gauge g, const double2* links) {
  const Lattice& L = ctx->lat;
  hipLaunchKernelGGL(k_wline, dim3((L.Vs2 + 63) / 64, 2), dim3(64), 0, ctx->stream, links, g->w_d, g->poly, L.g,
                     L.V, double(ctx->bc));
  LAUNCH_CHECK();
}

void launch_links(tp_ctx ctx, tp_gauge g, const double2* links, int* flags) {
  const Lattice& L = ctx->lat;
  hipLaunchKernelGGL(k_links, dim3(sub_blocks(L)), dim3(256), 0, ctx->stream, links, g->w_d, g->u3_d, g->u3_f,
                     g->u3_h, g->u4_d, g->u4_f, L.g, L.V, double(ctx->bc), flags);
  LAUNCH_CHECK();
}

void launch_closure(tp_ctx ctx, tp_op op, double* cond) {
  const Lattice& L = ctx->lat;
  double mu_mlt = pow(op->mu, -double(L.L[3]));
  hipLaunchKernelGGL(k_closure, dim3((L.Vs2 + 63) / 64, 2), dim3(64), 0, ctx->stream,
                     op->g->poly, op->gclos, op->gclos_f, cond, L.g, op->mu, mu_mlt);
  LAUNCH_CHECK();
}

void launch_clover_build(tp_ctx ctx, tp_clover c, const double sig[6][2][2][2][2]) {
  const Lattice& L = ctx->lat;
  SigTab t;
  uint32_t planes = 0;  // planes with a nonzero coefficient
  for (int p = 0; p < 6; ++p)
    for (int ch = 0; ch < 2; ++ch)
      for (int r = 0; r < 2; ++r)
        for (int q = 0; q < 2; ++q) {
          t.s[p][ch][r][q] = make_double2(sig[p][ch][r][q][0], sig[p][ch][r][q][1]);
          if (sig[p][ch][r][q][0] != 0.0 || sig[p][ch][r][q][1] != 0.0) planes |= 1u << p;
        }
  hipLaunchKernelGGL((k_clover_build<true, kClovWaves>), dim3(sub_blocks(L)), dim3(64 * kClovWaves), 0, ctx->stream, c->g->u3_d, c->a3_d,
                     c->a3_f, c->a3_h, L.g, t, planes);
  LAUNCH_CHECK();
  hipLaunchKernelGGL((k_clover_build<false, kClovWaves>), dim3(sub_blocks(L)), dim3(64 * kClovWaves), 0, ctx->stream, c->g->u4_d, c->a4_d,
                     c->a4_f, (__half2*)nullptr, L.g, t, planes);
  LAUNCH_CHECK();
}

void launch_clover_derived(tp_ctx ctx, tp_op op, int* bad) {
  const Lattice& L = ctx->lat;
  const double2* a4 = op->c ? op->c->a4_d : nullptr;
  const double2* a3 = op->c ? op->c->a3_d : nullptr;
  hipLaunchKernelGGL(k_clover_derived, dim3(nblk(L.V2, 64), 2), dim3(64), 0, ctx->stream, a4,
                     op->a4_mu, op->a4_inv, op->a4_mu_f, op->a4_inv_f, (__half2*)nullptr,
                     (__half2*)nullptr, L.V2, op->mu, bad);
  LAUNCH_CHECK();
  hipLaunchKernelGGL(k_clover_derived, dim3(nblk(L.V2, 64), 2), dim3(64), 0, ctx->stream, a3,
                     op->a3_mu, op->a3_inv, op->a3_mu_f, op->a3_inv_f, op->a3_mu_h, op->a3_inv_h,
                     L.V2, op->mu, bad);
  LAUNCH_CHECK();
}

int64_t plaquette_partials(tp_ctx ctx) { return sub_blocks(ctx->lat); }
void launch_plaquette(tp_ctx ctx, tp_gauge g, double* part) {
  const Lattice& L = ctx->lat;
  hipLaunchKernelGGL(k_plaquette, dim3(sub_blocks(L)), dim3(192), 0, ctx->stream, g->u4_d, L.g, part);
  LAUNCH_CHECK();
  hipLaunchKernelGGL(k_plaquette_sum, dim3(1), dim3(kBlock), 0, ctx->stream, part, plaquette_partials(ctx));
  LAUNCH_CHECK();
}
