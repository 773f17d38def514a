// M, D_s and the clover term on canonical complex128 spinors, in the original frame: one pass
// from the caller's field to the caller's field.
//
// The internal layouts pay when a field is used many times; a single FP64 apply spent more time
// converting it to and from the p3 layout (528 bytes per site each way: the field twice and W)
// than a kernel on the canonical field needs.  The links (p4 planes, phase b folded) and the
// clover blocks (p4) of the original frame are those of the 4D even-odd operator.
#include "tp_internal.h"
#include "tp_links.h"

namespace {

struct CanonArgs {
  const double2* src;
  double2* dst;
  const double2* u4;    // [4 dir][2 parity][9][V2]
  const double2* clov;  // [2 parity][36][V2] or null
  double c_mu, c_A, c_t, c_s;
  Geom g;
};

struct CPt {
  int64_t n;  // canonical site
  int p;      // p4 parity
  int64_t i;  // p4 index
};
TP_DEV CPt canon_point(const Geom& g, int x, int y, int z, int t) {
  x = x < 0 ? x + g.Lx : (x >= g.Lx ? x - g.Lx : x);
  y = y < 0 ? y + g.Ly : (y >= g.Ly ? y - g.Ly : y);
  z = z < 0 ? z + g.Lz : (z >= g.Lz ? z - g.Lz : z);
  t = t < 0 ? t + g.Lt : (t >= g.Lt ? t - g.Lt : t);
  CPt q;
  q.n = x + (int64_t)g.Lx * (y + (int64_t)g.Ly * (z + (int64_t)g.Lz * t));
  q.p = (x + y + z + t) & 1;
  q.i = q.n >> 1;
  return q;
}

// Components [c0, c0 + N) of gamma5 psi (G5) or psi at canonical site n.
template <bool G5, int N>
TP_DEV void ld_canon(const double2* __restrict__ f, int64_t n, int c0, cx<double>* v) {
#pragma unroll
  for (int c = 0; c < N; ++c) {
    const int k = c0 + c;
    const double2 e = f[n * 12 + (G5 ? (k < 6 ? k + 6 : k - 6) : k)];
    v[c] = G5 ? cx<double>{-e.x, -e.y} : cx<double>{e.x, e.y};
  }
}
TP_DEV su3<double> ld_u4(const CanonArgs& a, int mu, const CPt& q) {
  su3<double> u;
  const double2* b = a.u4 + (int64_t)(mu * 2 + q.p) * 9 * a.g.V2 + q.i;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const double2 e = b[(int64_t)k * a.g.V2];
    u.e[k] = cx<double>{e.x, e.y};
  }
  return u;
}

// Forward and backward hop in direction K.
template <bool G5, int K>
TP_DEV void canon_hop(const CanonArgs& a, const C3& c, int t, const CPt& q, double w, cx<double>* out) {
  const CPt f = canon_point(a.g, c.x + (K == 0), c.y + (K == 1), c.z + (K == 2), t + (K == 3));
  const CPt b = canon_point(a.g, c.x - (K == 0), c.y - (K == 1), c.z - (K == 2), t - (K == 3));
  cx<double> h[6], g[6];
  if constexpr (K == 3) {
    ld_canon<G5, 6>(a.src, f.n, 6, h);
    const su3<double> U = ld_u4(a, 3, q);
    mv(U, h, g);
    mv(U, h + 3, g + 3);
#pragma unroll
    for (int k = 0; k < 6; ++k) out[6 + k] += w * g[k];
    ld_canon<G5, 6>(a.src, b.n, 0, h);
    const su3<double> V = ld_u4(a, 3, b);
    mvd(V, h, g);
    mvd(V, h + 3, g + 3);
#pragma unroll
    for (int k = 0; k < 6; ++k) out[k] += w * g[k];
  } else {
    cx<double> psi[12];
    ld_canon<G5, 12>(a.src, f.n, 0, psi);
    proj_minus<K, double>(psi, h);
    const su3<double> U = ld_u4(a, K, q);
    mv(U, h, g);
    mv(U, h + 3, g + 3);
    recon_minus<K, double>(out, g, 0.5 * w);
    ld_canon<G5, 12>(a.src, b.n, 0, psi);
    proj_plus<K, double>(psi, h);
    const su3<double> V = ld_u4(a, K, b);
    mvd(V, h, g);
    mvd(V, h + 3, g + 3);
    recon_plus<K, double>(out, g, 0.5 * w);
  }
}

// dst = c_mu psi + c_A A psi + c_t D_t psi + c_s D_s psi, between two gamma5 when G5.
// A workgroup handles the 64 sites of a sub-block.  Wavefront d < 3 forms the two hops of spatial
// direction d, wavefront 3 those in time and the diagonal terms (HOPS; else one wavefront forms
// the diagonal terms alone); their sums meet in LDS and every wavefront stores a share of the
// components.  Bound by bytes on large lattices and by latency on small ones, where a thread per
// site would wait for its eight hops one after another.  With the conversions replaced: M at 4^3x16
// (Wilson) 29 -> 8.9 us; at 24^3x128 M 1.26 -> 0.80 ms (clover), D_s 0.90 -> 0.54, A 0.84 -> 0.36.
template <bool G5, bool HOPS, bool TIME, bool CLOV>
__global__ void __launch_bounds__(HOPS ? 256 : 64) k_site_canon(CanonArgs a) {
  constexpr int NW = HOPS ? (TIME ? 4 : 3) : 1;
  __shared__ cx<double> sum[HOPS ? NW * 12 * kSub : 1];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const SubSite ss = sub_site(a.g, lane);
  const C3 c = p3_coords(a.g, ss.p, ss.s);
  const CPt q = canon_point(a.g, c.x, c.y, c.z, ss.t);
  cx<double> out[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) out[k] = czero<double>();
  if (!HOPS || wave == 3) {
    cx<double> psi[12];
    ld_canon<G5, 12>(a.src, q.n, 0, psi);
#pragma unroll
    for (int k = 0; k < 12; ++k) out[k] = a.c_mu * psi[k];
    if constexpr (CLOV) {
      cx<double> ap[12];
      clover_apply<double, double2, int64_t>(a.clov + (int64_t)q.p * 36 * a.g.V2, a.g.V2, q.i, psi, ap);
#pragma unroll
      for (int k = 0; k < 12; ++k) out[k] += a.c_A * ap[k];
    }
    if constexpr (HOPS && TIME) canon_hop<G5, 3>(a, c, ss.t, q, a.c_t, out);
  } else if (wave == 0) {
    canon_hop<G5, 0>(a, c, ss.t, q, a.c_s, out);
  } else if (wave == 1) {
    canon_hop<G5, 1>(a, c, ss.t, q, a.c_s, out);
  } else {
    canon_hop<G5, 2>(a, c, ss.t, q, a.c_s, out);
  }
  auto store = [&](int k, cx<double> v) {
    // the component that gamma5 moves k to
    const int o = G5 ? (k < 6 ? k + 6 : k - 6) : k;
    a.dst[q.n * 12 + o] = G5 ? make_double2(-v.re, -v.im) : make_double2(v.re, v.im);
  };
  if constexpr (!HOPS) {
    if (ss.ok) {
#pragma unroll
      for (int k = 0; k < 12; ++k) store(k, out[k]);
    }
  } else {
#pragma unroll
    for (int k = 0; k < 12; ++k) sum[(wave * 12 + k) * kSub + lane] = out[k];
    __syncthreads();
    if (!ss.ok) return;
#pragma unroll
    for (int r = 0; r < 12 / NW; ++r) {
      const int k = wave * (12 / NW) + r;
      cx<double> v = sum[k * kSub + lane];
#pragma unroll
      for (int w = 1; w < NW; ++w) v += sum[(w * 12 + k) * kSub + lane];
      store(k, v);
    }
  }
}

template <bool G5>
void canon_go(tp_ctx ctx, const CanonArgs& a, bool hops, bool time) {
  const dim3 grid(sub_blocks(ctx->lat));
  const bool cl = a.clov != nullptr;
  if (hops && time) {
    if (cl) hipLaunchKernelGGL((k_site_canon<G5, true, true, true>), grid, dim3(256), 0, ctx->stream, a);
    else hipLaunchKernelGGL((k_site_canon<G5, true, true, false>), grid, dim3(256), 0, ctx->stream, a);
  } else if (hops) {
    hipLaunchKernelGGL((k_site_canon<G5, true, false, false>), grid, dim3(192), 0, ctx->stream, a);
  } else {
    hipLaunchKernelGGL((k_site_canon<G5, false, false, true>), grid, dim3(64), 0, ctx->stream, a);
  }
  LAUNCH_CHECK();
}

}  // namespace

void launch_site_canon(tp_op op, const double2* src, double2* dst, bool g5, SiteCoef cf, const double2* clov) {
  tp_ctx ctx = op->g->ctx;
  const Lattice& L = ctx->lat;
  CanonArgs a{src, dst, op->g->u4_d, clov, cf.c_mu, cf.c_A, cf.c_t, cf.c_s, L.g};
  const bool hops = cf.c_s != 0.0, time = cf.c_t != 0.0;
  if (!hops && !clov) TP_THROW(TP_EINVAL, "site apply without a term");
  ProfScope ps(ctx, KID_SITE_P3, double(L.V) * (2 * 192 + (hops ? 3 * 144 : 0) + (time ? 144 : 0) + (clov ? 576 : 0)));
  if (g5) canon_go<true>(ctx, a, hops, time);
  else canon_go<false>(ctx, a, hops, time);
}
