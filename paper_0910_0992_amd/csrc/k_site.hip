// Site-parallel stencil kernels: the fermion matrix and its pieces on the p3
// ("line") layout and the 4D even-odd Schur pieces on the p4 layout.  One thread per output
// site; spin projection in the Dirac-Pauli basis (only two colour matvecs per hop direction).
#include <type_traits>

#include "tp_internal.h"
#include "tp_hop.h"

namespace {

constexpr int kBlock = 256;

// Order in which the workgroups visit the chunks of 256 sites and the right-hand sides.
// Workgroups go to the 8 XCDs (each with its own L2) in turn, so workgroup b runs on XCD b % 8.
//   tiles: a launch of one workgroup per chunk whose chunks are whole parts of the tiles of 4
//     lines (Q = Lt / 64 chunks each): XCD x takes the time range x % Q of the tiles in part
//     x / Q of a z-blocked tile sequence (x fastest, then z inside blocks of BZ planes, then y,
//     then the z block), so that the tiles holding a site's x, y and z neighbours were visited by
//     the same XCD 1, TX*BZ and TX workgroups earlier;
//   parts: each XCD takes one contiguous part of the chunks, in memory order, and every
//     right-hand side of a chunk: y and z neighbours are then in its L2 as long as it holds the
//     sites of one z plane;
//   plain: in turn.
enum { kOrderPlain = 0, kOrderTiles = 1, kOrderParts = 2 };
struct TileOrder {
  uint32_t Q, TX, Ly, BZ, per_part;
  int mode;
};

TP_DEV uint32_t tile_block(const TileOrder& o, uint32_t b) {
  const uint32_t x = b & 7u, n = b >> 3;
  const uint32_t q = (x / o.Q) * o.per_part + n;
  const uint32_t tx = q % o.TX;
  uint32_t r = q / o.TX;
  const uint32_t zi = r % o.BZ;
  r /= o.BZ;
  const uint32_t y = r % o.Ly, zb = r / o.Ly;
  const uint32_t tile = tx + o.TX * (y + o.Ly * (zb * o.BZ + zi));
  return tile * o.Q + x % o.Q;
}

// Measured rules.  Tiles, against plain: 4-19% faster hops in F32 and F16N at 16^3x128, 24^3x128
// and (F32) 32^3x256, but 2-5% slower for FP16 storage with four chunks per tile (256-slice
// lines), which keeps the plain order.  Parts, where the launch has no whole tiles, while the
// neighbour spinors of a plane stay below
//   6 MB without the clover term: D_s, plain and parts in us, F32 14x14x12x107 27.6 and 16.3, F64
//     24^3x84 (4.6 MB) 179 and 153, 24^3x107 (5.9 MB) 239 and 198, F16N 32^3x160 (4.6 MB) 177 and 171
//     (batches of 12 right-hand sides, F16N 16^3x128, 11 MB: 117 and 121);
//   4.2 MB (FP16 storage: 2.5 MB) with it, whose blocks pass through the same L2: D_s and A, F64 24^3x72
//     (4.0 MB) gains 5%, 24^3x84 (4.6 MB) 252 and 250 or 243 and 248, 32^3x60 (5.9 MB) 397 and 432; F32
//     32^3x75 (3.7 MB) 259 and 254, 32^3x88 (4.3 MB) 299 and 304; F16N 32^3x80 (2.3 MB) 138 and 132, 48^3x40
//     (2.6 MB) 210 and 223, 40^3x80 (3.6 MB) 265 and 281.
TileOrder tile_order(const Lattice& L, int64_t nblocks, int nr, double spinor, bool clov) {
  TileOrder o{1, 1, 1, 1, 0, kOrderPlain};
  const Geom& g = L.g;
  const double most = !clov || nr != 1 ? 6e6 : (spinor < 60 ? 2.5e6 : 4.2e6);
  if (double(g.Lxh) * g.Ly * g.Lt * nr * spinor <= most) o.mode = kOrderParts;
  if (nr != 1 || int64_t(nblocks) * kBlock != g.V2) return o;
  if (g.Lt % 64 || (8 % (g.Lt / 64)) || g.Lxh % kTile) return o;
  const uint32_t Q = uint32_t(g.Lt / 64), tiles = uint32_t(g.Vs2 / kTile);
  if ((uint64_t(tiles) * Q) % 8) return o;
  o.Q = Q;
  o.TX = uint32_t(g.Lxh / kTile);
  o.Ly = uint32_t(g.Ly);
  o.BZ = g.Lz % 8 == 0 ? 8u : g.Lz % 4 == 0 ? 4u : g.Lz % 2 == 0 ? 2u : 1u;
  o.per_part = tiles * Q / 8;
  o.mode = spinor < 60 && Q >= 4 ? kOrderPlain : kOrderTiles;
  return o;
}

template <typename S>
struct SiteArgsP3 {
  // for output parity p: self[p] (parity p operand of mu, A, D_t), nb[p] (parity 1-p
  // operand of D_s), in2[p]
  SpinorF<S> self[2], nb[2], dst[2], in2[2];
  LinkF<typename Prec<S>::L> u[2][4];  // [parity][direction]
  const typename Prec<S>::L* clov[2];
  double c_mu, c_A, c_t, c_s, c_in;
  Geom g;
  int par;  // output parity of this launch
  int nr;   // right-hand sides
  double* partial;
  TileOrder ord;
};

// DS: 0 = no spatial hop, 3 = spatial links read whole, 2 = read as two rows (SU(3))
template <typename S, bool DT, int DS, bool CLOV, bool IN2, bool NORM>
__global__ void __launch_bounds__(kBlock) k_site_p3(SiteArgsP3<S> a) {
  using R = typename Prec<S>::R;
  using Lt = typename Prec<S>::L;
  __shared__ double red[kBlock / 64];
  double acc = 0.0;
  const int p = a.par;  // one parity per launch: every field plane address is uniform
  const uint32_t nr = uint32_t(a.nr), nblk = gridDim.x / nr;
  const uint32_t id = a.ord.mode == kOrderTiles   ? tile_block(a.ord, blockIdx.x)
                      : a.ord.mode == kOrderParts ? xcd_block(blockIdx.x, gridDim.x)
                                                  : blockIdx.x;
  const uint32_t rhs = id % nr, first = id / nr;
  const SpinorF<S> self = rhs_view(a.self[p], rhs), nbf = rhs_view(a.nb[p], rhs);
  const SpinorF<S> in2 = rhs_view(a.in2[p], rhs), dst = rhs_view(a.dst[p], rhs);
  for (uint32_t i = first * blockDim.x + threadIdx.x; i < uint32_t(a.g.V2); i += nblk * blockDim.x) {
    int t, s;
    p3_ts32(a.g, i, t, s);
    cx<R> out[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) out[c] = czero<R>();
    if (a.c_mu != 0.0 || CLOV) {
      cx<R> psi[12];
      load_spinor<S, R>(self, i, psi);
      R cm = R(a.c_mu);
#pragma unroll
      for (int c = 0; c < 12; ++c) out[c] = cm * psi[c];
      if constexpr (CLOV) {
        cx<R> ap[12];
        clover_apply<R, Lt>(a.clov[p], a.g.V2, i, psi, ap);
        R ca = R(a.c_A);
#pragma unroll
        for (int c = 0; c < 12; ++c) out[c] += ca * ap[c];
      }
    }
    if constexpr (DT) {
      hop_time_p3<S, R, Lt>(self, a.u[p][3], a.g, t, s, R(a.c_t), out);
    }
    if constexpr (DS != 0) {
      hop_space_p3<S, R, Lt, DS>(nbf, a.u[p], a.u[1 - p], a.g, p, t, s, R(0.5 * a.c_s), out);
    }
    if constexpr (IN2) {
      cx<R> e[12];
      load_spinor<S, R>(in2, i, e);
      R ci = R(a.c_in);
#pragma unroll
      for (int c = 0; c < 12; ++c) out[c] += ci * e[c];
    }
    if constexpr (NORM) {
#pragma unroll
      for (int c = 0; c < 12; ++c) acc += double(norm2(out[c]));
    }
    store_spinor<S, R>(dst, i, out);
  }
  if constexpr (NORM) {
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      double s = 0;
      for (int w = 0; w < kBlock / 64; ++w) s += red[w];
      a.partial[(int64_t)blockIdx.x * 8] = s;
    }
  }
}

// The same for launches too small to fill the card, one wavefront per hop: wavefront 0 holds the
// output sites (64 a workgroup) with the terms of the site itself, wavefronts 1..6 bring the six
// spatial hops' half spinors to LDS, two more the time hops'; wavefront 0 then adds them in
// k_site_p3's order, so that the results are the same bits.
template <bool DT> constexpr int split_waves() { return DT ? 9 : 7; }

template <typename S, bool DT, int DS, bool CLOV, bool IN2>
__global__ void __launch_bounds__(64 * split_waves<DT>()) k_site_split(SiteArgsP3<S> a) {
  using R = typename Prec<S>::R;
  using Lt = typename Prec<S>::L;
  __shared__ cx<R> hop[(split_waves<DT>() - 1) * 6 * 64];
  const int p = a.par;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t nr = uint32_t(a.nr), id = xcd_block(blockIdx.x, gridDim.x);
  const uint32_t rhs = id % nr, V2 = uint32_t(a.g.V2);
  const uint32_t at = id / nr * 64 + uint32_t(lane);
  const uint32_t i = at < V2 ? at : V2 - 1;  // lanes past the end repeat the last site, unstored
  int t, s;
  p3_ts32(a.g, i, t, s);
  cx<R> out[12], e[12];
  if (wave == 0) {
    const SpinorF<S> self = rhs_view(a.self[p], rhs);
    if constexpr (IN2) load_spinor<S, R>(rhs_view(a.in2[p], rhs), i, e);
#pragma unroll
    for (int c = 0; c < 12; ++c) out[c] = czero<R>();
    if (a.c_mu != 0.0 || CLOV) {
      cx<R> psi[12];
      load_spinor<S, R>(self, i, psi);
      R cm = R(a.c_mu);
#pragma unroll
      for (int c = 0; c < 12; ++c) out[c] = cm * psi[c];
      if constexpr (CLOV) {
        cx<R> ap[12];
        clover_apply<R, Lt>(a.clov[p], a.g.V2, i, psi, ap);
        R ca = R(a.c_A);
#pragma unroll
        for (int c = 0; c < 12; ++c) out[c] += ca * ap[c];
      }
    }
  } else {
    cx<R> w[6];
    const SpinorF<S> nb = rhs_view(a.nb[p], rhs);
    const HopIdx x = hop_idx(a.g, p, t, s);
    switch (wave) {
      case 1: hop_half<0, true, S, R, Lt, DS>(nb, x.j[0], a.u[p][0], i, w); break;
      case 2: hop_half<0, false, S, R, Lt, DS>(nb, x.j[1], a.u[1 - p][0], x.j[1], w); break;
      case 3: hop_half<1, true, S, R, Lt, DS>(nb, x.j[2], a.u[p][1], i, w); break;
      case 4: hop_half<1, false, S, R, Lt, DS>(nb, x.j[3], a.u[1 - p][1], x.j[3], w); break;
      case 5: hop_half<2, true, S, R, Lt, DS>(nb, x.j[4], a.u[p][2], i, w); break;
      case 6: hop_half<2, false, S, R, Lt, DS>(nb, x.j[5], a.u[1 - p][2], x.j[5], w); break;
      default:
        if constexpr (DT) hop_time_half<S, R, Lt>(rhs_view(a.self[p], rhs), a.u[p][3], a.g, t, s, wave == 7, w);
    }
#pragma unroll
    for (int c = 0; c < 6; ++c) hop[((wave - 1) * 6 + c) * 64 + lane] = w[c];
  }
  __syncthreads();
  if (wave != 0 || at >= V2) return;
  auto take = [&](int h, cx<R>* w) {
#pragma unroll
    for (int c = 0; c < 6; ++c) w[c] = hop[(h * 6 + c) * 64 + lane];
  };
  cx<R> w[6];
  if constexpr (DT) {
    const R ct = R(a.c_t);
    take(6, w);
#pragma unroll
    for (int c = 0; c < 6; ++c) out[6 + c] += ct * w[c];
    take(7, w);
#pragma unroll
    for (int c = 0; c < 6; ++c) out[c] += ct * w[c];
  }
  const R cs = R(0.5 * a.c_s);
  take(0, w); recon_minus<0, R>(out, w, cs);
  take(1, w); recon_plus<0, R>(out, w, cs);
  take(2, w); recon_minus<1, R>(out, w, cs);
  take(3, w); recon_plus<1, R>(out, w, cs);
  take(4, w); recon_minus<2, R>(out, w, cs);
  take(5, w); recon_plus<2, R>(out, w, cs);
  if constexpr (IN2) {
    R ci = R(a.c_in);
#pragma unroll
    for (int c = 0; c < 12; ++c) out[c] += ci * e[c];
  }
  store_spinor<S, R>(rhs_view(a.dst[p], rhs), i, out);
}

// ---- 4D even-odd Schur (p4 layout) ---------------------------------------------------------
template <typename S>
struct ArgsP4 {
  SpinorF<S> src, dst, in2;  // src on parity 1-p; dst and in2 on parity p
  LinkF<typename Prec<S>::L> u[2][4];
  const typename Prec<S>::L* clov;  // blocks on parity p
  double c_h, c_in, inv_gf;
  Geom g;
  int p;
  int parts;  // each XCD takes a contiguous part of the sites (else workgroups in memory order)
};

// CL: 0 none; 1 clover applied to (c_in*in2 + c_h*D_w src); 2 clover applied to in2,
// then + c_h*D_w src.
template <typename S, bool HOP, bool IN2, int CL>
__global__ void __launch_bounds__(kBlock) k_schur4d(ArgsP4<S> a) {
  using R = typename Prec<S>::R;
  using Lt = typename Prec<S>::L;
  int64_t i = (int64_t)(a.parts ? xcd_block(blockIdx.x, gridDim.x) : blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= a.g.V2) return;
  cx<R> v[12];
#pragma unroll
  for (int c = 0; c < 12; ++c) v[c] = czero<R>();
  if constexpr (IN2) {
    cx<R> e[12];
    load_spinor<S, R>(a.in2, i, e);
    if constexpr (CL == 2) {
      clover_apply<R, Lt>(a.clov, a.g.V2, i, e, v);
    } else {
      R ci = R(a.c_in);
#pragma unroll
      for (int c = 0; c < 12; ++c) v[c] = ci * e[c];
    }
  }
  if constexpr (HOP) {
    hop_4d_p4<S, R, Lt>(a.src, a.u[a.p], a.u[1 - a.p], a.g, a.p, i, R(a.c_h), R(a.c_h * a.inv_gf), v);
  }
  if constexpr (CL == 1) {
    cx<R> w[12];
    clover_apply<R, Lt>(a.clov, a.g.V2, i, v, w);
    store_spinor<S, R>(a.dst, i, w);
  } else {
    store_spinor<S, R>(a.dst, i, v);
  }
}

template <typename S>
SpinorF<S> view(const Field* f, int p) {
  if (!f) {
    SpinorF<S> z;
    z.p[0] = z.p[1] = nullptr;
    z.stride = 0;
    return z;
  }
  return f->template par<S>(p);
}

template <typename S>
struct LinkSrc;
template <> struct LinkSrc<double2> {
  static const double2* get(tp_gauge g, bool l4) { return l4 ? g->u4_d : g->u3_d; }
};
template <> struct LinkSrc<float2> {
  static const float2* get(tp_gauge g, bool l4) { return l4 ? g->u4_f : g->u3_f; }
};
template <> struct LinkSrc<__half2> {
  // F16N runs only in the p3 layout (the 4D scheme is F64/F32)
  static const __half2* get(tp_gauge g, bool l4) { return l4 ? nullptr : g->u3_h; }
};

template <typename S>
void fill_links(tp_gauge g, bool l4, LinkF<typename Prec<S>::L> (&u)[2][4], int64_t V2) {
  const typename Prec<S>::L* base = LinkSrc<S>::get(g, l4);
  for (int p = 0; p < 2; ++p)
    for (int d = 0; d < 4; ++d) {
      u[p][d].p = base + (int64_t)(d * 2 + p) * 9 * V2;
      u[p][d].stride = V2;
    }
}

template <typename S>
const typename Prec<S>::L* clover_base(tp_op op, int kind, bool l4);
template <> const double2* clover_base<double2>(tp_op op, int kind, bool l4) {
  if (kind == 1) return op->c ? (l4 ? op->c->a4_d : op->c->a3_d) : nullptr;
  if (kind == 2) return l4 ? op->a4_mu : op->a3_mu;
  if (kind == 3) return l4 ? op->a4_inv : op->a3_inv;
  return nullptr;
}
template <> const float2* clover_base<float2>(tp_op op, int kind, bool l4) {
  if (kind == 1) return op->c ? (l4 ? op->c->a4_f : op->c->a3_f) : nullptr;
  if (kind == 2) return l4 ? op->a4_mu_f : op->a3_mu_f;
  if (kind == 3) return l4 ? op->a4_inv_f : op->a3_inv_f;
  return nullptr;
}
template <> const __half2* clover_base<__half2>(tp_op op, int kind, bool l4) {
  if (l4) return nullptr;
  if (kind == 1) return op->c ? op->c->a3_h : nullptr;
  if (kind == 2) return op->a3_mu_h;
  if (kind == 3) return op->a3_inv_h;
  return nullptr;
}

// Up to two workgroups of k_site_split a CU (64 sites each): k_site_p3 has less than one wavefront
// a SIMD there and waits for one hop after another.  k_site_p3 and k_site_split, D_s alone / with the
// clover term, in us: FP64 4^3x16 9.1 / 10.4 and 5.0 / 5.2, 8^3x64 12.2 / 14.0 and 6.8 / 7.4,
// 10^3x64 15.6 / 18.0 and 9.9 / 14.2, 12x12x8x64 14.2 / 17.4 and 12.2 / 17.7, 12^3x64 15.4 / 20.4
// and 15.1 / 24.1; FP32 (alone) 6.1 and 4.6, 10^3x64 9.1 and 6.1, 12^3x64 9.7 and 9.1, 16^3x64 14.1
// and 15.8; FP16 6.0 / 6.8 and 4.7 / 4.4, 10^3x64 7.9 / 8.7 and 5.7 / 5.7, 16^3x64 12.2 / 14.0 and
// 13.3 / 16.1.  Not with a fused norm, whose partial sums are k_site_p3's.
constexpr int64_t kSplitSites = 1 << 15;

template <typename S, bool DT, int DS, bool CLOV, bool IN2, bool NORM>
void site_go(tp_op op, SiteArgsP3<S> a, int64_t nblocks, int par0, int npar) {
  tp_ctx ctx = op->g->ctx;
  for (int q = 0; q < npar; ++q) {
    a.par = par0 + q;
    a.partial = ctx->red_partial + (int64_t)q * nblocks * 8;
    if constexpr (DS != 0 && !NORM) {
      if (a.g.V2 * a.nr <= kSplitSites) {
        hipLaunchKernelGGL((k_site_split<S, DT, DS, CLOV, IN2>), dim3(unsigned((a.g.V2 + 63) / 64 * a.nr)),
                           dim3(64 * split_waves<DT>()), 0, ctx->stream, a);
        LAUNCH_CHECK();
        continue;
      }
    }
    hipLaunchKernelGGL((k_site_p3<S, DT, DS, CLOV, IN2, NORM>), dim3((unsigned)(nblocks * a.nr)), dim3(kBlock),
                       0, ctx->stream, a);
    LAUNCH_CHECK();
  }
}

template <typename S, bool DT, int DS, bool CLOV>
void site_in2(tp_op op, SiteArgsP3<S>& a, int64_t nb, bool in2, bool norm, int par0, int npar) {
  if (in2) {
    if (norm) site_go<S, DT, DS, CLOV, true, true>(op, a, nb, par0, npar);
    else site_go<S, DT, DS, CLOV, true, false>(op, a, nb, par0, npar);
  } else {
    if (norm) site_go<S, DT, DS, CLOV, false, true>(op, a, nb, par0, npar);
    else site_go<S, DT, DS, CLOV, false, false>(op, a, nb, par0, npar);
  }
}

template <typename S>
SpinorF<S> halves(const Field* up, const Field* lo, int p) {
  SpinorF<S> a = view<S>(up, p), b = view<S>(lo, p);
  a.p[1] = b.p[1];
  if (!up) a.stride = b.stride;
  return a;
}

template <typename S>
int site_t(tp_op op, const SiteIO& io, Field& dst, SiteCoef cf, int ck, int par0, int npar, bool norm) {
  tp_ctx ctx = op->g->ctx;
  const Lattice& L = ctx->lat;
  const Field* in2 = io.in2;
  SiteArgsP3<S> a;
  for (int p = 0; p < 2; ++p) {
    a.self[p] = halves<S>(io.self_up, io.self_lo, p);
    a.nb[p] = halves<S>(io.nb_up, io.nb_lo, 1 - p);
    a.dst[p] = view<S>(&dst, p);
    a.in2[p] = view<S>(in2, p);
  }
  fill_links<S>(op->g, false, a.u, L.V2);
  const typename Prec<S>::L* cb = clover_base<S>(op, ck, false);
  bool clov = cb != nullptr && cf.c_A != 0.0;
  for (int p = 0; p < 2; ++p) a.clov[p] = cb ? cb + (int64_t)p * 36 * L.V2 : nullptr;
  a.c_mu = cf.c_mu;
  a.c_A = cf.c_A;
  a.c_t = cf.c_t;
  a.c_s = cf.c_s;
  a.c_in = cf.c_in;
  a.g = L.g;
  // one launch per output parity; with a norm, each launch's partials follow the previous
  a.nr = dst.nr;
  if (norm && a.nr != 1) TP_THROW(TP_EINVAL, "a fused norm needs a single right-hand side");
  int64_t nb = (L.V2 + kBlock - 1) / kBlock;
  if (norm) nb = std::min<int64_t>(nb, kRedBlocks / 2);
  a.ord = tile_order(L, nb, a.nr, 2.0 * Field::half_bytes(dst.prec), clov);
  bool dt = cf.c_t != 0.0, ds = cf.c_s != 0.0;
  bool i2 = in2 != nullptr;
  // spatial hops read SU(3) links as two rows (FP64: only links SU(3) to 1e-13)
  constexpr bool kReduced = !std::is_same<S, double2>::value;
  const bool two = kReduced ? op->g->su3_spatial : op->g->su3_spatial_f64;
  if (dt && ds) {
    if (two) {
      if (clov) site_in2<S, true, 2, true>(op, a, nb, i2, norm, par0, npar);
      else site_in2<S, true, 2, false>(op, a, nb, i2, norm, par0, npar);
    } else {
      if (clov) site_in2<S, true, 3, true>(op, a, nb, i2, norm, par0, npar);
      else site_in2<S, true, 3, false>(op, a, nb, i2, norm, par0, npar);
    }
  } else if (ds) {
    if (two) {
      if (clov) site_in2<S, false, 2, true>(op, a, nb, i2, norm, par0, npar);
      else site_in2<S, false, 2, false>(op, a, nb, i2, norm, par0, npar);
    } else {
      if (clov) site_in2<S, false, 3, true>(op, a, nb, i2, norm, par0, npar);
      else site_in2<S, false, 3, false>(op, a, nb, i2, norm, par0, npar);
    }
  } else if (dt) {
    if (clov) site_in2<S, true, 0, true>(op, a, nb, i2, norm, par0, npar);
    else site_in2<S, true, 0, false>(op, a, nb, i2, norm, par0, npar);
  } else {
    if (clov) site_in2<S, false, 0, true>(op, a, nb, i2, norm, par0, npar);
    else site_in2<S, false, 0, false>(op, a, nb, i2, norm, par0, npar);
  }
  return norm ? int(nb * npar) : 0;
}

template <typename S, bool HOP, bool IN2, int CL>
void s4_go(tp_ctx ctx, ArgsP4<S>& a) {
  unsigned nb = (unsigned)((a.g.V2 + kBlock - 1) / kBlock);
  hipLaunchKernelGGL((k_schur4d<S, HOP, IN2, CL>), dim3(nb), dim3(kBlock), 0, ctx->stream, a);
  LAUNCH_CHECK();
}

template <typename S>
void schur4d_t(tp_op op, int mode, int p, const Field* src, Field& dst, const Field* in2, double c_h,
               double c_in, int ck) {
  tp_ctx ctx = op->g->ctx;
  const Lattice& L = ctx->lat;
  ArgsP4<S> a;
  a.src = view<S>(src, 1 - p);
  a.dst = view<S>(&dst, p);
  a.in2 = view<S>(in2, p);
  fill_links<S>(op->g, true, a.u, L.V2);
  const typename Prec<S>::L* cb = clover_base<S>(op, ck, true);
  a.clov = cb ? cb + (int64_t)p * 36 * L.V2 : nullptr;
  a.c_h = c_h;
  a.c_in = c_in;
  a.inv_gf = 1.0 / op->gf;
  a.g = L.g;
  a.p = p;
  // Each XCD takes a contiguous part while its L2 holds the neighbour slices' spinors, up to 2 MB a
  // slice and parity.  Parts against memory order, F64: 16^3x128 (0.4 MB) 153 -> 125 us, 24^3x128 (1.3
  // MB) 425 -> 408 us, but 32^3x128 (3.1 MB) 1010 -> 1045 us.
  a.parts = double(L.Vs2) * 2.0 * Field::half_bytes(dst.prec) <= 2e6;
  switch (mode) {
    case 0: s4_go<S, true, false, 1>(ctx, a); break;
    case 1: s4_go<S, true, true, 2>(ctx, a); break;
    case 2: s4_go<S, true, true, 0>(ctx, a); break;
    case 3: s4_go<S, true, true, 1>(ctx, a); break;
    default: s4_go<S, false, true, 2>(ctx, a); break;
  }
}

}  // namespace

int launch_site(tp_op op, int prec, const SiteIO& io, Field& dst, SiteCoef cf, int ck, int par0,
                int npar, bool norm) {
  tp_ctx ctx = op->g->ctx;
  const Lattice& L = ctx->lat;
  double S = spinor_bytes(prec), Lb = link_bytes(prec), C = clov_bytes(prec);
  // spatial links read as two rows (12 reals) when they are SU(3) (to 1e-13 for FP64)
  double Ls = (prec != TP_F64 ? op->g->su3_spatial : op->g->su3_spatial_f64) ? Lb * 2 / 3 : Lb;
  bool self = cf.c_mu != 0 || (ck && cf.c_A != 0);
  // spinor bytes per right-hand side; links and clover once for a whole batch
  double sp = S + (self ? S : 0) + (cf.c_s != 0 ? S : 0) + (cf.c_t != 0 ? S : 0) + (io.in2 ? S : 0);
  double lk = (cf.c_s != 0 ? 6 * Ls : 0) + (cf.c_t != 0 ? 2 * Lb : 0) + (ck && cf.c_A != 0 ? C : 0);
  double bytes = double(npar) * L.V2 * (dst.nr * sp + lk);
  // the time-line pipeline's stencils are accounted separately from M / residual applies
  const int kid = cf.c_t != 0 || io.in2 ? KID_SITE_P3 : (ck && cf.c_A != 0 ? KID_HOP_CLOVER : KID_HOP_DS);
  ProfScope ps(ctx, kid, bytes);
  switch (prec) {
    case TP_F64: return site_t<double2>(op, io, dst, cf, ck, par0, npar, norm);
    case TP_F32: return site_t<float2>(op, io, dst, cf, ck, par0, npar, norm);
    default: return site_t<__half2>(op, io, dst, cf, ck, par0, npar, norm);
  }
}

int launch_site_p3(tp_op op, int prec, const Field& src, Field& dst, const Field* in2, SiteCoef cf,
                   int ck, int par0, int npar, bool norm) {
  SiteIO io;
  io.self_up = io.self_lo = io.nb_up = io.nb_lo = &src;
  io.in2 = in2;
  return launch_site(op, prec, io, dst, cf, ck, par0, npar, norm);
}

void launch_schur4d(tp_op op, int prec, int mode, int p, const Field* src, Field& dst, const Field* in2,
                    double c_h, double c_in, int ck) {
  tp_ctx ctx = op->g->ctx;
  const Lattice& L = ctx->lat;
  double S = 2.0 * Field::half_bytes(prec);
  double Lb = prec == TP_F64 ? 144 : 72;
  double C = prec == TP_F64 ? 576 : 288;
  double bytes = double(L.V2) * (S + (mode != 4 ? S + 8 * Lb : 0) + (in2 ? S : 0) + (ck ? C : 0));
  ProfScope ps(ctx, mode == 0 ? KID_SCHUR4D_EO : KID_SCHUR4D_OE, bytes);
  switch (prec) {
    case TP_F64: schur4d_t<double2>(op, mode, p, src, dst, in2, c_h, c_in, ck); break;
    default: schur4d_t<float2>(op, mode, p, src, dst, in2, c_h, c_in, ck); break;
  }
}
