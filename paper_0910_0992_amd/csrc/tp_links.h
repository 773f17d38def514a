// 3x3 matrix products, link loads from the layouts' planes and the site order of the kernels
// that walk the links: set-up (k_setup.hip) and the link gradient (k_force.hip).
#pragma once
#include "tp_internal.h"

TP_DEV void mm3(const cx<double>* a, const cx<double>* b, cx<double>* c) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      cx<double> s = cmul(a[3 * i], b[j]);
      s += cmul(a[3 * i + 1], b[3 + j]);
      s += cmul(a[3 * i + 2], b[6 + j]);
      c[3 * i + j] = s;
    }
}

TP_DEV void dag3(const cx<double>* a, cx<double>* b) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) b[3 * i + j] = conj(a[3 * j + i]);
}
// U_mu(x) from the planes [4 dir][2 parity][9][V2] of a layout: p3 (the axial frame) when AX,
// else p4 (the original frame).  The phase b folded into U_t(Lt-1) cancels in closed loops.
template <bool AX>
TP_DEV void load_soa(const double2* __restrict__ u, const Geom& g, int mu, int x, int y, int z, int t,
                     cx<double>* m) {
  x = x < 0 ? x + g.Lx : (x >= g.Lx ? x - g.Lx : x);
  y = y < 0 ? y + g.Ly : (y >= g.Ly ? y - g.Ly : y);
  z = z < 0 ? z + g.Lz : (z >= g.Lz ? z - g.Lz : z);
  t = t < 0 ? t + g.Lt : (t >= g.Lt ? t - g.Lt : t);
  const int s = p3_index(g, x, y, z), p = AX ? (x + y + z) & 1 : (x + y + z + t) & 1;
  const int64_t i = AX ? p3_idx(g, t, s) : s + (int64_t)g.Vs2 * t;
  const double2* src = u + (int64_t)(mu * 2 + p) * 9 * g.V2 + i;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const double2 e = src[(int64_t)k * g.V2];
    m[k] = cx<double>{e.x, e.y};
  }
}

// The kernels that walk the links (set-up, plaquette, link gradient) work on sub-blocks of 16 spatial indices x 4 time slices of one p3
// parity: 64 sites that are runs of 256 bytes both in the p4 planes (s fastest) and in the p3
// planes (four tiles of 4 lines x 4 slices).  Workgroups go to the 8 XCDs in turn; each XCD takes
// one contiguous part of the sequence parity, s, t (fastest first), so that a site's neighbours
// in x, y and z were read through the same L2 at most one z plane x 4 slices (1.3 MB of links at
// 24^2) earlier.
constexpr int kSub = 64;
struct SubSite {
  int p, s, t;
  bool ok;  // false past the lattice's ends: s and t are then those of the last valid site
};
inline unsigned sub_blocks(const Lattice& L) { return 2u * unsigned((L.Vs2 + 15) / 16) * unsigned((L.L[3] + 3) / 4); }
// The id-th sub-block of the sequence.
TP_DEV SubSite sub_site_at(const Geom& g, uint32_t id, int lane) {
  const uint32_t blk = id >> 1, nsb = uint32_t(g.Vs2 + 15) / 16;
  const int s = int(blk % nsb) * 16 + (lane & 15), t = int(blk / nsb) * 4 + (lane >> 4);
  SubSite q;
  q.p = int(id & 1u);
  q.ok = s < g.Vs2 && t < g.Lt;
  q.s = s < g.Vs2 ? s : g.Vs2 - 1;
  q.t = t < g.Lt ? t : g.Lt - 1;
  return q;
}
// That of a workgroup, for launches of one workgroup per sub-block.
TP_DEV SubSite sub_site(const Geom& g, int lane) { return sub_site_at(g, xcd_block(blockIdx.x, gridDim.x), lane); }
