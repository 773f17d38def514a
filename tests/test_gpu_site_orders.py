"""The site kernels with a thread per site, on lattices above the limit of those with a wavefront
per hop: every order of their workgroups, links read as two rows and whole, against the FP64
oracle; and the two kinds of kernel against each other.

Tolerances: those of the parity tests (FP64 results re-express the oracle's, 1e-12; FP32 and F16N as
measured margins of the storage: 6e-6 and 4e-3 for one stencil, 2e-5 and 1.5e-2 for composites).
"""
import numpy as np
import pytest
import torch

import synth
from oracle.schemes import Operator as OOp

pytestmark = pytest.mark.gpu

SPLIT_SITES = 1 << 15
TOL = {"F64": (1e-12, 1e-12), "F32": (6e-6, 2e-5), "F16N": (4e-3, 1.5e-2)}
XI, M0, CS, CT = 3.5, -0.05, 1.6 / 3.5, 1.0


def _order(dims, prec, clover):
    """The rule of tile_order for one field: which workgroup order a launch takes."""
    lx, ly, lz, lt = dims
    v2, spinor = int(np.prod(dims)) // 2, {"F64": 192, "F32": 96, "F16N": 56}[prec]
    q = lt // 64
    if v2 % 256 == 0 and lt % 64 == 0 and q and 8 % q == 0 and (lx // 2) % 4 == 0:
        tiles = lx // 2 * ly * lz // 4
        if tiles * q % 8 == 0:
            return "plain" if prec == "F16N" and q >= 4 else "tiles"
    most = 6e6 if not clover else (2.5e6 if prec == "F16N" else 4.2e6)
    return "parts" if lx // 2 * ly * lt * spinor <= most else "plain"


# one, two, four and eight workgroups per tile, two tiles and one per x row, several z blocks; then
# lattices without whole tiles: parts, parts for D_s alone (5.5 MB a plane in FP64) and plain (7.4 MB)
ORDERS = [((16, 8, 12, 64), "tiles", "tiles"), ((16, 8, 8, 128), "tiles", "tiles"), ((16, 4, 8, 256), "tiles", "tiles"),
          ((8, 8, 4, 512), "tiles", "tiles"), ((12, 10, 10, 66), "parts", "parts"), ((24, 24, 2, 100), "parts", "plain"),
          ((24, 24, 2, 134), "plain", "plain")]


@pytest.mark.parametrize("dims,hop,clover", ORDERS)
@pytest.mark.parametrize("links", ["SU(3)", "U(3)"])
def test_site_kernels_in_every_order(dims, hop, clover, links):
    from paper_0910_0992_amd import Operator
    assert int(np.prod(dims)) // 2 > SPLIT_SITES
    assert (_order(dims, "F64", False), _order(dims, "F64", True)) == (hop, clover)
    U = synth.make_links(dims, 0.35, 0.12, 1000)
    if links == "U(3)":
        U[:3] *= np.exp(0.4j)
    o = OOp(U, M0, XI, -1.0, CS, CT)
    g = Operator(torch.from_numpy(U).cuda(), M0, XI, CS, CT, -1)
    eta = synth.make_source(dims, 2000)
    refs = {s: o.prec(s, eta) for s in ("UNPREC", "TEMPORAL_SCHUR")}
    for prec in ("F64", "F32", "F16N"):
        print(f"[order] {dims} {links} {prec} {_order(dims, prec, False)} {_order(dims, prec, True)}", flush=True)
        f = g.to_field(torch.from_numpy(eta).cuda(), "P3", prec)
        for k, (scheme, ref) in enumerate(refs.items()):
            y = g.from_field(g.apply_prec_field(f, scheme))[0].cpu().numpy()
            assert np.linalg.norm(y - ref) < TOL[prec][k] * np.linalg.norm(ref), (prec, scheme)
    g.close()


@pytest.mark.parametrize("links", ["SU(3)", "U(3)"])
@pytest.mark.parametrize("clover", [True, False])
@pytest.mark.parametrize("prec", ["F64", "F32", "F16N"])
def test_a_field_alone_and_in_a_batch(links, clover, prec):
    """Alone the field takes the kernels with a wavefront per hop, in a batch of three those with a
    thread per site: the same bits in F64 and F32.  In F16N the multiply-adds of two-row hops may pair
    differently, which moves a stored value by its last bit: 2^-11 of its half spinor's largest in
    each of the real and the imaginary part (up to twice that where the scale moves as well), mixed
    over three colours on the way out."""
    from paper_0910_0992_amd import Operator
    dims = (8, 8, 8, 64)
    assert int(np.prod(dims)) // 2 <= SPLIT_SITES < 3 * int(np.prod(dims)) // 2
    U = synth.make_links(dims, 0.35, 0.12, 1001)
    if links == "U(3)":
        U[:3] *= np.exp(0.4j)
    print(f"[case] {links} {clover} {prec}", flush=True)
    g = Operator(torch.from_numpy(U).cuda(), M0, XI, CS if clover else 0.0, CT if clover else 0.0, -1)
    etas = torch.stack([torch.from_numpy(synth.make_source(dims, 2010 + k)).cuda() for k in range(3)])
    batch = g.to_field(etas, "P3", prec)
    for scheme in ("UNPREC",) if prec == "F16N" else ("UNPREC", "TEMPORAL", "TEMPORAL_SCHUR"):
        ys = g.from_field(g.apply_prec_field(batch, scheme))
        for k in range(3):
            y = g.from_field(g.apply_prec_field(g.to_field(etas[k], "P3", prec), scheme))[0]
            if prec != "F16N":
                assert torch.equal(y, ys[k]), (scheme, k, float((y - ys[k]).abs().max()))
            else:
                d = (y - ys[k]).abs().unflatten(-2, (2, 2)).amax((-1, -2))
                m = y.abs().unflatten(-2, (2, 2)).amax((-1, -2))
                assert bool((d <= 2 * 6 ** 0.5 * 2 ** -11 * m).all()), float((d / m).max())
                print(f"[last bit] {float((d / m).max()):.2e}", flush=True)
    g.close()
