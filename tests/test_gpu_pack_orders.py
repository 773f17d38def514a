"""Canonical fields into the internal layouts, in every order of the sites (sub-blocks, canonical
order and its parts), at the lengths of a line and sizes between which the order changes.

Tolerances: into the 4D layout and back is a permutation in FP64, exact.  Into the axial frame and back
is two 3x3 rotations of unitary matrices known to 1e-15 (1e-13 leaves two orders for long products of
links), plus the storage's rounding: 2^-24 per value in FP32, 2^-11 of a half spinor's largest in F16N
(1e-6 and 2e-3 of the norm).
"""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

TOL = {"F64": 1e-13, "F32": 1e-6, "F16N": 2e-3}
# up to 65536 sites sub-blocks; beyond, into p3, canonical order for lines of 5 to 27 slices that are no
# multiple of four and for odd lines of 64 slices or more in fields of more than 256 MB
SMALL = [(2, 2, 2, n) for n in (2, 3, 4, 5, 7, 8)] + [(6, 4, 2, n) for n in (5, 24, 27, 33)] + [(16, 16, 16, 16)]
P3 = [(32, 32, 32, n) for n in (3, 4, 5, 6, 7, 8)] + [(16, 18, 14, n) for n in (17, 26, 27, 28, 29)]
LARGE = [(24, 24, 24, n) for n in (95, 97, 98)]
# into p4 canonical order, in parts up to 2^20 sites
P4 = [(16, 16, 16, 18), (18, 14, 10, 30), (32, 32, 32, 32), (32, 32, 32, 34)]


def _rel(a, b):
    return float((a - b).norm() / b.norm())


@pytest.mark.parametrize("dims", SMALL + P3 + LARGE + P4)
def test_pack_orders(dims):
    from paper_0910_0992_amd import Operator
    print(f"[case] {dims}", flush=True)
    lx, ly, lz, lt = dims
    gen = torch.Generator(device="cuda").manual_seed(5)
    e = torch.view_as_complex(torch.randn((lt, lz, ly, lx, 4, 3, 2), generator=gen, device="cuda", dtype=torch.float64))
    # links of a few distinct matrices, which rotate every line differently
    u = torch.from_numpy(synth.make_links((4, 4, 4, 8), 0.35, 0.2, 1100)[:, :, 0, 0, 0]).cuda().reshape(-1, 3, 3)
    n = torch.randint(0, len(u), (4, lt, lz, ly, lx), generator=gen, device="cuda")
    g = Operator(u[n].contiguous(), 0.05, 3.0, 0.0, 0.0, -1)
    for prec, tol in TOL.items():
        assert _rel(g.from_field(g.to_field(e, "P3", prec))[0], e) < tol, prec
    for dagger in (False, True):  # through the layout, and on the canonical field itself
        assert _rel(g.apply_prec(e, "UNPREC", dagger=dagger), g.apply_M(e, dagger=dagger)) < 1e-12
    if lt % 2 == 0:
        assert torch.equal(g.from_field(g.to_field(e, "P4", "F64"))[0], e)
        assert _rel(g.from_field(g.to_field(e, "P4", "F32"))[0], e) < TOL["F32"]
    g.close()
