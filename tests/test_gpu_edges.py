"""Kernels at the edges of their blocks: lattices smaller than a block, and remainders in every
extent that a block splits, against the FP64 oracle.

Tolerance: FP64 results are re-expressions of the oracle's, a few hundred operations of 1.1e-16
deep, so 1e-12 of the field's norm (as for every FP64 apply) leaves two orders of magnitude.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import force as oforce, wilson
from oracle.schemes import Operator as OOp

pytestmark = pytest.mark.gpu

TOL64 = 1e-12


def _make(dims, xi=3.0, m0=0.05, cs=1.6, ct=1.0, bc=-1, seed=1100):
    from paper_0910_0992_amd import Operator
    U = synth.make_links(dims, 0.35, 0.2, seed)
    print(f"[case] {dims}", flush=True)
    return U, OOp(U, m0, xi, float(bc), cs / xi, ct), Operator(torch.from_numpy(U).cuda(), m0, xi, cs / xi, ct, bc)


def _rel(a, b):
    a = a.cpu().numpy()
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _dag(m):
    return np.conj(np.swapaxes(m, -1, -2))


# sub-blocks of the set-up kernels are 16 spatial indices (of one parity) x 4 slices
SUB_DIMS = [(2, 2, 2, 2), (2, 2, 2, 5), (4, 2, 4, 4), (8, 2, 2, 3), (6, 2, 6, 9), (4, 4, 4, 16)]


@pytest.mark.parametrize("dims", SUB_DIMS)
@pytest.mark.parametrize("planes", ["all", "time", "space"])
def test_clover_term(dims, planes):
    """The clover term in the axial frame (apply_clover) and in the original one (the 4D scheme)."""
    U, o, g = _make(dims, cs=0.0 if planes == "time" else 1.6, ct=0.0 if planes == "space" else 1.0)
    eta = synth.make_source(dims, 2100)
    t = torch.from_numpy(eta).cuda()
    for plus in (0, 1, -1):
        ref = {0: o.Aop, 1: o.Amu, -1: o.Amu_inv}[plus](eta)
        assert _rel(g.apply_clover(t, "F64", plus), ref) < TOL64
    if dims[3] % 2 == 0:
        assert _rel(g.apply_prec(t, "SCHUR4D", "F64"), o.prec("SCHUR4D", eta)) < TOL64
    g.close()


@pytest.mark.parametrize("dims", SUB_DIMS)
@pytest.mark.parametrize("bc", [-1, 1])
def test_link_gradient(dims, bc):
    """Raw and projected link gradient, with and without the SW term's part."""
    U, o, g = _make(dims, bc=bc)
    x, lam = synth.make_source(dims, 2101), synth.make_source(dims, 2102)
    tx, tl = torch.from_numpy(x).cuda(), torch.from_numpy(lam).cuda()
    for (raw, proj), only in ((oforce.link_gradient(o, x, lam), True), (oforce.full_link_gradient(o, x, lam), False)):
        assert _rel(g.force(tx, tl, projected=False, hopping_only=only), raw) < TOL64
        assert _rel(g.force(tx, tl, projected=True, hopping_only=only), proj) < TOL64
    g.close()


@pytest.mark.parametrize("dims", SUB_DIMS)
@pytest.mark.parametrize("host", [True, False])
def test_links_and_plaquette(dims, host):
    """Every layout of the links (M in the axial frame and, through the 4D scheme, the original
    one, in F64 and F32) from host and device links, and the plaquette."""
    from paper_0910_0992_amd import Operator
    U = synth.make_links(dims, 0.35, 0.2, 1101)
    o = OOp(U, 0.05, 3.0, -1.0, 0.5, 1.0)
    tu = torch.from_numpy(U)
    g = Operator(tu if host else tu.cuda(), 0.05, 3.0, 0.5, 1.0, -1)
    eta = synth.make_source(dims, 2103)
    t = torch.from_numpy(eta).cuda()
    for prec, tol in (("F64", TOL64), ("F32", 6e-6)):
        assert _rel(g.apply_M(t, prec), o.M(eta)) < tol
        if dims[3] % 2 == 0:
            assert _rel(g.apply_prec(t, "SCHUR4D", prec), o.prec("SCHUR4D", eta)) < tol
    tr = lambda m: np.trace(m, axis1=-2, axis2=-1).real.mean() / 3
    pl = lambda a, b: tr(wilson._chain([U[a], wilson.link_shift(U[b], a, 1), _dag(wilson.link_shift(U[a], b, 1)),
                                        _dag(U[b])]))
    ps, pt = g.plaquette()
    assert abs(ps - (pl(0, 1) + pl(0, 2) + pl(1, 2)) / 3) < 1e-13
    assert abs(pt - (pl(0, 3) + pl(1, 3) + pl(2, 3)) / 3) < 1e-13
    g.close()


# canonical FP64 applies: time extents around the line kernels' chunks (one, two and four slices a
# thread; multiples of 16 and not), line counts that are no multiple of a workgroup's
CANON_DIMS = SUB_DIMS + [(6, 10, 2, 45), (2, 4, 2, 128), (2, 2, 4, 130), (2, 2, 2, 256), (2, 2, 2, 260), (10, 6, 2, 16)]


@pytest.mark.parametrize("dims", CANON_DIMS)
@pytest.mark.parametrize("clover", [True, False])
@pytest.mark.parametrize("cut", [0.0, 1e-3])
def test_canonical_applies(dims, clover, cut):
    """The FP64 applies that work on canonical fields directly, against the oracle and against the
    FP64 path through the internal layout (which overlapping buffers take, as before)."""
    U, o, g = _make(dims, cs=1.6 if clover else 0.0, ct=1.0 if clover else 0.0, bc=1 if dims[0] == 6 else -1)
    eta = synth.make_source(dims, 2104)
    t = torch.from_numpy(eta).cuda()
    calls = {"Tinv": lambda v: g.apply_Tinv(v), "Tdinv": lambda v: g.apply_Tinv(v, dagger=True), "CL": g.apply_CL,
             "CR": g.apply_CR, "prep": lambda v: g.prepare_source(v, "TEMPORAL"),
             "rec": lambda v: g.reconstruct(v, "TEMPORAL")}
    if cut == 0.0:
        refs = {"Tinv": o.tmp.Tinv(eta), "Tdinv": o.tmp.Tdaginv(eta), "CL": o.tmp.CL(eta), "CR": o.tmp.CR(eta)}
        refs.update(prep=refs["CL"], rec=refs["CR"])
        for k, r in refs.items():
            assert _rel(calls[k](t), r) < TOL64, k
        assert _rel(g.apply_M(t), o.M(eta)) < TOL64
        assert _rel(g.apply_M(t, dagger=True), o.Mdag(eta)) < TOL64
        assert _rel(g.apply_prec(t, "UNPREC", dagger=True), o.Mdag(eta)) < TOL64
        assert _rel(g.apply_Ds(t), o.Ds(eta)) < TOL64
        for plus, f in ((1, o.Amu), (-1, o.Amu_inv)) + (((0, o.Aop),) if clover else ()):
            assert _rel(g.apply_clover(t, "F64", plus), f(eta)) < TOL64
    else:
        g.set_cutoff(cut)
    # overlapping buffers: dst starts one site behind src
    n = eta.size
    buf = torch.zeros(n + 12, dtype=torch.complex128, device="cuda")
    import ctypes as C
    L = g._lib
    for name, fn in (("Tinv", lambda d, s: L.tp_apply_Tinv(g._op, 0, d, s, 0)), ("Tdinv", lambda d, s: L.tp_apply_Tinv(g._op, 0, d, s, 1)),
                     ("CL", lambda d, s: L.tp_apply_CL(g._op, 0, d, s)), ("CR", lambda d, s: L.tp_apply_CR(g._op, 0, d, s))):
        buf[:n] = t.reshape(-1)
        assert fn(C.c_void_p(buf[12:].data_ptr()), C.c_void_p(buf.data_ptr())) == 0
        assert _rel(calls[name](t).reshape(-1), buf[12:].cpu().numpy()) < TOL64, name
    buf[:n] = t.reshape(-1)
    assert L.tp_apply_M(g._op, 0, C.c_void_p(buf[12:].data_ptr()), C.c_void_p(buf.data_ptr()), 0) == 0
    assert _rel(g.apply_M(t).reshape(-1), buf[12:].cpu().numpy()) < TOL64
    g.close()


# reductions end in the kernel's last workgroup up to 256 workgroups (8^3 x 64 in FP64) and in a
# launch of their own beyond; single and batched, in every precision
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 4, 4, 8), (8, 8, 8, 64), (8, 8, 8, 66)])
@pytest.mark.parametrize("prec", ["F64", "F32", "F16N"])
def test_reductions_around_the_ticket_limit(dims, prec):
    U = synth.make_links(dims, 0.3, 0.1, 1105)
    from paper_0910_0992_amd import Operator
    g = Operator(torch.from_numpy(U).cuda(), 0.05, 3.0, 0.5, 1.0, -1)
    etas = torch.stack([torch.from_numpy(synth.make_source(dims, 2105 + k)).cuda() for k in range(3)])
    print(f"[case] {dims} {prec}", flush=True)
    for rep in range(2):  # the tickets are back at zero
        x, info = g.solve(etas[0], prec=prec, tol=1e-10)
        assert float((g.apply_M(x) - etas[0]).norm() / etas[0].norm()) < 1.05e-10
        xs, infos = g.solve_multi(etas, prec=prec, tol=1e-10)
        for k in range(3):
            assert float((g.apply_M(xs[k]) - etas[k]).norm() / etas[k].norm()) < 1.05e-10
            assert infos[k]["true_rel_resid"] <= 1e-10
    g.close()


# the line kernels take 16 lines a workgroup below 16 chunks of the line, 8 below 32 and 4 from
# there; 12 and 60 lines of a parity leave a workgroup part empty
TOL_LINES = {"F64": TOL64, "F32": 2e-5, "F16N": 1.5e-2}  # composites


@pytest.mark.parametrize("dims", [(6, 2, 2, 14), (6, 2, 2, 16), (10, 6, 2, 15), (10, 6, 2, 30), (6, 2, 2, 32), (10, 6, 2, 34)])
@pytest.mark.parametrize("prec", ["F64", "F32", "F16N"])
def test_lines_per_workgroup(dims, prec):
    U, o, g = _make(dims)
    etas = [synth.make_source(dims, 2106 + k) for k in range(2)]
    f = g.to_field(torch.stack([torch.from_numpy(e).cuda() for e in etas]), "P3", prec)
    for scheme in ("TEMPORAL_SCHUR", "TEMPORAL"):
        y = g.from_field(g.apply_prec_field(f, scheme))
        for k, e in enumerate(etas):
            assert _rel(y[k], o.prec(scheme, e)) < TOL_LINES[prec], (scheme, k)
    g.close()


# one wavefront per hop up to 32768 sites of a parity times right-hand sides, one thread per site
# beyond; 64 sites a workgroup, the last one part empty
@pytest.mark.parametrize("dims,nr", [((2, 2, 2, 3), 1), ((6, 2, 2, 9), 5), ((8, 8, 8, 43), 3), ((8, 8, 8, 42), 3), ((8, 8, 8, 128), 1),
                                     ((8, 8, 8, 130), 1)])
@pytest.mark.parametrize("prec", ["F64", "F32", "F16N"])
def test_site_kernels_around_the_split(dims, nr, prec):
    big = np.prod(dims) > 10000
    U, o, g = _make(dims, bc=1)
    etas = [synth.make_source(dims, 2108 + k) for k in range(nr)]
    f = g.to_field(torch.stack([torch.from_numpy(e).cuda() for e in etas]), "P3", prec)
    for scheme, dagger in (("UNPREC", False), ("UNPREC", True), ("TEMPORAL_SCHUR", False)):
        y = g.from_field(g.apply_prec_field(f, scheme, dagger))
        for k in range(0, nr, 2 if big else 1):
            ref = (o.prec_dag if dagger else o.prec)(scheme, etas[k])
            assert _rel(y[k], ref) < TOL_LINES[prec], (scheme, dagger, k)
    g.close()


# the exact inverse loads its factors 2 steps ahead on FP32 lines of up to 8 slices, 4 and 8 beyond (FP64:
# 2 and 4)
@pytest.mark.parametrize("lt", [2, 3, 4, 7, 8, 9, 10, 17])
@pytest.mark.parametrize("scheme", ["TEMPORAL_SCHUR3D", "TEMPORAL_FULLSW"])
def test_exact_inverse_of_short_lines(lt, scheme):
    dims = (4, 2, 4, lt)
    U, o, g = _make(dims)
    eta = synth.make_source(dims, 2107)
    t = torch.from_numpy(eta).cuda()
    for prec in ("F64", "F32"):
        assert _rel(g.apply_prec(t, scheme, prec), o.prec(scheme, eta)) < TOL_LINES[prec], prec
        assert _rel(g.apply_prec(t, scheme, prec, dagger=True), o.prec_dag(scheme, eta)) < TOL_LINES[prec], prec
    g.close()
