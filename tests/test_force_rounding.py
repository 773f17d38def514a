"""Rounding of the link gradient, measured against the same gradient in extended precision.

Tolerance, from the kernel's order of operations replayed in numpy (each multiply-add rounded once)
on these inputs: 1.7e-16 of the norm (raw) and 1.9e-16 (projected) where every plaquette is summed
before it joins the gradient, 4.0e-16 and 3.9e-16 where all 72 multiply-adds of the six plaquettes
round the running sum.  2.6e-16 lies between the two.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import force as oforce
from oracle.dirac import sigma
from oracle.schemes import Operator as OOp
from oracle.wilson import AXIS

DIMS, XI, CS, CT = (4, 4, 4, 8), 3.0, 1.6 / 3.0, 1.0
TOL = 2.6e-16
EXT = np.clongdouble


def _dag(m):
    return np.conj(np.swapaxes(m, -1, -2))


def _sh(f, mu, d):
    return np.roll(f, -d, axis=AXIS[mu])


def _project(U, g):
    iug = 1j * (U @ _dag(g))
    h = (iug + _dag(iug)) / 2
    return h - (np.trace(h, axis1=-2, axis2=-1) / 3)[..., None, None] * np.eye(3, dtype=U.dtype)


class _Hopping:
    """What the oracle's hopping gradient reads of an operator."""

    def __init__(self, U):
        self.U, self.gamma_f, self.b = U, U.real.dtype.type(XI), -1.0


def _gradient(U, x, lam):
    """The raw gradient in the type of its inputs: the SW part as the sum over the plaquettes up and
    down from each link of its two sides' corner insertions, added to the hopping part."""
    real = U.real.dtype.type
    grad, _ = oforce.link_gradient(_Hopping(U), x, lam)
    for a, b in ((0, 3), (1, 3), (2, 3), (0, 1), (0, 2), (1, 2)):
        W = np.einsum("st,...tb,...sa->...ba", sigma(a, b).astype(U.dtype), x, lam.conj())
        Z = W / 8 - (np.trace(W, axis1=-2, axis2=-1) / 24)[..., None, None] * np.eye(3, dtype=U.dtype)
        Y = real(CT if b == 3 else CS) / 2 * (Z - _dag(Z))
        for mu, nu, sign in ((a, b, 1), (b, a, -1)):
            E = Y @ U[nu] + U[nu] @ _sh(Y, nu, 1)
            Ef, Bf, Mf = _sh(E, mu, 1), _sh(U[nu], mu, 1), _sh(U[mu], nu, 1)
            up = U[nu] @ Mf @ _dag(Ef) - E @ Mf @ _dag(Bf)
            down = _dag(U[nu]) @ U[mu] @ Ef - _dag(E) @ U[mu] @ Bf
            grad[mu] += sign * (up + _sh(down, nu, -1))
    return grad


def _inputs():
    return synth.make_links(DIMS, 0.35, 0.2, 1100), synth.make_source(DIMS, 2101), synth.make_source(DIMS, 2102)


def test_extended_gradient_against_the_oracle():
    U, x, lam = _inputs()
    raw, proj = oforce.full_link_gradient(OOp(U, 0.05, XI, -1.0, CS, CT), x, lam)
    g = _gradient(*(v.astype(EXT) for v in (U, x, lam)))
    for got, ref in ((g, raw), (_project(U.astype(EXT), g), proj)):
        assert np.linalg.norm(got.astype(complex) - ref) < 1e-14 * np.linalg.norm(ref)


@pytest.mark.gpu
@pytest.mark.parametrize("projected", [False, True])
def test_link_gradient_rounding(projected):
    from paper_0910_0992_amd import Operator
    U, x, lam = _inputs()
    op = Operator(torch.from_numpy(U).cuda(), 0.05, XI, CS, CT, -1)
    got = op.force(torch.from_numpy(x).cuda(), torch.from_numpy(lam).cuda(), projected=projected).cpu().numpy()
    op.close()
    ref = _gradient(*(v.astype(EXT) for v in (U, x, lam)))
    if projected:
        ref = _project(U.astype(EXT), ref)
    err = np.linalg.norm((got - ref).astype(complex)) / np.linalg.norm(ref.astype(complex))
    print(f"[rounding] projected={projected} {err:.3e}", flush=True)
    assert err < TOL
