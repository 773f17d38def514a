"""BiCGStab iterations that break down: the solver's steps on the host, and solves that meet them."""
import os
import subprocess

import numpy as np
import pytest
import torch

import synth
from oracle.schemes import Operator as OOp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_scalar_steps(tmp_path):
    """tests/bicg_steps.hip on the host: ordinary, vanishing, infinite and NaN inner products."""
    from paper_0910_0992_amd.build import FLAGS, HIPCC
    exe = str(tmp_path / "bicg_steps")
    r = subprocess.run([HIPCC, "-x", "hip", os.path.join(ROOT, "tests", "bicg_steps.hip"), "-o", exe] + FLAGS,
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "bicg steps ok" in r.stdout, r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("scale", [1e100, 1e-100])
@pytest.mark.parametrize("scheme", ["UNPREC", "TEMPORAL_SCHUR"])
def test_sources_whose_inner_products_leave_the_range(scale, scheme):
    """|<rhat, v>|^2 overflows or vanishes in every iteration: the FP64 solve goes on with CGNR,
    whose scalars stay in range, and reaches its target."""
    from paper_0910_0992_amd import Operator
    dims = (4, 4, 4, 8)
    U = synth.make_links(dims, 0.35, 0.12, 1000)
    print(f"[case] {scale} {scheme}", flush=True)
    g = Operator(torch.from_numpy(U).cuda(), -0.05, 3.0, 0.5, 1.0, -1)
    eta = scale * synth.make_source(dims, 2000)
    x, info = g.solve(torch.from_numpy(eta).cuda(), scheme=scheme, tol=1e-10)
    g.close()
    o = OOp(U, -0.05, 3.0, -1.0, 0.5, 1.0)
    x = x.cpu().numpy() / scale
    e = eta / scale
    assert np.linalg.norm(e - o.M(x)) <= 1.05e-10 * np.linalg.norm(e), info


@pytest.mark.gpu
def test_half_step_is_kept_when_t_overflows():
    """A spatial link of 1e308 three sites from a point source: the second iteration's t = M s is
    the first vector beyond the range.  Its half step counts, and the residual that the recurrence
    reports (|s|, the true one of UNPREC; a rounding of 1e-16 per operation) is that of the result."""
    from paper_0910_0992_amd import Operator
    dims = (2, 2, 8, 4)
    U = synth.unit_links(dims)
    U[2, 0, 3, 0, 0] *= 1e308
    g = Operator(torch.from_numpy(U).cuda(), 0.05, 3.0, 0.0, 0.0, -1)
    eta = 1e10 * synth.make_point_source(dims, 0, 0)
    x, info = g.solve(torch.from_numpy(eta).cuda(), scheme="UNPREC", tol=1e-10, max_iter=2, raise_on_noconv=False)
    g.close()
    assert info["iters"] == 2 and torch.isfinite(torch.view_as_real(x)).all()
    assert info["true_rel_resid"] < 0.5
    assert abs(info["prec_rel_resid"] - info["true_rel_resid"]) < 1e-12
