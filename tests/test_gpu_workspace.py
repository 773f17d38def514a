"""Device memory that an operator keeps between calls."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def test_link_gradient_shares_the_solves_and_applies_fields():
    """After a solve and a canonical scheme apply the gradient needs no memory of its own, and the
    three do not disturb each other."""
    from paper_0910_0992_amd import Operator
    dims = (4, 4, 4, 8)
    U = torch.from_numpy(synth.make_links(dims, 0.35, 0.2, 1100)).cuda()
    eta, lam = (torch.from_numpy(synth.make_source(dims, k)).cuda() for k in (2101, 2102))
    fresh, g = (Operator(U, 0.05, 3.0, 0.5, 1.0, -1) for _ in range(2))
    alone = fresh.force(eta, lam)
    x, _ = g.solve(eta)
    y = g.apply_prec(eta, "TEMPORAL_SCHUR")
    kept = g.device_bytes()
    assert torch.equal(g.force(eta, lam), alone)
    assert g.device_bytes() == kept
    assert torch.equal(g.solve(eta)[0], x) and torch.equal(g.apply_prec(eta, "TEMPORAL_SCHUR"), y)
    assert torch.equal(g.force(eta, lam), alone)
    fresh.close()
    g.close()
