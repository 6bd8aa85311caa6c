"""Derivatives at given points: blocks queue the points that pass the cuts and
evaluate them a full block at a time."""
import numpy as np
import pytest

import seeded_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2105_10529_amd as mf  # noqa: E402


@pytest.mark.parametrize("n,pt", [(1, 0.0), (63, 20.0), (65, 20.0), (255 * 64 + 1, 20.0), (256 * 256 - 1, 0.0),
                                  (256 * 512 + 3, 0.0), (256 * 600 + 77, 20.0), (5000, 1.0e6)])
def test_compacted_derivatives_are_those_of_single_points(n, pt):
    """Shares of fewer points than a wave, of one and several passes with and
    without a remainder, all or no points kept.  An event's derivatives are the
    same arithmetic wherever it is evaluated: bit for bit those of a call with
    only the points that pass, in reverse order, and of a call with that point
    alone; zeros where the integrand is zero."""
    p = mf.Process(mf.Config(process="gg>ttxg", pt_min=pt, eta_max=4.0 if pt else 50.0, seed=5))
    u = torch.from_numpy(np.ascontiguousarray(si.unit_points(n, 7, seed=n % 1000).T)).to("cuda")
    w, dw = p.integrand_grad(u)
    w0 = p.integrand(u)
    assert torch.equal(w == 0.0, w0 == 0.0)
    assert torch.all(dw[:, w == 0.0] == 0.0)
    kept = torch.nonzero(w).flatten().flip(0)
    if len(kept):
        w2, dw2 = p.integrand_grad(u[:, kept].contiguous())
        assert torch.equal(w2, w[kept]) and torch.equal(dw2, dw[:, kept])
    for e in sorted({0, n // 2, n - 1, max(0, n - 65)}):
        w1, dw1 = p.integrand_grad(u[:, e:e + 1].contiguous())
        assert w1[0] == w[e] and torch.equal(dw1[:, 0], dw[:, e])
