"""Derivatives at given points do not depend on the batch (marker gpu)."""
import pytest

import seeded_inputs as si
from gpu_util import to_dev_soa

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2105_10529_amd as mf  # noqa: E402


@pytest.mark.parametrize("process,precision", [("gg>ttxg", "fp32"), ("gg>ttxg", "fp64"), ("qg>ttxq", "fp64")])
def test_compacted_points_and_points_as_they_come_agree(process, precision):
    """65537 points are more than a block per compute unit, 65536 and fewer are
    not: every point has the same weight and derivatives, bit for bit."""
    p = mf.Process(mf.Config(process=process, precision=precision))
    u = to_dev_soa(si.points_above_threshold(65537, 7, 13000.0, 173.0, seed=23))
    w, dw = p.integrand_grad(u)
    assert int((w != 0.0).sum()) > 10000
    a = 0
    for m in (65536, 1):
        w1, dw1 = p.integrand_grad(u[:, a:a + m].contiguous())
        assert torch.equal(w1, w[a:a + m]) and torch.equal(dw1, dw[:, a:a + m])
        a += m
