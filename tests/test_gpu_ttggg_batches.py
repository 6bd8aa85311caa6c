"""g g -> t t~ g g g: an event's weight does not depend on the batch it is
evaluated in (marker gpu)."""
import pytest

import seeded_inputs as si
from gpu_util import to_dev_soa

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2105_10529_amd as mf  # noqa: E402


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_sums_do_not_depend_on_the_batch(precision):
    """Batches that take 4 to 32 polarisation states per pass, one and several
    chunks of events: the same sum in the same order, bit for bit."""
    p = mf.Process(mf.Config(process="gg>ttxggg", precision=precision, dr_min=0.4))
    x = si.points_above_threshold(400_000, 13, 13000.0, 173.0, seed=15)
    u = to_dev_soa(x)
    whole = p.integrand(u)
    assert int((whole != 0).sum()) > 131072
    a = 0
    for m in (1, 70, 500, 3000, 9000, 24000, 70000, 140000):
        assert torch.equal(p.integrand(u[:, a:a + m].contiguous()), whole[a:a + m]), m
        a += m
