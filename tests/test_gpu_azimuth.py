"""Azimuth coordinates outside (0, 1): a value that is not finite never gives a
weight, and whole turns do not matter (marker gpu)."""
import numpy as np
import pytest

import seeded_inputs as si
from gpu_util import to_dev_soa

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2105_10529_amd as mf  # noqa: E402

PROCESSES = [("gg>ttx", "fp64"), ("gg>ttx", "fp32"), ("uux>ttx", "fp64"), ("gg>ttxg", "fp64"), ("gg>ttxg", "fp32"),
             ("qg>ttxq", "fp64"), ("gg>ttxgg", "fp64"), ("gg>ttxgg", "fp32"), ("gg>ttxggg", "fp32")]


def _ng(process):
    return {"gg>ttx": 0, "uux>ttx": 0, "gg>ttxg": 1, "qg>ttxq": 1, "gg>ttxgg": 2, "gg>ttxggg": 3}[process]


def _case(process, precision):
    """A process, 192 of its points and the coordinates that are azimuths (one
    per emitted parton, the last one the top pair's)."""
    ng = _ng(process)
    p = mf.Process(mf.Config(process=process, precision=precision, dr_min=0.4 if ng >= 2 else 0.0))
    x = si.points_above_threshold(192, p.ndim, 13000.0, 173.0, seed=60)
    return p, x, [2 + ng + 2 * i + 1 for i in range(ng + 1)]


@pytest.mark.parametrize("process,precision", PROCESSES)
@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
def test_an_azimuth_that_is_not_finite_gives_no_weight(process, precision, value):
    p, x, phi = _case(process, precision)
    assert np.count_nonzero(p.integrand(to_dev_soa(x)).cpu().numpy()) > 20
    for j in phi:
        y = x.copy()
        y[:, j] = value
        u = to_dev_soa(y)
        assert torch.all(p.integrand(u) == 0.0), j
        if _ng(process) <= 1:
            w, dw = p.integrand_grad(u)
            assert torch.all(w == 0.0) and torch.all(dw == 0.0), j


@pytest.mark.parametrize("process,precision", [("gg>ttx", "fp64"), ("gg>ttxg", "fp64"), ("gg>ttxgg", "fp64")])
@pytest.mark.parametrize("turns", [-200, -3, 3, 200, 100000])
def test_whole_turns_do_not_change_the_weight(process, precision, turns):
    """Azimuths are multiples of 2^-12 here, so that x + turns is exact, and
    x - floor(x) is.  A rounding of the angle, 2^-53 of at most 2 pi, would change
    a weight by that times its logarithmic derivative, below 1e3 for these points
    but where the cuts or a cancellation decide: 1e-9 is wide of it."""
    p, x, phi = _case(process, precision)
    x[:, phi] = np.round(x[:, phi] * 4096) / 4096
    a = p.integrand(to_dev_soa(x)).cpu().numpy()
    y = x.copy()
    y[:, phi] += turns
    b = p.integrand(to_dev_soa(y)).cpu().numpy()
    assert np.count_nonzero(a) > 20
    assert np.all(np.abs(a - b) <= 1e-9 * np.abs(a))
