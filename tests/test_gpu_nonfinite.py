"""Events whose weight is not finite are dropped and counted, whichever kernels
an iteration runs (marker gpu)."""
import numpy as np
import pytest

from gpu_util import to_dev_soa

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2105_10529_amd as mf  # noqa: E402


def _p(process, precision, sqrt_s, **kw):
    return mf.Process(mf.Config(process=process, precision=precision, sqrt_s=sqrt_s, dr_min=0.4, **kw))


@pytest.mark.parametrize("sqrt_s", [1e39, 1e41])
@pytest.mark.parametrize("n", [300, 20000])
def test_staged_and_fused_iterations_count_the_same_events(sqrt_s, n):
    """At 1e39 GeV some FP32 amplitudes overflow, at 1e41 all of them.  With
    observables the iteration stays in the fused kernel."""
    p = _p("gg>ttxgg", "fp32", sqrt_s)
    a = p.integrate(1, n, adapt=False)
    b = p.integrate(1, n, adapt=False, observables={"nbins": 8, "lo": (0, 0, 0), "hi": (1000, 2000, 1000)})
    assert b.n_nonfinite > 0
    assert (a.n_nonfinite, a.n_nonzero) == (b.n_nonfinite, b.n_nonzero)
    if sqrt_s == 1e41:
        assert a.n_nonzero == 0 and a.integral == 0.0


@pytest.mark.parametrize("process,precision,sqrt_s,kw", [
    ("gg>ttxgg", "fp32", 1e41, {}), ("gg>ttxgg", "fp64", 1e110, {}), ("gg>ttxgg", "fp32", 1e41, {"colour_form": 2}),
    ("gg>ttxggg", "fp32", 1e41, {}), ("gg>ttxggg", "fp64", 1e110, {})])
def test_all_kept_events_are_counted(process, precision, sqrt_s, kw):
    """Where no kept event's weight is finite, the count is the number of kept
    events: far above threshold the cuts do not depend on the energy, so that
    of 1e12 GeV (in FP64: the 5-gluon sum underflows there in FP32).  The integrand at given points stays 0 there."""
    far, near = _p(process, precision, sqrt_s, **kw), _p(process, "fp64", 1e12)
    a, b = far.integrate(1, 3000, adapt=False), near.integrate(1, 3000, adapt=False)
    assert b.n_nonfinite == 0 and b.n_nonzero > 300
    assert a.n_nonfinite == b.n_nonzero and a.n_nonzero == 0 and a.integral == 0.0
    x = np.random.default_rng(3).random((500, far.ndim))
    assert torch.all(far.integrand(to_dev_soa(x)) == 0.0)
    assert torch.any(near.integrand(to_dev_soa(x)) != 0.0)


@pytest.mark.parametrize("process,precision,sqrt_s", [("gg>ttxgg", "fp64", 1e110), ("gg>ttxggg", "fp32", 1e41)])
def test_staged_fallback_of_a_learned_proposal_stays_accepted(process, precision, sqrt_s):
    """A first flow iteration without a finite weight falls back to VEGAS; the
    integrand's own non-finite values are not taken for a broken proposal."""
    p = _p(process, precision, sqrt_s)
    r = p.integrate(3, 1000, adapt=False, flow=mf.Flow(p.ndim, max_batch=64), fallback_rel_var=1.0)
    assert r.fallback_iter == 1 and r.n_iter_done == 3 and r.n_nonzero == 0
