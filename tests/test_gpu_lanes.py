"""Integrands evaluated by several lanes per event, at the sizes where the
lists of kept points and the groups of lanes have remainders (marker gpu)."""
import numpy as np
import pytest

import oracle
import seeded_inputs as si
from gpu_util import assert_close, to_dev_soa

import paper_2105_10529_amd as mf

pytestmark = pytest.mark.gpu


# one group of lanes, a wave (16 events), a block (64), a selection block (256
# points) and their neighbours; no point kept (all below threshold)
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 63, 64, 65, 255, 256, 257, 1500])
def test_ttgg_fp64_four_lanes_match_the_oracle(n):
    """FP64 on both sides: the tolerance of the other FP64 integrand tests (1e-11 relative, 1e-14 of the
    largest weight)."""
    x = si.points_above_threshold(8 * n + 64, 10, 13000.0, 173.0, seed=100 + n)
    orc = oracle.Oracle(oracle.Config(n_g=2, dr_min=0.4))
    ref = orc.integrand(x)
    # n points of which at least one passes, in their drawn order
    first = int(np.flatnonzero(ref)[0])
    x, ref = x[first:first + n], ref[first:first + n]
    p = mf.Process(mf.Config(process="gg>ttxgg", dr_min=0.4))
    import torch

    u = to_dev_soa(x)
    w = p.integrand(u)
    assert_close(w.cpu().numpy(), ref, 1e-11)
    w2 = torch.empty_like(w)
    p.integrand_noalloc(u, w2)
    assert torch.equal(w, w2)


def test_ttgg_fp64_no_point_kept():
    p = mf.Process(mf.Config(process="gg>ttxgg", dr_min=0.4))
    u = to_dev_soa(np.full((300, 10), 1e-3))  # x1 x2 far below threshold
    assert float(p.integrand(u).abs().max()) == 0.0


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_ttggg_pass_sizes_agree(precision):
    """Batches that take different numbers of polarisation states per pass give each point the same sum up to
    its order: at most 256 double additions of positive terms, 256 x 1.1e-16 = 3e-14; tolerance 1e-13."""
    import torch

    n = 24000
    x = si.points_above_threshold(n, 13, 13000.0, 173.0, seed=5)
    p = mf.Process(mf.Config(process="gg>ttxggg", precision=precision, dr_min=0.4))
    u = to_dev_soa(x)
    whole = p.integrand(u)
    assert int((whole != 0).sum()) > 2000
    a = 0
    for m in (1, 70, 500, 3000, 9000):
        part = p.integrand(u[:, a:a + m].contiguous())
        ref = whole[a:a + m]
        assert torch.all((part - ref).abs() <= 1e-13 * ref.abs())
        a += m


def test_ttgg_fp32_lane_counts_give_the_same_bits():
    """Batches whose kept points are evaluated by 16, 8 and 4 lanes each agree bit for bit (the lanes add the
    states' sums in the order of one lane), and with the oracle to the FP32 tolerance of 1e-5."""
    import torch

    n = 90000
    x = si.points_above_threshold(n, 10, 13000.0, 173.0, seed=9)
    p = mf.Process(mf.Config(process="gg>ttxgg", precision="fp32", dr_min=0.4))
    u = to_dev_soa(x)
    whole = p.integrand(u)
    a = 0
    for m in (1, 17, 300, 1000, 9000, 24000, 45000):
        part = p.integrand(u[:, a:a + m].contiguous())
        assert torch.equal(part, whole[a:a + m]), m
        a += m
    ref = oracle.Oracle(oracle.Config(n_g=2, dr_min=0.4)).integrand(x[:3000])
    got = whole[:3000].cpu().numpy()
    assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref))


@pytest.mark.parametrize("n", [2, 4000, 1 << 17])
def test_ttgg_fp32_staged_and_fused_iterations_agree(n):
    """With observables a small iteration stays in the fused kernel; both sum the same weights in double-double,
    so the estimates agree to FP64 rounding (1e-12, as the oracle's iteration tests)."""
    p = mf.Process(mf.Config(process="gg>ttxgg", precision="fp32", dr_min=0.4))
    a = p.integrate(1, n, adapt=False)
    b = p.integrate(1, n, adapt=False, observables={"nbins": 8, "lo": (0, 0, 0), "hi": (1000, 2000, 1000)})
    assert a.n_nonzero == b.n_nonzero
    assert abs(a.integral - b.integral) <= 1e-12 * abs(b.integral)
    assert abs(a.error - b.error) <= 1e-12 * abs(b.error)
