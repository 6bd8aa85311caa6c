"""Grid refinement, weight statistics and derivative sums at the edges of
their kernels: one lane per bin, blocks of 256 weights, up to 1024 blocks."""
import numpy as np
import pytest

import oracle
import seeded_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2105_10529_amd as mf  # noqa: E402


@pytest.mark.parametrize("nb", [1, 2, 3, 63, 64])
def test_refine_one_lane_per_bin(nb):
    """Histograms with all, some and one filled bin.  Edges lie in [0, 1] and
    follow from about 2 nb roundings of sums and a logarithm and a power of a
    few units in the last place: 1e-12 leaves a factor above ten."""
    rng = np.random.default_rng(nb)
    h = rng.exponential(size=(5, nb)) ** 3
    h[1, rng.random(nb) < 0.5] = 0.0
    h[2] = 0.0
    h[2, nb // 2] = 1.0
    h[3] = 0.0
    e = si.random_grid(5, nb, seed=nb)
    ed = torch.from_numpy(e).to("cuda")
    mf.vegas_refine(ed, torch.from_numpy(h).to("cuda"), 0.75)
    assert np.max(np.abs(ed.cpu().numpy() - oracle.vegas_refine(e, h, 0.75))) < 1e-12
    assert np.array_equal(ed.cpu().numpy()[3], e[3])


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 262145])
def test_weight_statistics_at_block_edges(n):
    """Order statistics are exact; the mean within the rounding of n sums."""
    w = np.random.default_rng(n).standard_normal(n)
    w[:: 7] = 0.0
    dev = torch.from_numpy(w).to("cuda")
    for q in (1e-9, 0.5, 0.999, 1.0):
        r = mf.weight_stats(dev, q)
        rank = max(1, int(np.ceil(q * n)))
        assert r["quantile"] == np.sort(w)[rank - 1]
        assert r["max"] == w.max() and r["nonzero"] == np.count_nonzero(w)
        assert abs(r["mean"] - w.mean()) <= n * 2.0 ** -52 * np.abs(w).mean()


@pytest.mark.parametrize("ng,n,nb", [(0, 1025, 64), (0, 63, 1), (1, 4097, 31), (1, 300, 32), (2, 2049, 64), (2, 129, 2)])
def test_iteration_histograms_at_bin_counts(ng, n, nb):
    """Histograms of few and of the most bins, ragged waves, one kernel per
    iteration (ng = 0, 1) and staged (ng = 2): the estimate to FP64 rounding and
    the refined edges, which follow from the histograms, to 1e-10, the bounds
    that full iterations are held to."""
    from test_gpu_parity import _oracle

    d = si.ndim(ng)
    p = mf.Process(mf.Config(process="gg>ttx" + "g" * ng, n_bins=nb, dr_min=0.4 if ng >= 2 else 0.0))
    edges = si.random_grid(d, nb, seed=nb)
    out = torch.empty((d, nb + 1), dtype=torch.float64, device="cuda")
    r = p.integrate(1, n, adapt=True, iter_offset=2, edges_in=torch.from_numpy(edges).to("cuda"), edges_out=out)
    S1, S2, hist, nnz, nbad = _oracle(ng).vegas_iteration(edges, 2, n, p.cfg.seed, purpose=0)
    I, s = oracle.iteration_estimate(S1, S2, n)
    assert r.n_nonzero == nnz > 0 and r.n_nonfinite == nbad == 0
    assert abs(r.iter_integral[0] / I - 1) < 1e-12 and abs(r.iter_error[0] / s - 1) < 1e-9
    assert np.max(np.abs(out.cpu().numpy() - oracle.vegas_refine(edges, hist, 1.5))) < 1e-10


@pytest.mark.parametrize("process,precision", [("gg>ttx", "fp64"), ("gg>ttx", "fp32"), ("uux>ttx", "fp64")])
@pytest.mark.parametrize("n", [2, 257, 100003])
def test_iterations_with_and_without_selection_lists(process, precision, n):
    """Without final-state partons an iteration takes all events as they are,
    with observables it takes those above threshold from lists: the same
    weights in other groups of a wave, so compensated sums that agree to
    rounding (1e-14), and histograms whose FP64 sums of n terms, and with them
    the edges, agree within n 2^-53 of their size (below 1e-10 here)."""
    p = mf.Process(mf.Config(process=process, precision=precision))
    edges = torch.from_numpy(si.random_grid(4, 50, seed=3)).to("cuda")
    out = [torch.empty_like(edges), torch.empty_like(edges)]
    obs = {"nbins": 20, "lo": (0.0, 300.0, 0.0), "hi": (500.0, 1300.0, 500.0)}
    a = p.integrate(1, n, edges_in=edges, edges_out=out[0])
    b = p.integrate(1, n, edges_in=edges, edges_out=out[1], observables=obs)
    assert a.n_nonzero == b.n_nonzero and a.n_nonfinite == b.n_nonfinite == 0
    assert abs(a.integral - b.integral) <= 1e-14 * abs(b.integral)
    assert abs(a.error - b.error) <= 1e-9 * abs(b.error)
    assert torch.max((out[0] - out[1]).abs()) < 1e-10
