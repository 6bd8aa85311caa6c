"""Flows whose weight-gradient operands do not all fit the memory (marker gpu)."""
import numpy as np
import pytest

import seeded_inputs as si
from oracle import flow as oflow

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2105_10529_amd as mf  # noqa: E402


def test_a_flow_is_created_where_part_of_its_layers_fit():
    """Four dimensions, eight layers, batches of up to 2^24 points: 2400 bytes
    of operands per point and layer, 322 GB, more than the card has; half of the
    layers fit.  The gradient of a batch is that of a flow that holds them all:
    up to 384 points both take chunks of 64 events, so bit for bit."""
    f, small = mf.Flow(4, n_layers=8, max_batch=1 << 24), mf.Flow(4, n_layers=8, max_batch=1000)
    shapes = [(int((~m).sum()), 256, int(m.sum()) * 65) for m in oflow.masks(4, 8)]
    params = mf.Flow.flatten(si.flow_params(shapes, seed=17, scale_out=0.1))
    f.set_params(params)
    small.set_params(params)
    for n in (1, 65, 384):
        y = torch.from_numpy(np.ascontiguousarray(si.unit_points(n, 4, seed=n).T.astype(np.float32))).cuda()
        w = torch.from_numpy(np.random.default_rng(n).exponential(size=n).astype(np.float32)).cuda()
        for loss in ("kl", "variance"):
            (a, g), (b, h) = f.loss_grad(y, w, loss=loss), small.loss_grad(y, w, loss=loss)
            assert a == b and torch.equal(g, h) and torch.any(g != 0.0)
