"""Weight gradients of large batches: the FP32 sums over events are split before
their rounding shows (marker gpu)."""
import pytest

import seeded_inputs as si
from oracle import flow as oflow

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

import paper_2105_10529_amd as mf  # noqa: E402


@pytest.mark.parametrize("d,layers,n", [(16, 8, 1 << 20), (10, 6, 1 << 18)])
def test_copies_of_one_event_sum_to_its_gradient(d, layers, n):
    """n = 2^k copies of one event with equal weights: each adds 2^-k of its
    gradient, every rounding but those of the sums being that of the event
    alone, so that the gradient of the batch is the event's.  A sum runs over at
    most 16384 events, 32 to an addition, and then over at most 64 of them, with
    relative roundings of 2^-24: (512 + 64 + 2) 2^-24 = 3.4e-5, and the same
    again for a first-layer weight, which adds two such sums of one sign.  One
    chain of 2^18 events would reach 8192 2^-24 = 4.9e-4."""
    f = mf.Flow(d, n_layers=layers, max_batch=n)
    shapes = [(int((~m).sum()), 256, int(m.sum()) * 65) for m in oflow.masks(d, layers)]
    f.set_params(mf.Flow.flatten(si.flow_params(shapes, seed=7, scale_out=0.1)))
    y = torch.from_numpy(si.unit_points(1, d, seed=8).T.astype("float32").copy()).cuda()
    one = f.loss_grad(y, torch.ones(1, device="cuda"))[1].double()
    many = f.loss_grad(y.expand(d, n).contiguous(), torch.ones(n, device="cuda"))[1].double()
    assert torch.any(one != 0.0)
    err = ((many - one).abs() / one.abs().clamp_min(1e-300))[one != 0.0].max().item()
    print(f"largest relative error {err:.2e}")
    assert torch.all(many[one == 0.0] == 0.0)
    assert err <= 7e-5
