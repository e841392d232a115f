"""Gradients at batch sizes where the backward kernels change shape, against the
FP64 reference (oracle/surrogate.py): one patch; batches ending inside a tile
of 32 patches, a K step of 16 or 2 patches; and both sides of the row-group
splits (128 and 256 patches). FP32: every sum has at most 3e5 terms whose
rounding errors (6e-8 each) add as a random walk after blocked sums of a few
thousand, so a parameter group stays within 1e-5 relative L2 (about 2^-24
times the square root of 3e4). bf16: the rounded operands (2^-9 each) bound a
group by 2e-2, as for the small batches of test_gpu_surrogate.py."""
import pytest

from oracle import surrogate as S
from test_gpu_surrogate import _net_and_data, ctx, rel  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 31, 33, 129, 257])
@pytest.mark.parametrize("bf16", [False, True])
def test_gradients_at_tile_edges(ctx, B, bf16):  # noqa: F811
    sur, p, x, tgt, xd, td = _net_and_data(ctx, B=B, seed=20 + B)
    sur.set_compute(bf16)
    loss, g = sur.loss_grad(xd, td)
    out, cache = S.forward(p, x, keep=True)
    want = S.backward(p, cache, out, tgt)
    got = S.unflatten(g.astype("float64"))
    bound = 2e-2 if bf16 else 1e-5
    assert abs(loss / S.loss(out, tgt) - 1.0) <= bound
    errs = {k: rel(got[k], want[k]) for k in want}
    worst = max(errs, key=errs.get)
    print("B=%d bf16=%d: worst group %s %.2e" % (B, bf16, worst, errs[worst]), flush=True)
    assert errs[worst] <= bound
    sur.free()
