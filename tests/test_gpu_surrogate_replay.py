"""Parameters that change where the host does not see it: a captured training
step updates them at every replay. Later calls have to use the values of their
time, in both arithmetics; the same kernels on the same values give the same
bits, so the results are compared for equality."""
import pytest

from test_gpu_surrogate import ctx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
def test_calls_after_a_replayed_training_step(ctx, bf16):  # noqa: F811
    import numpy as np
    import torch
    from paper_2404_07293_amd.surrogate import Surrogate
    net, fresh = (Surrogate(ctx, max_batch=3, seed=s) for s in (5, 6))
    for n in (net, fresh):
        n.set_compute(bf16)
    torch.manual_seed(1)
    x = torch.rand(3, 16, 32, 32, device="cuda")
    t = torch.randn(3, 3, 15, 15, device="cuda", dtype=torch.complex64)
    net.forward(x)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        net.train_step(x, t, lr=0.05, want_loss=False)
    net.forward(x)
    torch.cuda.synchronize()
    before = net.get_params()
    for replay in range(3):
        g.replay()
        torch.cuda.synchronize()
        now = net.get_params()
        assert not np.array_equal(now, before)
        before = now
        fresh.set_params(now)
        assert torch.equal(net.forward(x), fresh.forward(x)), replay
        for a, b in zip(net.loss_grad(x, t), fresh.loss_grad(x, t)):
            assert np.array_equal(a, b), replay
    net.free()
    fresh.free()
