"""bf16 inference under capture. Its mixing weights are a copy made from the
parameters: a graph has to make its own, and a copy that was only captured has
not been made yet. The same kernels on the same values give the same bits."""
import pytest

from test_gpu_surrogate import ctx  # noqa: F401

pytestmark = pytest.mark.gpu


def _nets(ctx, *seeds):  # noqa: F811
    from paper_2404_07293_amd.surrogate import Surrogate
    nets = [Surrogate(ctx, max_batch=3, seed=s) for s in seeds]
    for n in nets:
        n.set_compute(True)
    return nets


def _captured(net, x):
    import torch
    out = torch.zeros(x.shape[0], 3, 15, 15, device="cuda", dtype=torch.complex64)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        net.forward(x, out=out)
    return g, out


def test_replay_sees_new_parameters(ctx):  # noqa: F811
    import torch
    net, other = _nets(ctx, 5, 8)
    x = torch.rand(3, 16, 32, 32, device="cuda")
    net.forward(x)
    g, out = _captured(net, x)
    for params in (other.get_params(), net.get_params()):
        net.set_params(params)
        other.set_params(params)
        want = other.forward(x)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
    for n in (net, other):
        n.free()


def test_eager_call_between_capture_and_replay(ctx):  # noqa: F811
    import torch
    net, other = _nets(ctx, 5, 5)
    x = torch.rand(3, 16, 32, 32, device="cuda")
    net.set_params(other.get_params())
    g, out = _captured(net, x)
    want = other.forward(x)
    assert torch.equal(net.forward(x), want)
    torch.cuda.synchronize()
    g.replay()
    torch.cuda.synchronize()
    assert torch.equal(out, want)
    for n in (net, other):
        n.free()
