"""Inference at the batch sizes where its launches change, and through the
accesses that depend on alignment and capture."""
import ctypes

import numpy as np
import pytest

from oracle import surrogate as S
from test_gpu_surrogate import _net_and_data, ctx, rel  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 2, 28, 29, 64, 65])
@pytest.mark.parametrize("bf16", [False, True])
def test_small_batches_against_oracle(ctx, B, bf16):  # noqa: F811
    """FP32: blocked sums of at most 1024 terms through ten layers' worth of
    products, 1e-5 with room; bf16: operands rounded to 2^-9 bound it by 2e-2."""
    sur, p, x, _, xd, _ = _net_and_data(ctx, B=B, seed=40 + B)
    sur.set_compute(bf16)
    out = sur.forward(xd).cpu().numpy()
    assert rel(out, S.forward(p, x)) <= (2e-2 if bf16 else 1e-5)
    sur.free()


@pytest.mark.parametrize("bf16,small,large", [(True, 300, 1300), (False, 300, 700)])
def test_large_batches_equal_small_ones(ctx, bf16, small, large):  # noqa: F811
    """A patch's result does not depend on the batch it comes in, also past the
    size from which the activations stream past the cache."""
    import torch
    sur, _, _, _, xd, _ = _net_and_data(ctx, B=4, seed=3)
    sur.free()
    from paper_2404_07293_amd.surrogate import Surrogate
    net = Surrogate(ctx, max_batch=large, seed=5)
    net.set_compute(bf16)
    rng = np.random.default_rng(6)
    n = (1.3 + 0.3 * rng.random((large, 8, 32, 32)) + 0.05j).astype(np.complex64)
    x = net.encode(n)
    assert torch.equal(net.encode(n[:small]), x[:small])
    assert torch.equal(net.forward(x[-small:].contiguous()), net.forward(x)[-small:])
    net.free()


def test_unaligned_arrays(ctx):  # noqa: F811
    """Arrays aligned to a float only, and an output in host memory: same values
    by the other accesses."""
    import torch
    from paper_2404_07293_amd.surrogate import Surrogate
    net, B = Surrogate(ctx, max_batch=2, seed=5), 2
    rng = np.random.default_rng(7)
    n = (1.3 + 0.3 * rng.random((B, 8, 32, 32)) + 0.05j).astype(np.complex64)
    x = net.encode(n)
    out = net.forward(x)
    nb = torch.empty(B * 16384 + 1, dtype=torch.float32, device="cuda")
    nb[1:] = torch.from_numpy(n.view(np.float32).reshape(-1)).cuda()
    xb = torch.zeros(x.numel() + 1, dtype=torch.float32, device="cuda")
    ob = torch.zeros(2 * out.numel() + 1, dtype=torch.float32, device="cuda")
    st = net._stream(None)
    assert net.lib.scw_sur_encode(net.handle, ctypes.c_void_p(nb.data_ptr() + 4), B,
                                  ctypes.c_void_p(xb.data_ptr() + 4), st) == 0
    assert torch.equal(xb[1:].reshape(x.shape), x)
    assert net.lib.scw_sur_forward(net.handle, ctypes.c_void_p(x.data_ptr()), B,
                                   ctypes.c_void_p(ob.data_ptr() + 4), st) == 0
    assert torch.equal(ob[1:], torch.view_as_real(out).reshape(-1))
    host = torch.empty(out.shape, dtype=out.dtype, pin_memory=True)
    assert net.lib.scw_sur_forward(net.handle, ctypes.c_void_p(x.data_ptr()), B,
                                   ctypes.c_void_p(host.data_ptr()), st) == 0
    torch.cuda.synchronize()
    assert torch.equal(host, out.cpu())
    net.free()


def test_captured_forward_sees_new_parameters(ctx):  # noqa: F811
    import torch
    from paper_2404_07293_amd.surrogate import Surrogate
    net = Surrogate(ctx, max_batch=3, seed=5)
    x = torch.rand(3, 16, 32, 32, device="cuda")
    out = torch.empty_like(net.forward(x))
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        net.forward(x, out=out)
    for seed in (8, 9):
        other = Surrogate(ctx, max_batch=3, seed=seed)
        net.set_params(other.get_params())
        want = other.forward(x)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        other.free()
    net.free()
