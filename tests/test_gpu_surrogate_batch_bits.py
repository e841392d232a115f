"""FP32 inference gives a patch the same bits in every batch: the kernels that a
batch's size selects add the same terms in the same order."""
import pytest

from test_gpu_surrogate import ctx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 2, 28, 29, 64, 65, 128, 129])
def test_a_patch_does_not_depend_on_its_batch(ctx, B):  # noqa: F811
    import torch
    from paper_2404_07293_amd.surrogate import Surrogate
    net = Surrogate(ctx, max_batch=300, seed=5)
    torch.manual_seed(B)
    x = torch.randn(300, 16, 32, 32, device="cuda")
    whole = net.forward(x)
    for first in (0, 300 - B):
        part = net.forward(x[first:first + B].contiguous())
        assert torch.equal(part, whole[first:first + B])
    net.free()
