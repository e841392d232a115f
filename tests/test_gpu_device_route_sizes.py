"""The device elimination on both sides of the order (2M = 512) from which a
single problem's triangular solves go one by one, with several illuminations'
right-hand sides too. Both routes are FP64 solutions of the same well-conditioned
boundary problem: 1e-10 leaves three digits for other orders of rounding, as in
test_gpu_solve_batch.py."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("U,V", [(15, 17), (17, 17)])
@pytest.mark.parametrize("waves", [0, 3])
def test_single_problem_against_the_host_route(U, V, waves):
    import paper_2404_07293_amd as P
    ctx = P.Context(0)
    prob = W.surrogate_problem(W.random_index_sample((2, 32, 32), 7))
    prob.px = prob.py = 1.0 / 6.0
    prob.U, prob.V = U, V
    w = [W.PlaneWave(0, v, 1.0, 0.5j) for v in range(waves)] or None
    dev = ctx.solve(prob, route="stable_device", eig="host", waves=w)
    host = ctx.solve(prob, route="stable", eig="host", waves=w)
    for a, b in zip(dev.exterior(), host.exterior()):
        assert np.linalg.norm(a - b) <= 1e-10 * np.linalg.norm(b)
    grid = W.Grid(fx=12, fy=10, fz=4, z_begin=0.0, z_end=prob.thickness)
    import torch
    f, g = (x.synthesize(grid, precision="fp64") for x in (dev, host))
    torch.cuda.synchronize()
    assert float(torch.linalg.norm(f - g)) <= 1e-10 * float(torch.linalg.norm(g))
