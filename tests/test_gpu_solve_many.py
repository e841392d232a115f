"""scw_solve_batch of so many small problems that their elimination's batches
pass the 65536 blocks of a launch's second and third dimension: 2100 problems of
16 layers have 67200 LU factorisations."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _problem(i):
    prob = W.surrogate_problem(W.random_index_sample((16, 4, 4), 100 + i))
    prob.px = prob.py = 0.27
    prob.U = prob.V = 1
    return prob


def test_many_small_problems():
    import paper_2404_07293_amd as P
    ctx = P.Context(0)
    probs = [_problem(i) for i in range(2100)]
    sols = ctx.solve_batch(probs, route="stable_device", eig="device")
    for i in (0, 1, 1000, 2046, 2047, 2048, 2099):
        one = ctx.solve(probs[i], route="stable", eig="host")
        for a, b in zip(sols[i].exterior(), one.exterior()):  # other orders of rounding in FP64
            assert np.linalg.norm(a - b) <= 1e-10 * np.linalg.norm(b), i
    for s in sols:
        s.free()
