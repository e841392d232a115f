"""scw_solve_batch where neighbouring problems share the device elimination:
mixed truncations, layer counts, routes and eigensolver placements, against
each problem's own scw_solve on the host routes. Both are FP64 solutions of
the same well-conditioned boundary problem; the two agree to 1e-13 on the
working sample, and 1e-10 leaves three digits for other orders of rounding."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _problem(seed, U, V, nz):
    prob = W.surrogate_problem(W.random_index_sample((nz, 24, 24), seed))
    prob.px = prob.py = 0.27
    prob.U, prob.V = U, V
    return prob


SHAPES = {
    "one": [(3, 3, 2)],
    "equal": [(5, 7, 3)] * 4,
    "mixed": [(5, 5, 2), (5, 5, 2), (3, 7, 2), (5, 5, 3), (5, 5, 3), (5, 5, 2), (1, 1, 1)],
}


@pytest.mark.parametrize("route", ["stable_device", "connection_device", "stable"])
@pytest.mark.parametrize("eig", ["device", "host"])
@pytest.mark.parametrize("shapes", sorted(SHAPES))
def test_batch_equals_single_solves(route, eig, shapes):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2404_07293_amd as P
    ctx = P.Context(0)
    probs = [_problem(40 + i, *sh) for i, sh in enumerate(SHAPES[shapes])]
    sols = ctx.solve_batch(probs, route=route, eig=eig)
    for prob, sol in zip(probs, sols):
        one = ctx.solve(prob, route="stable", eig="host")
        for a, b in zip(sol.exterior(), one.exterior()):
            assert np.linalg.norm(a - b) <= 1e-10 * np.linalg.norm(b)
        grid = W.Grid(fx=12, fy=10, fz=2 * prob.nz, z_begin=0.0, z_end=prob.thickness)
        f, g = (x.synthesize(grid, precision="fp64") for x in (sol, one))
        torch.cuda.synchronize()
        assert float(torch.linalg.norm(f - g)) <= 1e-10 * float(torch.linalg.norm(g))
