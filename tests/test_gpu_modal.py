"""The modal sums at the edges of their forms: FP64 phases made in the sum's
blocks or in a launch before it (up to 1536 per task), one and several steps of
64 columns, and every number of planes per task, against the oracle."""
import numpy as np
import pytest

import workloads as W
from oracle import cwt

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2404_07293_amd as P
    return P.Context(0)


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("fp32", 1e-6)])
@pytest.mark.parametrize("U,V,fz", [(1, 1, 2), (1, 3, 5), (5, 7, 7), (7, 9, 16), (5, 13, 3),
                                    (9, 9, 16), (9, 11, 15), (3, 43, 6)])
def test_modal_sum_edges(ctx, precision, tol, U, V, fz):
    rng = np.random.default_rng(100 * U + V)
    n = 1.3 + 0.3 * rng.random((2, max(V, 4), max(U, 4))) + 0.02j
    prob = W.Problem(n=n.astype(complex), px=0.11, py=0.13, pz=0.2, lam=1.0, U=U, V=V, n_top=1.0,
                     n_bot=1.45, plane_wave=W.PlaneWave(0, 0, 0.8, 0.3 - 0.2j))
    grid = W.Grid(fx=12, fy=10, fz=fz, z_begin=0.0, z_end=prob.thickness)
    _, _, want = cwt.simulate(prob, grid)
    got = ctx.solve(prob).synthesize(grid, precision).cpu().numpy()
    assert np.linalg.norm(got - want) <= tol * np.linalg.norm(want)
