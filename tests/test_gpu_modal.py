"""The modal sums at the edges of their forms: FP64 phases made in the sum's
blocks or in a launch before it (up to 1536 per task), one and several steps of
64 columns, and every number of planes per task, against the oracle."""
import dataclasses

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


@pytest.mark.parametrize("U,V,fz,count", [(1, 1, 3, 2), (3, 1, 2, 33), (3, 3, 8, 5), (5, 5, 5, 9),
                                          (5, 13, 4, 3), (9, 11, 16, 4)])
def test_many_illuminations_edges(ctx, U, V, fz, count):
    """Row tiles of 16, K steps of 16 with fewer steps than waves, and partial
    column groups, against the synthesis of each illumination by itself."""
    rng = np.random.default_rng(U + 100 * V)
    n = 1.3 + 0.3 * rng.random((2, max(V, 4), max(U, 4))) + 0.02j
    prob = W.Problem(n=n.astype(complex), px=0.11, py=0.13, pz=0.2, lam=1.0, U=U, V=V, n_top=1.0,
                     n_bot=1.45, plane_wave=W.PlaneWave(0, 0, 0.8, 0.3 - 0.2j))
    ws = [W.PlaneWave(int(rng.integers(-(U // 2), U // 2 + 1)),
                      int(rng.integers(-(V // 2), V // 2 + 1)), *(rng.random(2) + 0.1))
          for _ in range(count)]
    grid = W.Grid(fx=10, fy=9, fz=fz, z_begin=0.0, z_end=prob.thickness)
    got = ctx.solve(prob, waves=ws).synthesize_illuminations(grid).cpu().numpy()
    for k in sorted({0, 1, count - 1}):
        one = ctx.solve(dataclasses.replace(prob, plane_wave=ws[k]))
        want = one.synthesize(grid, "fp64").cpu().numpy()
        assert np.linalg.norm(got[k] - want) <= 1e-6 * np.linalg.norm(want)
