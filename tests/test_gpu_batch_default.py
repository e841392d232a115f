"""The batched launch's default shape at the edges of its rule: radix 8 where fy
allows, and items grabbed by fours, twos and singly, against an explicit shape."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2404_07293_amd as P
    return P.Context(0)


@pytest.mark.parametrize("fx,fy,fz,jobs", [(64, 16, 8, 600), (40, 32, 4, 1100), (64, 64, 4, 1100),
                                           (33, 8, 2, 3), (65, 4, 2, 5), (64, 128, 3, 40)])
def test_default_shape_matches_explicit_one(ctx, fx, fy, fz, jobs):
    """The same sums in another order: 17 x 17 terms, each rounded a few times."""
    sols = []
    for U, V in ((3, 5), (7, 5)):
        rng = np.random.default_rng(U)
        n = (1.3 + 0.3 * rng.random((1, 8, 8))).astype(complex)
        prob = W.Problem(n=n, px=0.11, py=0.13, pz=0.2, lam=1.0, U=U, V=V, n_top=1.0, n_bot=1.45,
                         plane_wave=W.PlaneWave(0, 0, 0.8, 0.3 - 0.2j))
        sols.append(ctx.solve(prob))
    grid = W.Grid(fx=fx, fy=fy, fz=fz, z_begin=0.3, z_end=0.9)
    batch = ctx.batch([sols[j % 2] for j in range(jobs)], grid)
    got = batch.launch().clone()
    batch.configure(2, 2, 1)
    want = batch.launch()
    err = (got - want).abs().pow(2).sum().sqrt() / want.abs().pow(2).sum().sqrt()
    assert float(err) <= 2e-6
