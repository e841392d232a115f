"""The batched launch's default radix on both sides of its bound on the terms (81
of the largest job, where fy = 64 asks for radix 4, else 8), alone and in one
batch with small jobs, against explicit shapes. Every value is a sum over U, then
one over V: the shapes differ in the order of at most 31 terms a sum and in
log2(radix) butterflies, at most some 36 roundings of 6e-8 in each of the two
that add as a random walk, so 5e-7 for each side; 1e-6 has room for both."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2404_07293_amd as P
    return P.Context(0)


@pytest.mark.parametrize("shapes", [[(9, 9)], [(9, 11)], [(11, 9)], [(3, 3), (9, 9)],
                                    [(3, 5), (9, 11), (5, 3)], [(31, 31)]])
@pytest.mark.parametrize("fy", [32, 64])
def test_default_radix_matches_explicit_ones(ctx, shapes, fy):
    sols = []
    for U, V in shapes:
        rng = np.random.default_rng(U)
        n = 1.3 + 0.3 * rng.random((1, 64, 64)) + 0.01j
        sols.append(ctx.solve(W.Problem(n=n, px=0.11, py=0.113, pz=0.2, lam=1.0, U=U, V=V,
                                        n_top=1.0, n_bot=1.45,
                                        plane_wave=W.PlaneWave(0, 0, 0.8, 0.3 - 0.2j)),
                              eig="device", route="stable_device"))
    grid = W.Grid(fx=40, fy=fy, fz=3, z_begin=0.3, z_end=0.9)
    batch = ctx.batch([sols[j % len(sols)] for j in range(7)], grid)
    got = batch.launch().clone()
    for radix in (2, 4, 8, 16):
        batch.configure(radix, 2, 1)
        want = batch.launch()
        err = (got - want).abs().pow(2).sum().sqrt() / want.abs().pow(2).sum().sqrt()
        assert float(err) <= 1e-6, radix
