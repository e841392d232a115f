"""The transform by conjugate pairs against the direct sums of the same
spectra: odd, even and single-point axes, the edges of its 32-pair tiles and of
its register blocks in V, row groups that meet themselves, fields past the
last-level cache, and its fused aperture and intensity."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2404_07293_amd as P
    return P.Context(0)


def problem(U, V):
    rng = np.random.default_rng(10 * U + V)
    n = 1.3 + 0.3 * rng.random((2, max(V, 4), max(U, 4)))
    return W.Problem(n=n.astype(complex), px=0.11, py=0.13, pz=0.2, lam=1.0, U=U, V=V, n_top=1.0,
                     n_bot=1.45, plane_wave=W.PlaneWave(0, 0, 0.8, 0.3 - 0.2j))


def rel(a, b):
    import torch
    a, b = (torch.view_as_real(x).double() for x in (a, b))
    return float((a - b).norm() / b.norm())


# sums of U and V terms, each term and partial sum rounded once, on either side
def tol(precision, U, V):
    return 4 * (U + V) * 2.0 ** -53 if precision == "fp64" else 2 * (U + V) * 2.0 ** -24


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("U,V,fx,fy,fz", [
    (3, 1, 1, 1, 3), (1, 3, 2, 3, 2), (3, 5, 3, 2, 4), (3, 7, 63, 4, 4), (5, 9, 64, 64, 2),
    (3, 13, 65, 6, 3), (3, 17, 128, 65, 3), (3, 21, 130, 34, 2), (3, 25, 31, 128, 2),
    (3, 33, 40, 258, 2), (17, 3, 66, 10, 2), (3, 35, 20, 22, 2), (3, 3, 401, 401, 70),
    (3, 3, 320, 322, 130)])
def test_pairs_match_direct_sums(ctx, precision, U, V, fx, fy, fz):
    prob = problem(U, V)
    sol = ctx.solve(prob)
    grid = W.Grid(fx=fx, fy=fy, fz=fz, z_begin=-0.1, z_end=prob.thickness + 0.1)
    got = sol.synthesize(grid, precision)
    sol.configure(transform="direct")
    want = sol.synthesize(grid, precision)
    assert rel(got, want) <= tol(precision, U, V)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("U,V,fx,fy", [(5, 5, 33, 1), (5, 9, 70, 50), (7, 5, 64, 31)])
def test_image_matches_direct_sums(ctx, precision, U, V, fx, fy):
    prob = problem(U, V)
    sol = ctx.solve(prob)
    grid = W.Grid(fx=fx, fy=fy, fz=5, z_begin=-0.1, z_end=prob.thickness + 0.1)
    E, I = sol.image(grid, 0.9, precision=precision)
    sol.configure(transform="direct")
    E1, I1 = sol.image(grid, 0.9, precision=precision)
    t = tol(precision, U, V)
    assert rel(E, E1) <= t
    assert float((I.double() - I1.double()).norm() / I1.double().norm()) <= 3 * t


@pytest.mark.parametrize("precision,eps", [("bf16x3", 2.0 ** -16), ("fp16x3", 2.0 ** -20)])
@pytest.mark.parametrize("U,V,fx,fy,fz", [(3, 1, 1, 1, 1), (5, 7, 63, 127, 3), (3, 9, 64, 128, 4),
                                          (7, 15, 65, 129, 2), (3, 17, 130, 40, 5),
                                          (3, 23, 33, 260, 70), (5, 25, 70, 31, 2),
                                          (3, 31, 200, 150, 60), (15, 31, 1000, 130, 70)])
def test_split_transform_matches_fp32(ctx, precision, eps, U, V, fx, fy, fz):
    """Every K of the split operands, ragged tiles, runs of one to three planes
    per block, and (the last) the two launches of large repeated sums. A product of two split values keeps the terms down to the
    square of their 8 or 11 bits, so its relative error is at most 3 eps."""
    prob = problem(U, V)
    sol = ctx.solve(prob)
    grid = W.Grid(fx=fx, fy=fy, fz=fz, z_begin=-0.1, z_end=prob.thickness + 0.1)
    got, want = sol.synthesize(grid, precision), sol.synthesize(grid, "fp32")
    assert rel(got, want) <= 3 * eps + tol("fp32", U, V)
