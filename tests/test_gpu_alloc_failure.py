"""Device allocations that fail. A call either gives up with SCW_ENOMEM or goes
on with less memory and the same result, and the error that a failed allocation
leaves in the HIP runtime does not reach a later call."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

ENOMEM = -2


@pytest.fixture(scope="module")
def ctx():
    import paper_2404_07293_amd as P
    return P.Context(0)


def _failing(ctx, k, call):
    """call() with the k-th allocation failing: (result or None, whether an
    allocation failed)."""
    from paper_2404_07293_amd import _native as N
    fail = ctx.lib.scw_internal_fail_allocation
    fail(k)
    try:
        res = call()
    except N.ScwError as e:
        assert e.code == ENOMEM, (k, e)
        res = None
    return res, fail(0) == 0


def _problems():
    probs = []
    for i in range(3):
        prob = W.surrogate_problem(W.random_index_sample((2, 24, 24), 40 + i))
        prob.px = prob.py = 0.27
        prob.U, prob.V = 5, 3
        probs.append(prob)
    return probs


def test_a_call_after_a_failed_one(ctx):
    import torch
    prob = _problems()[0]
    grid = W.Grid(fx=8, fy=8, fz=2, z_begin=0.0, z_end=prob.thickness)

    def solve():
        sol = ctx.solve(prob, route="stable_device", eig="device")
        return sol, sol.exterior()

    sol, want = solve()
    field = sol.synthesize(grid)
    assert _failing(ctx, 1, solve) == (None, True)
    for a, b in zip(solve()[1], want):
        assert np.array_equal(a, b)
    assert _failing(ctx, 2, solve) == (None, True)
    torch.cuda.synchronize()
    assert torch.equal(sol.synthesize(grid), field)


def test_eigensolver_goes_on_with_a_shorter_record(ctx):
    """n = 100: the rotation record falls to less than a sweep's sum and the
    iteration takes several launches. The same rotations are applied, in other
    groups: 1e-12 of the norm, as the eigensolver's other tests."""
    import torch
    rng = np.random.default_rng(3)
    n, count = 100, 3
    A = torch.from_numpy(rng.standard_normal((count, n, n)) +
                         1j * rng.standard_normal((count, n, n))).cuda()
    norm = float(torch.linalg.matrix_norm(A, ord=2).max())
    survived = 0
    for k in range(1, 20):
        res, failed = _failing(ctx, k, lambda: ctx.eig_batched(A))
        if not failed:
            break
        if res is not None:
            survived += 1
            w, X = res
            r = A @ X.contiguous() - X * w[:, None, :]
            assert float(torch.linalg.vector_norm(r, dim=1).max()) <= 1e-12 * norm * n
    assert not failed and survived == 1


@pytest.mark.parametrize("n", [2, 3, 8, 16, 40, 64])
def test_small_matrices_with_a_shorter_record(ctx, n):
    """Orders whose whole iteration is recorded in one launch, and with the record
    that is taken when that does not fit: several launches, the same rotations."""
    import torch
    rng = np.random.default_rng(n)
    A = torch.from_numpy(rng.standard_normal((5, n, n)) +
                         1j * rng.standard_normal((5, n, n))).cuda()
    norm = float(torch.linalg.matrix_norm(A, ord=2).max())
    for k in (0, 1):  # no allocation, the first one
        w, X = _failing(ctx, k, lambda: ctx.eig_batched(A))[0]
        r = A @ X.contiguous() - X * w[:, None, :]
        assert float(torch.linalg.vector_norm(r, dim=1).max()) <= 1e-12 * norm * n
        assert float((torch.linalg.vector_norm(X, dim=1) - 1).abs().max()) <= 1e-14 * n


def test_solve_batch_goes_on_in_smaller_groups(ctx):
    """Three problems that share an elimination: each of the group's allocations
    may fail and leave smaller groups. 1e-10, as other orders of rounding."""
    probs = _problems()
    want = [s.exterior() for s in ctx.solve_batch(probs, route="stable_device", eig="device")]
    survived = 0
    for k in range(1, 400):
        sols, failed = _failing(
            ctx, k, lambda: ctx.solve_batch(probs, route="stable_device", eig="device"))
        if not failed:
            break
        if sols is not None:
            survived += 1
            for s, w in zip(sols, want):
                for a, b in zip(s.exterior(), w):
                    assert np.linalg.norm(a - b) <= 1e-10 * np.linalg.norm(b)
                s.free()
    print("allocations %d, survived %d" % (k - 1, survived), flush=True)
    # the eigensolver's record, the elimination's 11 + 2 + 3 arrays
    assert not failed and survived == 17
