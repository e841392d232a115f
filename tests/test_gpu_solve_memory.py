"""The device memory that a batch's eigendecompositions take, in blocks of one
2M x 2M complex128 matrix per layer: the header's bound on a round counts seven."""
import threading

import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def test_eigensolver_round_stays_within_its_count():
    import torch
    import paper_2404_07293_amd as P
    ctx = P.Context(0)
    probs = []
    for i in range(4):
        prob = W.surrogate_problem(W.random_index_sample((16, 24, 24), 60 + i))
        prob.px = prob.py = 0.27
        prob.U = prob.V = 11
        probs.append(prob)

    def solve():
        for s in ctx.solve_batch(probs, route="stable", eig="device"):
            s.free()

    solve()  # the library handles' own workspace
    free0, done, least = torch.cuda.mem_get_info()[0], threading.Event(), []

    def watch():
        low = free0
        while not done.is_set():
            low = min(low, torch.cuda.mem_get_info()[0])
        least.append(low)

    t = threading.Thread(target=watch)
    t.start()
    solve()
    done.set()
    t.join()
    n2 = 2 * 11 * 11
    blocks = (free0 - least[0]) / (n2 * n2 * 16 * 16 * len(probs))
    print("%.2f blocks per layer" % blocks, flush=True)
    # 60 MB to a block of every layer; the rest is the small arrays and pages
    assert 4 <= blocks <= 7.5
