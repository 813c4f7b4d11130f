"""Device memory of plans: what a plan holds is what its rows need."""
import numpy as np
import pytest

import paper_2106_01445_amd as g
from oracle import approx, model
from workloads import csr_from_lists, small_model

pytestmark = pytest.mark.gpu
MIB = 2 ** 20


def used():
    import torch
    torch.cuda.synchronize()
    free, total = torch.cuda.mem_get_info(0)
    return total - free


@pytest.mark.parametrize("order", [1, 2])
def test_plan_of_long_rows(order):
    """Four rows of 110 clicks: their eigenvectors and twice as much again (9 MB)
    and the cluster sums; no copy of M(w) per workgroup (200 MB), which orders 1
    and 2 never store."""
    M = 112
    U, r, eta = small_model(M, 5, n_squeezed=50, r_range=(1.1, 1.4), eta_range=(0.3, 0.6))
    rng = np.random.default_rng(1)
    off, mod = csr_from_lists([sorted(rng.choice(M, 110, replace=False).tolist()) for _ in range(4)])
    ctx = g.Context(0)
    ctx.gbs_set_model(U, r, eta)
    before = used()
    plan = ctx.gbs_plan_create(off, mod, order)
    grown = used() - before
    plan.close()
    ctx.close()
    assert grown < 32 * MIB, grown


def test_order1_rows_of_any_length(gpu_ctx):
    """Order 1 on 41 to 128 clicks, all with the diagonal blocks of M(w) on chip,
    against the oracle (1e-9 in log p, as the other parity tests)."""
    M = 130
    U, r, eta = small_model(M, 6, n_squeezed=60, r_range=(1.0, 1.4), eta_range=(0.3, 0.6))
    gpu_ctx.gbs_set_model(U, r, eta)
    Q = model.q_matrix(model.covariance(U, r, eta))
    rng = np.random.default_rng(2)
    rows = [sorted(rng.choice(M, n, replace=False).tolist()) for n in (41, 68, 69, 70, 96, 128)]
    out = gpu_ctx.gbs_prob_approx(*csr_from_lists(rows), 1)
    assert np.all(out["status"] == 0)
    for i, C in enumerate(rows):
        assert abs(out["logp"][i] - approx.prob_approx(Q, C, 1)) <= 1e-9, len(C)


def test_small_plan_after_a_large_call():
    """A plan of a few rows made after a large host call leaves the call's block
    (50 MB) to the next call: that one allocates nothing."""
    M, P = 20, 700
    U, r, eta = small_model(M, 7, n_squeezed=10)
    rng = np.random.default_rng(3)
    off, mod = csr_from_lists([sorted(rng.choice(M, 5, replace=False).tolist()) for _ in range(P)])
    ctx = g.Context(0)
    ctx.gbs_set_model(U, r, eta)
    first = ctx.gbs_prob_approx(off, mod, 3)["logp"]
    before = used()
    plan = ctx.gbs_plan_create(off[:4], mod[: off[3]], 3)
    again = ctx.gbs_prob_approx(off, mod, 3)["logp"]
    grown = used() - before
    plan.close()
    ctx.close()
    assert np.array_equal(first, again) and grown < 16 * MIB, grown


def test_large_call_gives_host_memory_back():
    """The context's host copy of a call's results (170 MB for six million empty
    rows) does not stay with it."""
    def resident():
        with open("/proc/self/statm") as f:
            return int(f.read().split()[1]) * 4096

    U, r, eta = small_model(4, 8)
    ctx = g.Context(0)
    ctx.gbs_set_model(U, r, eta)
    few = csr_from_lists([[0], [1, 2]])
    ref = ctx.gbs_prob_exact(*few)["p"]
    off, mod = np.zeros(6_000_001, np.int32), np.zeros(1, np.int32)
    before = resident()
    out = ctx.gbs_prob_exact(off, mod)
    assert np.all(out["p"] == out["p"][0])
    del out
    grown = resident() - before
    assert np.array_equal(ctx.gbs_prob_exact(*few)["p"], ref)
    ctx.close()
    assert grown < 100 * MIB, grown
