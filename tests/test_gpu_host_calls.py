"""Host calls share one kept block of device memory per context: calls of
different sizes and kinds in turn, with a plan living (and destroyed) in
between, and a plan that outlives its context, give what they give alone."""
import numpy as np
import pytest

from workloads import csr_from_lists, device30_model, make_workload

import paper_2106_01445_amd as g

pytestmark = pytest.mark.gpu


def test_calls_in_turn(gpu_ctx):
    import torch
    wl = make_workload(2, P=200)
    small, none = wl.subset(range(3)), csr_from_lists([])
    w = np.ones(wl.P)

    def fresh(fn):
        ctx = g.Context(0)
        ctx.gbs_set_model(wl.U, wl.r, wl.eta)
        try:
            return fn(ctx)
        finally:
            ctx.close()

    calls = {"exact": lambda c: c.gbs_prob_exact(wl.offsets, wl.modes)["p"],
             "exact3": lambda c: c.gbs_prob_exact(small.offsets, small.modes)["p"],
             "none": lambda c: c.gbs_prob_approx(*none, 2)["logp"],
             "order3": lambda c: c.gbs_prob_approx(wl.offsets, wl.modes, 3)["logp"],
             "order2": lambda c: c.gbs_prob_approx(small.offsets, small.modes, 2)["logp"],
             "grad": lambda c: np.r_[(o := c.gbs_grad(wl.offsets, wl.modes, 2, w))["logp"], o["grad_r"]],
             "dist": lambda c: np.r_[(o := c.gbs_click_distribution(2, ks=(3, 9)))["p_n"], o["p_k"].ravel()]}
    ref = {k: fresh(f) for k, f in calls.items()}
    gpu_ctx.gbs_set_model(wl.U, wl.r, wl.eta)
    lp = torch.zeros(wl.P, dtype=torch.float64, device="cuda:0")
    torch.cuda.synchronize()
    for turn in range(2):
        for k, f in calls.items():
            plan = gpu_ctx.gbs_plan_create(wl.offsets, wl.modes, 3)
            gpu_ctx.gbs_prob_approx_dev(plan, lp)
            if turn:
                plan.close()  # (its work may still run: the next call's block follows it in the stream)
            assert np.allclose(f(gpu_ctx), ref[k], rtol=1e-11, atol=1e-13), (turn, k)
            torch.cuda.synchronize()
            assert np.array_equal(lp.cpu().numpy(), ref["order3"])
            plan.close()


def test_plan_outlives_context():
    U, r, eta = device30_model()
    ctx = g.Context(0)
    ctx.gbs_set_model(U, r, eta)
    plan = ctx.gbs_plan_create(*csr_from_lists([[0, 3, 7]]), 2)
    ctx.gbs_prob_approx(*csr_from_lists([[1, 2]]), 2)
    ctx.close()
    plan.close()
