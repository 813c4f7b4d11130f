"""What the fits' fallback to fewer moments leaves, and a plan's end after its
context's.

At order >= n - 1 the moments determine a row's distribution and the estimate is
the exact probability.  Lossless rows hold sectors whose last moments lie at the
transform's rounding, where fits drop moments; such sectors carry less than 1e-10
of the transform's largest and moved estimates by at most 1e-5 between equally good
roundings, so ten times that bounds the difference from the exact path.
"""
import numpy as np
import pytest

import paper_2106_01445_amd as g
from paper_2106_01445_amd import gbs
from workloads import accuracy_workload, csr_from_lists, small_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,r0", [(8, 1.0), (12, 0.6), (12, 1.2), (20, 1.0)])
def test_determined_rows_equal_the_exact_path(gpu_ctx, M, r0):
    U, r, eta = small_model(M, 31 + M, r_range=(0.8 * r0, r0), eta_range=(1.0, 1.0))
    gpu_ctx.gbs_set_model(U, r, eta)
    rng = np.random.default_rng(M)
    for n in (1, 2, 3, 4, 5):
        off, mod = csr_from_lists([sorted(rng.choice(M, n, replace=False).tolist()) for _ in range(200)])
        exact = gpu_ctx.gbs_prob_exact(off, mod)
        assert np.all(exact["status"] == 0)
        for order in range(max(1, n - 1), 5):
            out = gpu_ctx.gbs_prob_approx(off, mod, order)
            assert np.all(out["status"] == 0), (n, order)
            assert np.abs(out["logp"] - exact["logp"]).max() <= 1e-4, (n, order)


def test_fallback_of_long_lossless_rows(gpu_ctx):
    """70 modes, 50 clicks: many sectors' fourth moments have no distribution.
    Every row has a result (at most its contour is flagged), and the orders
    converge: their steps shrink."""
    wl = accuracy_workload(70, 1.6, 50, P=256)
    gpu_ctx.gbs_set_model(wl.U, wl.r, wl.eta)
    out = [gpu_ctx.gbs_prob_approx(wl.offsets, wl.modes, order) for order in (1, 2, 3, 4)]
    for o in out:
        assert np.all((o["status"] & ~gbs.GBS_PS_CONTOUR) == 0) and np.all(np.isfinite(o["logp"]))
    step = [np.abs(b["logp"] - a["logp"]) for a, b in zip(out, out[1:])]
    assert np.all(step[1] < step[0]) and np.all(step[2] < step[1])


def test_destroy_after_the_context():
    """gbs_plan_destroy of a plan whose context is gone succeeds, whether its block
    came from the context's pool or not, and another context goes on."""
    U, r, eta = small_model(12, 3)
    few, many = csr_from_lists([[0, 3, 7]]), csr_from_lists([[i, 11] for i in range(11)] * 20)
    ctx, other = g.Context(0), g.Context(0)
    for c in (ctx, other):
        c.gbs_set_model(U, r, eta)
    ref = other.gbs_prob_approx(*many, 2)["logp"]
    ctx.gbs_prob_approx(*few, 2)
    plans = [ctx.gbs_plan_create(*few, 2), ctx.gbs_plan_create(*many, 3)]
    ctx.close()
    for p in plans:
        assert gbs.load().gbs_plan_destroy(p.handle) == 0
        p.handle = None
    assert np.array_equal(other.gbs_prob_approx(*many, 2)["logp"], ref)
    other.close()
