"""The sector fits' two rounds, their adjoint in the same kernel, and the sector
transform's sizes.

  - every odd factor of the contour size (K = r 2^a, r <= 15) against the oracle
    at order 1 (1e-9 in log p, as the other parity tests);
  - rows whose contour is re-tilted get their cotangents from the second pass:
    a gradient call that re-tilts agrees with one on the plan frozen afterwards,
    whose first pass runs at the same radii (both carry the rounding of the
    moments, err per row, magnified by no more than the clicks' number: 1e-6 of
    the largest component);
  - rows of weight 0 or without a finite weight take no part in the gradient
    (the same sums without them: 1e-12 of the largest component, the spread of
    the atomics).
"""
import numpy as np
import pytest

from oracle import approx, model
from workloads import accuracy_workload, csr_rows, make_workload

pytestmark = pytest.mark.gpu


def _grad(ctx, plan, M, P, w):
    import torch
    d = lambda n: torch.zeros(n, dtype=torch.float64, device="cuda:0")  # noqa: E731
    lp, gr, ge, wt = d(P), d(M), d(M), torch.tensor(w, device="cuda:0")
    st = torch.zeros(P, dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()
    ctx.gbs_grad_dev(plan, wt, lp, gr, ge, st)
    torch.cuda.synchronize()
    return lp.cpu().numpy(), np.concatenate([gr.cpu().numpy(), ge.cpu().numpy()]), st.cpu().numpy()


def test_contour_sizes(gpu_ctx):
    wl = make_workload(2, P=1024)
    gpu_ctx.gbs_set_model(wl.U, wl.r, wl.eta)
    plan = gpu_ctx.gbs_plan_create(wl.offsets, wl.modes, 1)
    import torch
    lp = torch.zeros(wl.P, dtype=torch.float64, device="cuda:0")
    torch.cuda.synchronize()
    gpu_ctx.gbs_prob_approx_dev(plan, lp)
    torch.cuda.synchronize()
    K = plan.info()["K"]
    plan.close()
    odd = K // (K & -K)
    Q = model.q_matrix(model.covariance(wl.U, wl.r, wl.eta))
    rows = csr_rows(wl.offsets, wl.modes)
    seen = {int(r): int(np.argmax(odd == r)) for r in np.unique(odd)}
    assert {1, 3, 5, 7, 9, 11, 13, 15} <= set(seen)
    for r, i in seen.items():
        assert abs(lp[i].item() - approx.prob_approx(Q, list(rows[i]), 1)) <= 1e-9, (r, K[i])


def test_gradient_of_retilted_rows(gpu_ctx):
    order = 2
    wl = accuracy_workload(70, 1.6, 50, P=4)
    gpu_ctx.gbs_set_model(wl.U, wl.r, wl.eta)
    w = np.array([1.0, 0.5, 2.0, 1.5])
    plan = gpu_ctx.gbs_plan_create(wl.offsets, wl.modes, order)
    lp1, g1, st1 = _grad(gpu_ctx, plan, 70, 4, w)
    rho = plan.info()["rho"]
    plan.freeze(True)
    lp2, g2, st2 = _grad(gpu_ctx, plan, 70, 4, w)
    assert np.array_equal(plan.info()["rho"], rho) and np.any(np.abs(rho - 1.0) > 0.01)  # (re-tilted from 1)
    plan.close()
    assert np.all(st1 == 0) and np.all(np.isfinite(g1))
    assert np.max(np.abs(lp1 - lp2)) <= 1e-9
    assert np.max(np.abs(g1 - g2)) <= 1e-6 * np.max(np.abs(g2)), np.max(np.abs(g1 - g2)) / np.max(np.abs(g2))


@pytest.mark.parametrize("order", [2, 3])
def test_rows_without_weight(gpu_ctx, order):
    wl = make_workload(2, P=12)
    gpu_ctx.gbs_set_model(wl.U, wl.r, wl.eta)
    w = np.linspace(0.5, 1.5, 12)
    w[[2, 7]] = [0.0, np.nan]
    plan = gpu_ctx.gbs_plan_create(wl.offsets, wl.modes, order)
    _, g, _ = _grad(gpu_ctx, plan, 20, 12, w)
    plan.close()
    keep = [i for i in range(12) if i not in (2, 7)]
    sub = wl.subset(keep)
    plan = gpu_ctx.gbs_plan_create(sub.offsets, sub.modes, order)
    _, h, _ = _grad(gpu_ctx, plan, 20, 10, w[keep])
    plan.close()
    assert np.all(np.isfinite(g)) and np.max(np.abs(g - h)) <= 1e-12 * np.max(np.abs(h))
