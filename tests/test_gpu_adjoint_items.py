"""Small batches cut a row's adjoint contour into more items than large ones (rows
fewer than the compute units; the cut is by contour points, at least 8 an item):
the gradient of a few rows equals the one of the same rows among many of weight
zero, to the rounding of sums in another order (1e-9 of the largest component, as
the parity of the floating-point gradient elsewhere)."""
import numpy as np
import pytest

from workloads import csr_from_lists, small_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [1, 2, 3, 4])
def test_few_rows_match_many(gpu_ctx, order):
    M = 24
    U, r, eta = small_model(M, 55, n_squeezed=12, r_range=(0.7, 1.2), eta_range=(0.4, 0.8))
    gpu_ctx.gbs_set_model(U, r, eta)
    rng = np.random.default_rng(order)
    few = [sorted(rng.choice(M, n, replace=False).tolist()) for n in (1, 2, 7, 8, 9, 16, 17, 20)]
    w = rng.uniform(0.5, 1.5, len(few))
    a = gpu_ctx.gbs_grad(*csr_from_lists(few), order, w)
    pad = [sorted(rng.choice(M, 3, replace=False).tolist()) for _ in range(600)]
    b = gpu_ctx.gbs_grad(*csr_from_lists(few + pad), order, np.r_[w, np.zeros(len(pad))])
    assert np.all(a["status"] == 0)
    for k in ("grad_r", "grad_eta"):
        assert np.max(np.abs(a[k] - b[k])) <= 1e-9 * np.max(np.abs(b[k])), (order, k)
