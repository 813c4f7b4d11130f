"""Sectors of many photons on few clicks, whose last moment lies below the fits'
absolute tolerance (1e-15) while the sector weighs percents of the estimate: a fit
that starts where the feature of that moment has no weight has converged at
once, and must not take a last Newton step by a covariance that is all rounding.

Three clicks at order 2: the moments determine the distribution, so the estimate
is the exact probability and its gradient the exact one's (central differences of
the exact path, step h = 1e-5: h^2 times the third derivative of log p, of order
ten, and 1e-16 / h of rounding).
"""
import numpy as np
import pytest

from workloads import csr_from_lists, small_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed", [0, 72, 122, 181, 289, 322])
def test_estimate_and_gradient_of_determined_rows(gpu_ctx, seed):
    M, h = 3 + seed % 4, 1e-5
    U, r, eta = small_model(M, 5000 + seed, n_squeezed=1 + seed % 3, r_range=(2.0, 3.5), eta_range=(0.6, 0.9))
    off, mod = csr_from_lists([[0, 1, 2], list(range(M - 3, M))])

    def exact(r, eta):
        gpu_ctx.gbs_set_model(U, r, eta)
        return gpu_ctx.gbs_prob_exact(off, mod)["logp"]

    ref = exact(r, eta)
    w = np.array([1.0, 0.5])
    out = gpu_ctx.gbs_grad(off, mod, 2, w)
    assert np.all(out["status"] == 0)
    assert np.abs(out["logp"] - ref).max() <= 1e-8
    assert np.array_equal(gpu_ctx.gbs_prob_approx(off, mod, 2)["logp"], out["logp"])
    for k, x in (("grad_r", r), ("grad_eta", eta)):
        for i in range(M):
            if x[i] == 0.0:
                continue
            d = h * (np.arange(M) == i)
            f = [exact(r + s * d, eta) if k == "grad_r" else exact(r, eta + s * d) for s in (1, -1)]
            assert abs(out[k][i] - w @ (f[0] - f[1]) / (2 * h)) <= 1e-6 * (1.0 + abs(out[k][i])), (k, i)
