"""Rows whose spectrum is computed with every sum in a fixed order (up to 8
clicks, and whole devices of up to 40 modes) beside those that split the sums (9
clicks on): both agree with the oracle, at the edges of the ranges and where a
device's 2M columns pass one wavefront (32 modes); the estimates at 1e-9 in log p
and the distribution at 1e-10, absolute, as the other parity tests.  And sectors
whose four moments have no distribution fall back to three moments and so on
down to one, which always succeeds: 256 lossless rows at order 4 are all finite."""
import numpy as np
import pytest

from oracle import approx, model
from workloads import accuracy_workload, csr_from_lists, small_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 7, 8, 9])
def test_short_rows_match_oracle(gpu_ctx, n):
    U, r, eta = small_model(12, 91, n_squeezed=6, r_range=(0.7, 1.1), eta_range=(0.4, 0.8))
    gpu_ctx.gbs_set_model(U, r, eta)
    rng = np.random.default_rng(n)
    rows = [sorted(rng.choice(12, n, replace=False).tolist()) for _ in range(3)]
    out = gpu_ctx.gbs_prob_approx(*csr_from_lists(rows + [list(range(12))]), 2)
    assert np.all(out["status"] == 0)
    Q = model.q_matrix(model.covariance(U, r, eta))
    for i, C in enumerate(rows):
        assert abs(out["logp"][i] - approx.prob_approx(Q, C, 2)) <= 1e-9, (n, i)


@pytest.mark.parametrize("M", [2, 8, 9, 32, 33, 40])
def test_whole_device_matches_oracle(gpu_ctx, M):
    U, r, eta = small_model(M, 92, n_squeezed=max(1, M // 2), r_range=(0.6, 1.0), eta_range=(0.5, 0.9))
    gpu_ctx.gbs_set_model(U, r, eta)
    ks = (M // 2, M)
    out = gpu_ctx.gbs_click_distribution(1, ks)
    assert out["status"] == 0
    Q = model.q_matrix(model.covariance(U, r, eta))
    p, curves, det = approx.click_distribution(Q, 1, ks=ks)
    assert det["nfail"] == 0
    assert np.max(np.abs(out["p_n"] - p)) < 1e-10
    for i, k in enumerate(ks):
        assert np.max(np.abs(out["p_k"][i] - curves[k])) < 1e-10


def test_infeasible_moments_fall_back(gpu_ctx):
    wl = accuracy_workload(70, 1.6, 50, P=256)
    gpu_ctx.gbs_set_model(wl.U, wl.r, wl.eta)
    out = gpu_ctx.gbs_prob_approx(wl.offsets, wl.modes, 4)
    assert np.all(np.isfinite(out["logp"]))
