"""The eigen-decomposition's launches: a batch of more rows than run at a time is
split into classes of click counts (above 36, 32-36, 26-31, up to 25) beside the
rows above 40; a row's estimate does not depend on which launch it was in, so
the batch reproduces, bit for bit, what a few rows give alone (one launch), and
those agree with the oracle (order 1, 1e-9 in log p as the other parity tests)."""
import numpy as np
import pytest

from oracle import approx, model
from workloads import csr_from_lists, small_model

pytestmark = pytest.mark.gpu

COUNTS = [1, 2, 24, 25, 26, 31, 32, 36, 37, 40, 41, 44]


def test_classes_match_single_launch(gpu_ctx):
    M = 48
    U, r, eta = small_model(M, 77, n_squeezed=24, r_range=(0.8, 1.3), eta_range=(0.4, 0.8))
    rng = np.random.default_rng(5)
    few = [sorted(rng.choice(M, n, replace=False).tolist()) for n in COUNTS] + [[]]
    gpu_ctx.gbs_set_model(U, r, eta)
    alone = gpu_ctx.gbs_prob_approx(*csr_from_lists(few), 1)
    assert np.all(alone["status"] == 0)
    pick = rng.permutation(np.resize(np.arange(len(few)), 1400))
    many = gpu_ctx.gbs_prob_approx(*csr_from_lists([few[i] for i in pick]), 1)
    assert np.array_equal(many["logp"], alone["logp"][pick]) and np.all(many["status"] == 0)
    Q = model.q_matrix(model.covariance(U, r, eta))
    for i in (0, 1, 4, 7, 9, 11, 12):
        assert abs(alone["logp"][i] - approx.prob_approx(Q, few[i], 1)) <= 1e-9, COUNTS[i:i + 1]
