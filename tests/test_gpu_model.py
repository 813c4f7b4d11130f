"""The model build's block sweeps at the sizes around their 16-row blocks (one
block, a remainder, an odd and an even number of blocks), through
gbs_get_model, against the oracle's Q inverted by numpy in fp64.

Tolerance: the device holds Q^{-1} in double-double and returns its high part
(2^-53 relative); numpy's inverse is off by at most a few N eps cond(Q) per
entry of a matrix of norm ||Q^{-1}||, and cond(Q) < 150 here, so
100 N 2^-53 ||Q^{-1}|| bounds the difference; log det likewise.
"""
import numpy as np
import pytest

from oracle import model
from workloads import small_model

from paper_2106_01445_amd import gbs

pytestmark = pytest.mark.gpu


def close(gpu_ctx, Q):
    N = Q.shape[0]
    qi, ld = gpu_ctx.gbs_get_model()
    ref = np.linalg.inv(Q)
    assert np.linalg.cond(Q) < 150
    assert np.abs(qi - ref).max() <= 100 * N * 2.0 ** -53 * np.linalg.norm(ref, 2)
    assert abs(ld - np.linalg.slogdet(Q)[1]) <= 100 * N * 2.0 ** -53
    assert np.array_equal(qi, qi.T)


@pytest.mark.parametrize("M", [1, 2, 7, 8, 9, 16, 17, 23, 24, 25, 40])
def test_block_sizes(gpu_ctx, M):
    U, r, eta = small_model(M, 500 + M, r_range=(0.2, 1.2))
    sigma = model.covariance(U, r, eta)
    gpu_ctx.gbs_set_model(U, r, eta)
    close(gpu_ctx, model.q_matrix(sigma))
    gpu_ctx.gbs_set_covariance(0.5 * (sigma + sigma.T))
    close(gpu_ctx, model.q_matrix(0.5 * (sigma + sigma.T)))


@pytest.mark.parametrize("at", [0, 20, 39])
def test_not_positive_definite(gpu_ctx, at):
    """A negative pivot in the first, a middle and the last block; the next
    model is not touched by it."""
    M = 20
    sigma = np.eye(2 * M)
    sigma[at, at] = -1.0
    with pytest.raises(gbs.GBSError) as e:
        gpu_ctx.gbs_set_covariance(sigma)
    assert e.value.code == gbs.GBS_E_NOTPD
    U, r, eta = small_model(M, 11, r_range=(0.2, 1.2))
    gpu_ctx.gbs_set_model(U, r, eta)
    close(gpu_ctx, model.q_matrix(model.covariance(U, r, eta)))
