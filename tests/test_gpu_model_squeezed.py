"""The model build at strong squeezing, where Q's condition number (e^{2r}/2) is
far above what fp64 holds and every digit of Q^{-1} comes from the double-double
sweeps.

Lossless, Q = O diag((1 + e^{-2r})/2, (1 + e^{2r})/2) O^T, so Q^{-1} and log det Q
are known in closed form up to how far the fp64 U is from unitary.  That is a
few 2^-53 per entry of O^T O and shifts Q^{-1} (norm 2) and log det Q by as much
times 2M, whatever r: tolerance 64 M 2^-53.
"""
import numpy as np
import pytest

from workloads import small_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [5, 8, 9, 12, 20, 24, 33])
@pytest.mark.parametrize("r0", [3.0, 8.0, 13.0])
def test_inverse_at_strong_squeezing(gpu_ctx, M, r0):
    U, r, eta = small_model(M, 900 + M, r_range=(0.9 * r0, r0), eta_range=(1.0, 1.0))
    gpu_ctx.gbs_set_model(U, r, eta)
    qi, ld = gpu_ctx.gbs_get_model()
    O = np.block([[U.real, -U.imag], [U.imag, U.real]])
    half = 0.5 * np.concatenate([1.0 + np.exp(-2 * r), 1.0 + np.exp(2 * r)])
    tol = 64 * M * 2.0 ** -53
    assert np.abs(qi - (O / half) @ O.T).max() <= tol
    assert abs(ld - np.log(half).sum()) <= tol * (1.0 + abs(ld))
