"""A whole device's click distribution, called again, is the same to the last bit:
p(n) as well as the sectors' curves (the sums over sectors have one order)."""
import numpy as np
import pytest

from workloads import device30_model, small_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [1, 2, 3, 4])
@pytest.mark.parametrize("M", [1, 2, 7, 30, 40])
def test_repeats_bit_for_bit(gpu_ctx, M, order):
    U, r, eta = device30_model() if M == 30 else small_model(M, 60 + M, r_range=(0.8, 1.3), eta_range=(0.7, 1.0))
    gpu_ctx.gbs_set_model(U, r, eta)
    ks = (0, 1, M, 2 * M)
    first = gpu_ctx.gbs_click_distribution(order, ks=ks)
    assert first["status"] == 0 and abs(first["p_n"].sum() - 1.0) < 1e-8
    for _ in range(10):
        again = gpu_ctx.gbs_click_distribution(order, ks=ks)
        for k in ("p_n", "p_k"):
            assert np.array_equal(first[k], again[k]), k
