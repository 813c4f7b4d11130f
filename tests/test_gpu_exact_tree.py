"""The exact path's subset tree at the click counts where its split changes
(rows of at most 8, 9, 10 and more clicks are divided differently between the
breadth-first levels, the lanes and the prefix; 13 and 14 clicks exceed the
prefix assignments that share a conditioned matrix), against binary128.

Tolerance: a term carries about n + 2 double-double operations in sequence, each
off by a few 2^-106, and the signed sum magnifies that by kappa, so p is held
to kappa (n + 2) 2^-102 plus the rounding of the result to fp64 (2^-52).
"""
import numpy as np
import pytest

from oracle import exact128
from workloads import csr_from_lists, csr_rows, random_patterns, small_model

pytestmark = pytest.mark.gpu


def check(gpu_ctx, M, U, r, eta, rows):
    off, mod = csr_from_lists(rows)
    gpu_ctx.gbs_set_model(U, r, eta)
    out = gpu_ctx.gbs_prob_exact(off, mod)
    ref = exact128.exact(M, U, r, eta, off, mod)
    p = ref["p_hi"] + ref["p_lo"]
    n = np.array([len(c) for c in rows])
    tol = ref["kappa"] * (n + 2) * 2.0 ** -102 + 2.0 ** -52
    assert np.all(out["status"] == 0), out["status"]
    assert np.all(np.abs(out["p"] / p - 1) <= tol), (np.abs(out["p"] / p - 1) / tol, ref["kappa"])
    assert np.allclose(out["kappa"], ref["kappa"], rtol=1e-9, atol=0)
    return out


@pytest.mark.parametrize("n", [1, 2, 3, 4, 7, 8, 9, 10, 11, 12, 13, 14])
def test_click_counts(gpu_ctx, n):
    M = 16
    U, r, eta = small_model(M, 40 + n, n_squeezed=9, r_range=(0.7, 1.3))
    off, mod = random_patterns(M, 6, n, n, np.random.default_rng(n))
    check(gpu_ctx, M, U, r, eta, [list(c) for c in csr_rows(off, mod)])


@pytest.mark.parametrize("n,r0", [(6, 0.05), (8, 0.1), (10, 0.2), (11, 0.25)])
def test_cancelling_rows(gpu_ctx, n, r0):
    """Weak squeezing: the signed sum cancels by 1e13 and more, so that the last
    digits of the double-double terms are seen."""
    M = 12
    U, r, eta = small_model(M, 70 + n, r_range=(r0, 1.2 * r0))
    off, mod = random_patterns(M, 5, n, n, np.random.default_rng(n))
    out = check(gpu_ctx, M, U, r, eta, [list(c) for c in csr_rows(off, mod)])
    assert out["kappa"].max() > 1e11


def test_parts_of_a_row(gpu_ctx):
    """A batch large enough that a 15-click row is one part gives what the row
    gives alone (32 parts), mixed with short, empty and malformed rows."""
    import torch
    M, P = 18, 20000
    U, r, eta = small_model(M, 90, n_squeezed=9, r_range=(0.7, 1.3))
    rng = np.random.default_rng(3)
    long_row = sorted(rng.choice(M, 15, replace=False).tolist())
    rows = [[], [5, 5], [2], long_row] + [sorted(rng.choice(M, int(rng.integers(1, 7)), replace=False).tolist())
                                          for _ in range(P - 4)]
    off, mod = csr_from_lists(rows)
    gpu_ctx.gbs_set_model(U, r, eta)
    d = lambda a: torch.tensor(a, device="cuda:0")  # noqa: E731
    p, st = torch.zeros(P, dtype=torch.float64, device="cuda:0"), torch.zeros(P, dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()
    gpu_ctx.gbs_prob_exact_dev(d(off), d(mod), 15, p, None, None, st)
    torch.cuda.synchronize()
    p, st = p.cpu().numpy(), st.cpu().numpy()
    assert st[1] == 32 and np.isnan(p[1]) and np.all(np.delete(st, 1) == 0)
    alone = gpu_ctx.gbs_prob_exact(*csr_from_lists([long_row, rows[4], []]))["p"]
    assert abs(p[3] / alone[0] - 1) < 1e-15 and p[4] == alone[1] and p[0] == alone[2]
