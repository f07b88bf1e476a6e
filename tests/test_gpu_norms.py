"""The residual norm a solve reports is that of its result: one workgroup's inner product, the last
size of it, the first of the two passes, and many values a workgroup."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F(gpu):
    import paper_2607_25161_amd as F
    return F


# 12 unknowns a body: 12, 32,760, 32,772 and 96,000
@pytest.mark.parametrize("n", [1, 2730, 2731, 8000])
@pytest.mark.parametrize("precision", [0, 1])
def test_reported_residual(F, n, precision):
    rng = np.random.default_rng(n)
    m = max(4, int(np.ceil(n ** (1 / 3) - 1e-9)))
    L = 2.6 * m
    x = (np.stack(np.unravel_index(rng.permutation(m ** 3)[:n], (m, m, m)), 1) + 0.5) * L / m - L / 2
    s = F.System(F.default_params(xi=0.6, ewald_tol=1e-4, gmres_tol=1e-6, precision=precision))
    s.init_box(L)
    s.init_aggregates(np.arange(n + 1), np.zeros((n, 3)), x, np.tile([1.0, 0, 0, 0], (n, 1)))
    s.set_forces(rng.normal(size=(n, 6)))
    U, lam, info = s.solve(True)
    b = np.asarray(s.rhs()).reshape(-1)
    r = b - s.apply_saddle(np.concatenate([lam.reshape(-1), U.reshape(-1)]))
    rel = np.linalg.norm(r) / np.linalg.norm(b)
    # the operator's rounding (1e-15) is far below residuals of 1e-7 and more
    assert rel <= 1e-6 and abs(info.rel_residual_fp64 - rel) < 1e-4 * rel + 1e-13
    s.close()
