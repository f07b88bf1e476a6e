"""A mixed system whose transform tiles were measured in FP32 still applies its operators in FP64, and the
other way round."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F(gpu):
    import paper_2607_25161_amd as F
    return F


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("grid", [24, 64, 72, 96, 100, 256])
def test_applies_after_tuning(F, grid, precision):
    n, L = 300, 24.0
    rng = np.random.default_rng(grid)
    x = (np.stack(np.unravel_index(rng.permutation(343)[:n], (7, 7, 7)), 1) + 0.5) * L / 7 - L / 2
    s = F.System(F.default_params(xi=0.3, grid=grid, ewald_tol=1e-4, r_lub=0.0, precision=precision))
    s.init_box(L)
    s.init_aggregates(np.arange(n + 1), np.zeros((n, 3)), x, np.tile([1.0, 0, 0, 0], (n, 1)))
    lam = rng.normal(size=6 * n)
    ref = {p: s.apply_mobility(lam, parts=2, precision=p) for p in (0, 1)}
    b, g = s.autotune_tiles(2)
    assert b >= 1 and g >= 1
    for p, tol in ((0, 64 * np.finfo(np.float64).eps), (1, 64 * np.finfo(np.float32).eps)):
        u = s.apply_mobility(lam, parts=2, precision=p)
        assert np.abs(u - ref[p]).max() < tol * np.abs(ref[p]).max()
    s.close()
