"""Spreading on the coarsest sheared grids, by scatter or by blocks: a few hundred beads give the same alone
and among thousands without forces, and switched back to the cube the same as a system of the cube."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F(gpu):
    import paper_2607_25161_amd as F
    return F


def _system(F, x, L, grid, P, strain):
    n = len(x)
    xi = 0.7 * 0.976 * np.sqrt(np.pi * P) / (P * L / grid)
    s = F.System(F.default_params(xi=xi, grid=grid, support=P, ewald_tol=0.9, r_lub=0.0))
    s.init_box(L)
    if strain is not None:
        s.set_lees_edwards(True, strain)
    s.init_aggregates(np.arange(n + 1), np.zeros((n, 3)), x, np.tile([1.0, 0, 0, 0], (n, 1)))
    return s


@pytest.mark.parametrize("n,grid,P", [(511, 16, 6), (512, 16, 6), (700, 8, 6), (2047, 16, 10), (2048, 16, 10),
                                      (2048, 16, 11), (4096, 24, 6)])
def test_among_others_as_alone(F, n, grid, P):
    rng = np.random.default_rng(n + P)
    m = int(np.ceil(n ** (1 / 3)))
    L = 3.0 * m
    x = (np.stack(np.unravel_index(rng.permutation(m ** 3)[:n], (m, m, m)), 1) + 0.5) * 3.0 - L / 2
    x += rng.uniform(-0.4, 0.4, (n, 3))
    k = 200
    lam = rng.normal(size=(n, 6))
    lam[k:] = 0
    few, many, cube = (_system(F, x[:k], L, grid, P, -0.4), _system(F, x, L, grid, P, -0.4), _system(F, x, L, grid, P, None))
    for precision, eps in ((0, np.finfo(np.float64).eps), (1, np.finfo(np.float32).eps)):
        ref = few.apply_mobility(lam[:k].reshape(-1), precision=precision)
        u = many.apply_mobility(lam.reshape(-1), precision=precision)[:6 * k]
        # the same sums in other orders
        assert np.abs(u - ref).max() < 64 * eps * np.abs(ref).max(), precision
    many.set_lees_edwards(False, 0.0)
    full = rng.normal(size=6 * n)
    assert np.array_equal(many.apply_mobility(full), cube.apply_mobility(full))
