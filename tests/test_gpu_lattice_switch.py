"""A system switched from the sheared lattice back to the cube runs as one that was always there."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F(gpu):
    import paper_2607_25161_amd as F
    return F


# 40: a plan of 8^3 blocks on both lattices; 36: one of 4^3 blocks on the cube and none on the sheared lattice;
# 45: none
@pytest.mark.parametrize("grid", [40, 36, 45])
@pytest.mark.parametrize("prepared", [False, True])
@pytest.mark.parametrize("precision", [0, 1])
def test_back_on_the_cube(F, grid, prepared, precision):
    n, L = 700, 30.0
    rng = np.random.default_rng(grid)
    x = (np.stack(np.unravel_index(rng.permutation(9 ** 3)[:n], (9, 9, 9)), 1) + 0.5) * L / 9 - L / 2
    x += rng.uniform(-0.5, 0.5, (n, 3))
    lam = rng.normal(size=6 * n)

    def system(sheared):
        s = F.System(F.default_params(xi=0.4, grid=grid, ewald_tol=1e-4, r_lub=0.0))
        s.init_box(L)
        if sheared:
            s.set_lees_edwards(True, 0.3)
        s.init_aggregates(np.arange(n + 1), np.zeros((n, 3)), x, np.tile([1.0, 0, 0, 0], (n, 1)))
        return s

    ref = system(False).apply_mobility(lam, precision=precision)
    s = system(True)
    if prepared:
        assert np.linalg.norm(s.apply_mobility(lam, precision=precision) - ref) > 1e-3 * np.linalg.norm(ref)
    s.set_lees_edwards(False, 0.0)
    out = [s.apply_mobility(lam, precision=precision) for _ in range(3)]
    if grid % 4 == 0:  # sums in a fixed order: the same bits
        for u in out:
            assert np.array_equal(u, ref)
    else:  # atomic adds: up to their order, P^3 terms of a point and as many of a bead
        for u in out:
            assert np.abs(u - ref).max() < 64 * np.finfo([np.float64, np.float32][precision]).eps * np.abs(ref).max()
