"""Interpolation by beads and by blocks on either side of the choice between them: the velocities of a few
hundred beads are the same whether they are alone (by beads) or among thousands without forces."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F(gpu):
    import paper_2607_25161_amd as F
    return F


def _system(F, x, L, grid, P, strain, precision=0):
    n = len(x)
    h = L / grid
    xi = 0.7 * 0.976 * np.sqrt(np.pi * P) / (P * h)
    s = F.System(F.default_params(xi=xi, grid=grid, support=P, ewald_tol=0.9, r_lub=0.0, precision=precision))
    s.init_box(L)
    if strain:
        s.set_lees_edwards(True, strain)
    s.init_aggregates(np.arange(n + 1), np.zeros((n, 3)), x, np.tile([1.0, 0, 0, 0], (n, 1)))
    return s


# by blocks: the first five on the cube in FP64, 4,100 and 20,000 also otherwise; by beads: the rest
@pytest.mark.parametrize("strain", [0.0, 0.31, -0.5])
@pytest.mark.parametrize("n,grid,P", [(1500, 96, 14), (3000, 64, 14), (1100, 64, 21), (4100, 128, 14), (20000, 72, 11),
                                      (4097, 16, 14), (5000, 24, 21), (16384, 48, 6), (513, 32, 10)])
def test_among_others_as_alone(F, n, grid, P, strain):
    rng = np.random.default_rng(n + grid)
    m = int(np.ceil(n ** (1 / 3)))
    L = 3.0 * m
    x = (np.stack(np.unravel_index(rng.permutation(m ** 3)[:n], (m, m, m)), 1) + 0.5) * 3.0 - L / 2
    x += rng.uniform(-0.4, 0.4, (n, 3))
    k = 300
    lam = rng.normal(size=(n, 6))
    lam[k:] = 0
    few, many = _system(F, x[:k], L, grid, P, strain), _system(F, x, L, grid, P, strain)
    for precision, eps in ((0, np.finfo(np.float64).eps), (1, np.finfo(np.float32).eps)):
        ref = few.apply_mobility(lam[:k].reshape(-1), parts=2, precision=precision)
        u = many.apply_mobility(lam.reshape(-1), parts=2, precision=precision)[:6 * k]
        # the same grid up to the order of its sums, P^3 terms a bead in another order
        assert np.abs(u - ref).max() < 64 * eps * np.abs(ref).max(), precision
    few.close()
    many.close()


# many systems on small grids together go by blocks, whose supports are as wide as the grid or enter a
# block twice; alone (by beads) they give the same
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("grid,P,L,m,systems", [(8, 8, 9.0, 4, 128), (16, 16, 11.0, 3, 96), (24, 21, 13.0, 3, 96)])
def test_batch_on_small_grids(F, grid, P, L, m, systems, precision):
    def system(k):
        rng = np.random.default_rng(k)
        n = m ** 3
        x = (np.stack(np.unravel_index(np.arange(n), (m, m, m)), 1) + 0.5) * L / m - L / 2
        h = L / grid
        xi = 0.7 * 0.976 * np.sqrt(np.pi * P) / (P * h)
        s = F.System(F.default_params(xi=xi, grid=grid, support=P, ewald_tol=1e-3, gmres_tol=1e-8, r_lub=0.0,
                                      precision=precision))
        s.init_box(L)
        s.init_aggregates(np.arange(n + 1), np.zeros((n, 3)), x, rng.normal(size=(n, 4)))
        s.set_forces(rng.normal(size=(n, 6)))
        return s

    live = [system(k) for k in range(systems)]
    b = F.Batch(1 << 38, len(live))
    for s in live:
        b.admit(s)
    assert b.solve() == 0
    tol = 1e-11 if precision == 0 else 1e-7
    for k in range(0, systems, 19):
        alone = system(k)
        U, _, _ = alone.solve()
        assert np.abs(live[k].velocities() - U).max() <= tol * np.abs(U).max()
        alone.close()
    b.close()
    for s in live:
        s.close()
