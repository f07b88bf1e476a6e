"""Interpolation by 8^3 blocks (large systems): supports as wide as the grid, blocks entered twice,
empty blocks, lists far longer and shorter than a staging round, both lattices and precisions; and
the same in a batch.  The beads are many copies of a few positions, so the dense oracle stays small."""
import numpy as np
import pytest

from oracle import pse

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F(gpu):
    import paper_2607_25161_amd as F
    return F


# Tolerances as for the spreading blocks: the cutoff rule's 1e-4 and truncated Gaussians, a small
# multiple of the two; FP32 sums of up to a few thousand terms 1e-5.
@pytest.mark.parametrize("grid,support,L,xi,strain,n,copies", [
    (8, 8, 6.5, 0.3, 0.0, 64, 64), (16, 14, 11.0, 0.35, 0.0, 1, 4097), (16, 16, 9.0, 0.35, 0.47, 128, 64),
    (24, 21, 11.0, 0.35, -0.5, 70, 118), (40, 10, 20.0, 0.5, 0.0, 1366, 3), (72, 13, 30.0, 0.6, 0.0, 65, 64),
    (80, 13, 30.0, 0.6, -0.17, 130, 64)])
def test_wave_part_of_many_beads(F, grid, support, L, xi, strain, n, copies):
    rng = np.random.default_rng(grid + n)
    x = np.repeat((rng.random((n, 3)) - 0.5) * L, copies, axis=0)
    s = F.System(F.default_params(xi=xi, grid=grid, support=support, ewald_tol=1e-4, r_lub=0.0))
    s.init_box(L)
    if strain:
        s.set_lees_edwards(True, strain)
    m = n * copies
    s.init_aggregates(np.array([0, m]), x, np.zeros((1, 3)), np.array([[1.0, 0, 0, 0]]))
    _, _, xl = s.state(beads=True)
    xl = np.asarray(xl)
    lam = rng.normal(size=(m, 6))
    # moments on at most 64 positions: rows and columns of the dense matrix
    keep = np.sort(rng.permutation(n)[:64])
    lam = lam.reshape(n, copies, 6)
    lam[np.setdiff1d(np.arange(n), keep)] = 0
    xs = xl.reshape(n, copies, 3)[keep, 0]
    M = pse.wave_mobility(xs, L, 1.0, 1.0, xi, **({"strain": strain} if strain else {}))
    ref = (M @ lam[keep].sum(1).reshape(-1)).reshape(-1, 6)
    u = s.apply_mobility(lam.reshape(-1), parts=2)
    got = u.reshape(n, copies, 6)[keep]
    assert np.abs(got - ref[:, None]).max() < 2e-3 * np.abs(ref).max()
    u32 = s.apply_mobility(lam.reshape(-1), parts=2, precision=F.FSD_MIXED)
    assert np.abs(u32 - u).max() < 1e-5 * np.abs(u).max()


def _system(F, k, precision):
    rng = np.random.default_rng(k)
    x_body = 2.1 * (np.stack(np.unravel_index(np.arange(27), (3, 3, 3)), 1) - 1.0)
    L, na = 40.0 + k, 34
    com = (np.stack(np.unravel_index(np.arange(na), (4, 4, 4)), 1) + 0.5) * L / 4 - L / 2
    s = F.System(F.default_params(xi=0.35, ewald_tol=1e-4, gmres_tol=1e-8, precision=precision))
    s.init_box(L)
    s.init_aggregates(np.arange(na + 1) * 27, np.concatenate([x_body] * na), com, rng.normal(size=(na, 4)))
    s.set_forces(rng.normal(size=(na, 6)))
    return s


# five systems of 918 beads: one launch by blocks in the batch, by beads alone
@pytest.mark.parametrize("precision", [0, 1])
def test_batch_by_blocks_equals_alone(F, precision):
    live = [_system(F, k, precision) for k in range(5)]
    b = F.Batch(1 << 38, len(live))
    for s in live:
        b.admit(s)
    assert b.solve() == 0
    # FP64: the same arithmetic up to summation order; FP32 matvecs: within the solver tolerance
    tol = 1e-11 if precision == 0 else 1e-7
    for k, s in enumerate(live):
        alone = _system(F, k, precision)
        U, _, _ = alone.solve()
        assert np.abs(s.velocities() - U).max() <= tol * np.abs(U).max()
        alone.close()
    b.close()
    for s in live:
        s.close()
