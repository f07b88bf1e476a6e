"""Batches whose grids are more than the last-level cache holds run in several groups of
systems: every system's solution is the one it has alone."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F(gpu):
    import paper_2607_25161_amd as F
    return F


def _system(F, k, grid, precision):
    rng = np.random.default_rng(k)
    m, n = 3, 2 + k % 3  # bodies per side, beads per body (a rod)
    L = 27.0
    x_body = np.concatenate([np.stack([2.0 * np.arange(n) - (n - 1), np.zeros(n), np.zeros(n)], 1)] * m ** 3)
    com = (np.stack(np.unravel_index(np.arange(m ** 3), (m, m, m)), 1) + 0.5) * L / m - L / 2
    quat = rng.normal(size=(m ** 3, 4))
    s = F.System(F.default_params(xi=0.5, grid=grid, ewald_tol=1e-5, gmres_tol=1e-8, precision=precision))
    s.init_box(L)
    s.init_aggregates(np.arange(m ** 3 + 1) * n, x_body, com, quat)
    s.set_forces(rng.normal(size=(m ** 3, 6)))
    return s


# FP64 grids of 48 N^3 bytes: five of 96^3 (42 MB) and one of 144^3 (143 MB) close a group at
# every kind of boundary; FP32 holds twice as many systems to a group
@pytest.mark.parametrize("precision,grids", [(0, (96, 96, 144, 96, 96, 48, 96)), (1, (144, 144, 144, 96))])
def test_grouped_batch_equals_alone(F, precision, grids):
    live = [_system(F, k, g, precision) for k, g in enumerate(grids)]
    b = F.Batch(1 << 38, len(live))
    slots = [b.admit(s) for s in live]
    assert b.solve() == 0
    # FP64: the same arithmetic up to summation order; FP32 matvecs: within the solver tolerance
    tol = 1e-11 if precision == 0 else 1e-7
    for k, g in enumerate(grids):
        s = _system(F, k, g, precision)
        U, _, _ = s.solve()
        assert np.abs(live[k].velocities() - U).max() <= tol * np.abs(U).max()
        assert b.info(slots[k]).rel_residual_fp64 <= 1e-8
        s.close()
    ms, by = b.time_kernel("fft_y", 2)  # replays every group
    assert ms > 0 and by == sum(2 * (24 if precision else 48) * g ** 3 for g in grids)
    b.close()
    for s in live:
        s.close()
