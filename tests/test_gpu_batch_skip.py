"""A group of systems that have all converged is launched no more while the other groups go on: every
solution and iteration count is the one that the system has alone."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F(gpu):
    import paper_2607_25161_amd as F
    return F


def _system(F, k, hard):
    """27 single beads far apart (a few iterations), or 27 rods close to each other with lubrication."""
    rng = np.random.default_rng(k)
    m = 3
    if hard:
        n, L = 4, 25.5
        x_body = np.concatenate([np.stack([2.0 * np.arange(n) - (n - 1), np.zeros(n), np.zeros(n)], 1)] * m ** 3)
        quat = np.tile([1.0, 0, 0, 0], (m ** 3, 1)) + 0.002 * rng.normal(size=(m ** 3, 4))
        gap = np.array([L / m, 2.06, 2.06])  # stacks of parallel rods
    else:
        n, L = 1, 90.0
        x_body, quat, gap = np.zeros((m ** 3, 3)), rng.normal(size=(m ** 3, 4)), np.full(3, L / m)
    com = (np.stack(np.unravel_index(np.arange(m ** 3), (m, m, m)), 1) - 1.0) * gap
    s = F.System(F.default_params(xi=0.5 if hard else 0.12, grid=96, ewald_tol=1e-5, gmres_tol=1e-9))
    s.init_box(L)
    s.init_aggregates(np.arange(m ** 3 + 1) * n, x_body, com, quat)
    s.set_forces(rng.normal(size=(m ** 3, 6)))
    return s


# FP64 grids of 42 MB each: eight systems make two groups of four
@pytest.mark.parametrize("timing", [False, True])
@pytest.mark.parametrize("first", [False, True])
def test_converged_group(F, first, timing):
    kinds = [first] * 4 + [not first] * 4
    live = [_system(F, k, hard) for k, hard in enumerate(kinds)]
    b = F.Batch(1 << 38, len(live))
    slots = [b.admit(s) for s in live]
    b.set_timing(timing)
    assert b.solve() == 0
    its = {True: [], False: []}
    for k, hard in enumerate(kinds):
        alone = _system(F, k, hard)
        U, _, info = alone.solve()
        its[hard].append(b.info(slots[k]).iterations)
        # the same arithmetic up to summation order
        assert np.abs(live[k].velocities() - U).max() <= 1e-11 * np.abs(U).max()
        assert abs(its[hard][-1] - info.iterations) <= 1
        alone.close()
    assert max(its[False]) + 8 <= min(its[True]), its  # a whole segment without the easy group
    b.close()
    for s in live:
        s.close()
