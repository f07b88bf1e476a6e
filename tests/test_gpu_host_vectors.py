"""Vectors from and to the caller, through pinned memory up to its size and past it, and read out by
several threads at once."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F(gpu):
    import paper_2607_25161_amd as F
    return F


def _system(F, m, L):
    g = (np.stack(np.unravel_index(np.arange(m ** 3), (m, m, m)), 1) + 0.5) * L / m - L / 2
    s = F.System(F.default_params(xi=0.3, ewald_tol=1e-2, gmres_tol=1e-6))
    s.init_box(L)
    n = m ** 3
    s.init_aggregates(np.arange(n + 1), np.zeros((n, 3)), g, np.tile([1.0, 0, 0, 0], (n, 1)))
    s.set_forces(np.random.default_rng(m).normal(size=(n, 6)))
    return s


# 45^3 beads: the input (547 k values) fits the pinned memory, input and output (1.1 M) do not
@pytest.mark.parametrize("m", [1, 5, 45])
def test_applies_are_additive(F, m):
    s = _system(F, m, 2.6 * max(m, 8))
    rng = np.random.default_rng(3)
    a, b = rng.normal(size=(2, 6 * m ** 3))
    ua, ub, u = (s.apply_mobility(v) for v in (a, b, a + b))
    assert np.abs(ua + ub - u).max() < 1e-12 * np.abs(u).max()
    parts = s.apply_mobility(a, parts=1) + s.apply_mobility(a, parts=2)
    assert np.abs(parts - ua).max() < 1e-12 * np.abs(ua).max()
    a, b = rng.normal(size=(2, 12 * m ** 3))
    ya, yb, y = (s.apply_saddle(v) for v in (a, b, a + b))
    assert np.abs(ya + yb - y).max() < 1e-12 * np.abs(y).max()


def test_read_outs_from_threads(F):
    s = _system(F, 8, 30.0)
    U, lam, _ = s.solve()
    com, quat, xb = s.state(beads=True)
    wrong = []

    def read():
        for _ in range(50):
            c, q, x = s.state(beads=True)
            same = np.array_equal(c, com) and np.array_equal(q, quat) and np.array_equal(x, xb)
            if not same or not np.array_equal(s.velocities(), U):
                wrong.append(1)

    ts = [threading.Thread(target=read) for _ in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not wrong
