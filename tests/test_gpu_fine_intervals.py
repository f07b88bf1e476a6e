"""The real-space sum where the smooth part takes twice the intervals (xi r_cut above 7): against the oracle's
quadrature, FP32 against FP64, every launch that it has part in, and in a batch beside a system that keeps
the base intervals."""
import numpy as np
import pytest

from oracle import pse

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F(gpu):
    import paper_2607_25161_amd as F
    return F


def _cloud(F, n, L, seed, **kw):
    """One body of n beads anywhere in the box (its own beads may overlap)."""
    rng = np.random.default_rng(seed)
    s = F.System(F.default_params(r_lub=0.0, **kw))
    s.init_box(L)
    s.init_aggregates(np.array([0, n]), (rng.random((n, 3)) - 0.5) * L, np.zeros((1, 3)), np.array([[1.0, 0, 0, 0]]))
    return s


# xi r_cut 8.1 and 10.0 (and 6.5: base intervals)
@pytest.mark.parametrize("xi,tol", [(2.0, 1e-10), (3.0, 1e-10), (2.0, 1e-5)])
@pytest.mark.parametrize("grid", [64, 50])
def test_against_oracle(F, xi, tol, grid):
    n, L = 40, 8.0
    s = _cloud(F, n, L, 3, xi=xi, ewald_tol=tol, grid=grid, support=8)
    i = s.info()
    assert (xi * i.r_cut > 7) == (tol < 1e-5)
    _, _, x = s.state(beads=True)
    lam = np.random.default_rng(4).normal(size=6 * n)
    ref = pse.real_mobility(np.asarray(x), L, 1.0, 1.0, xi, i.r_cut) @ lam
    u = s.apply_mobility(lam, parts=1)
    # the polynomials' 5e-13 of a self mobility, a few tens of pairs a bead and the quadrature's 1e-13
    assert np.abs(u - ref).max() < 1e-11 * np.abs(ref).max()
    # the fused first launch (side 64) or the separate one, and FP32
    both = s.apply_mobility(lam)
    assert np.abs(both - u - s.apply_mobility(lam, parts=2)).max() < 1e-13 * n * np.abs(both).max()
    u32 = s.apply_mobility(lam, parts=1, precision=F.FSD_MIXED)
    assert np.linalg.norm(u32 - u) < 2e-6 * np.linalg.norm(u)
    s.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_batch_of_both(F, precision):
    def system(k, precision=precision, tol=1e-8):
        rng = np.random.default_rng(k)
        L = 9.0 + k
        x = (np.stack(np.unravel_index(np.arange(27), (3, 3, 3)), 1) + 0.5) * L / 3 - L / 2
        s = F.System(F.default_params(xi=(0.6, 2.5)[k % 2], ewald_tol=1e-6, gmres_tol=tol, r_lub=0.0, grid=64, support=10,
                                      precision=precision))
        s.init_box(L)
        s.init_aggregates(np.arange(28), np.zeros((27, 3)), x, rng.normal(size=(27, 4)))
        s.set_forces(rng.normal(size=(27, 6)))
        return s

    live = [system(k) for k in range(4)]
    assert live[1].info().r_cut * 2.5 > 7 > live[0].info().r_cut * 0.6
    b = F.Batch(1 << 38, len(live))
    for s in live:
        b.admit(s)
    assert b.solve() == 0
    for k, s in enumerate(live):
        exact = system(k, precision=0, tol=1e-12)
        U = exact.solve()[0]
        M, Mp = (np.stack([exact.apply_mobility(e, precision=p) for e in np.eye(6 * 27)], 1) for p in (0, precision))
        # residuals of 1e-8 on either side of the preconditioner, and the operator's own rounding (twice: the
        # batch sums in another order)
        tol = np.linalg.cond(M) * (2e-8 + 2 * np.linalg.norm(Mp - M, 2) / np.linalg.norm(M, 2))
        alone = system(k)
        for V in (s.velocities(), alone.solve()[0]):
            assert np.linalg.norm(V - U) <= tol * np.linalg.norm(U), (k, np.linalg.norm(V - U) / np.linalg.norm(U), tol)
        alone.close()
        exact.close()
    b.close()
    for s in live:
        s.close()
