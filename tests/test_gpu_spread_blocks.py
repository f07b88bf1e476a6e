"""Gather spreading on 8^3 blocks where its candidate lists wrap: supports as wide as the grid, blocks
that a support enters twice, one to nine blocks a side, both lattices, both precisions."""
import numpy as np
import pytest

from oracle import pse, rpy

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F(gpu):
    import paper_2607_25161_amd as F
    return F


# The grid resolves the damped multipliers to 1e-4 (the cutoff rule) and a support of 8 points or
# more truncates its Gaussians below 1e-5; the operator's error is a small multiple of the two.
@pytest.mark.parametrize("grid,support,L,xi,strain", [
    (8, 8, 6.5, 0.3, 0.0), (16, 14, 11.0, 0.35, 0.0), (16, 16, 9.0, 0.35, 0.47), (24, 21, 11.0, 0.35, -0.5),
    (32, 9, 11.0, 0.5, 0.31), (40, 10, 20.0, 0.5, 0.0), (72, 13, 30.0, 0.6, -0.17)])
@pytest.mark.parametrize("n", [1, 70])
def test_wave_part_where_lists_wrap(F, grid, support, L, xi, strain, n):
    rng = np.random.default_rng(grid + n)
    # one bead body each, anywhere in the box (the wave part does not mind overlaps; r_lub is off)
    x = (rng.random((n, 3)) - 0.5) * L
    s = F.System(F.default_params(xi=xi, grid=grid, support=support, ewald_tol=1e-4, r_lub=0.0))
    s.init_box(L)
    if strain:
        s.set_lees_edwards(True, strain)
    m = 1 if n == 1 else n  # all beads in one body: no overlap check between bodies
    s.init_aggregates(np.array([0, m]), x, np.zeros((1, 3)), np.array([[1.0, 0, 0, 0]]))
    _, _, xl = s.state(beads=True)
    lam = rng.normal(size=6 * n)
    ref = pse.wave_mobility(xl, L, 1.0, 1.0, xi, **({"strain": strain} if strain else {})) @ lam
    u = s.apply_mobility(lam, parts=2)
    assert np.abs(u - ref).max() < 2e-3 * np.abs(ref).max()
    u32 = s.apply_mobility(lam, parts=2, precision=F.FSD_MIXED)
    assert np.abs(u32 - u).max() < 1e-5 * np.abs(u).max()
