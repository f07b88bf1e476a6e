"""Cell search of the pair lists: three to six cells a side, beads at the box's edges and in few
cells, more and fewer candidates than a round of the search, both lattices."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F(gpu):
    import paper_2607_25161_amd as F
    return F


def _pairs(x, L, gam, rc):
    """Ordered pairs of different beads closer than rc, over the images of the (sheared) lattice."""
    n = 0
    for k in np.ndindex(5, 3, 3):
        kx, ky, kz = k[0] - 2, k[1] - 1, k[2] - 1
        d = x[:, None] - x[None] + L * np.array([kx + gam * ky, ky, kz])
        near = (d ** 2).sum(-1) < rc * rc
        np.fill_diagonal(near, False)
        n += near.sum()
    return n


# L / r_cut sets the cells a side; `box` squeezes the beads into a corner of the box, whose
# neighbourhood wraps around its edges
@pytest.mark.parametrize("cells,n,box,strain", [
    (3, 2, 1.0, 0.0), (3, 700, 1.0, 0.0), (4, 63, 0.2, 0.0), (4, 600, 0.15, 0.0), (6, 900, 1.0, 0.0),
    (3, 500, 1.0, 0.41), (5, 700, 0.3, -0.5)])
def test_counts_and_shift_invariance(F, cells, n, box, strain):
    rng = np.random.default_rng(n + cells)
    prm = dict(xi=0.8, ewald_tol=1e-4)
    probe = F.System(F.default_params(**prm))  # the cutoff follows from xi and the tolerance
    probe.init_box(30.0)
    probe.init_aggregates(np.array([0, 1]), np.zeros((1, 3)), np.zeros((1, 3)), np.array([[1.0, 0, 0, 0]]))
    rc = probe.info().r_cut
    probe.close()
    L = (cells + 0.3) * rc * np.sqrt(1 + strain * strain)
    x = (rng.random((n, 3)) - 0.5) * L * box
    lam = rng.normal(size=6 * n)
    got = []
    pairs = _pairs(x, L, strain, rc)
    for shift in (0.0, 0.5, 0.31):
        s = F.System(F.default_params(r_lub=0.0, **prm))
        s.init_box(L)
        if strain:
            s.set_lees_edwards(True, strain)
        y = x + shift * L
        # one body, so the beads may overlap
        s.init_aggregates(np.array([0, n]), y - y.mean(0), y.mean(0)[None], np.array([[1.0, 0, 0, 0]]))
        u = s.apply_mobility(lam, parts=1)
        info = s.info()
        assert info.r_cut == rc
        assert info.nnz_real == pairs
        got.append((info.nnz_real, u))
        s.close()
    for nnz, u in got[1:]:
        assert nnz == got[0][0]
        # the same sums in another order, from positions a few ulps of L apart
        assert np.abs(u - got[0][1]).max() < 1e-10 * np.abs(u).max()


# boxes of less than three cutoffs: every image within the cutoff, a bead's own included, around the
# 64 neighbours that a wavefront takes at a time
@pytest.mark.parametrize("ratio,n,strain", [
    (2.9, 1, 0.0), (2.9, 64, 0.0), (1.3, 65, 0.0), (0.7, 3, 0.0), (2.2, 130, 0.41), (0.9, 63, -0.5)])
def test_counts_in_small_boxes(F, ratio, n, strain):
    prm = dict(xi=0.4, ewald_tol=1e-4, r_lub=0.0)
    got = []
    for shift in (0.0, 0.37):
        rc = L = None
        for _ in range(2):  # the cutoff first, then the box from it
            s = F.System(F.default_params(**prm))
            s.init_box(L or 60.0)
            if strain:
                s.set_lees_edwards(True, strain)
            if L:
                x = (np.random.default_rng(n).random((n, 3)) - 0.5) * L
                y = x + shift * L
                s.init_aggregates(np.array([0, n]), y - y.mean(0), y.mean(0)[None], np.array([[1.0, 0, 0, 0]]))
            else:
                s.init_aggregates(np.array([0, 1]), np.zeros((1, 3)), np.zeros((1, 3)), np.array([[1.0, 0, 0, 0]]))
                rc = s.info().r_cut
                L = ratio * rc
        lam = np.random.default_rng(n + 1).normal(size=6 * n)
        u = s.apply_mobility(lam, parts=1)
        pairs = 0
        for k in np.ndindex(9, 9, 9):
            kx, ky, kz = (v - 4 for v in k)
            d = x[:, None] - x[None] + L * np.array([kx + strain * ky, ky, kz])
            near = (d ** 2).sum(-1) < rc * rc
            if kx == ky == kz == 0:
                np.fill_diagonal(near, False)
            pairs += near.sum()
        assert s.info().r_cut == rc and s.info().nnz_real == pairs
        got.append(u)
    # the same sums in another order, from positions a few ulps of L apart
    assert np.abs(got[0] - got[1]).max() < 1e-10 * np.abs(got[0]).max()
