"""The real-space pair sum: its piecewise polynomials at interval edges, and its FP32 form against
the FP64 one for every lane count and row split of the launch."""
import numpy as np
import pytest

from oracle import pse, rpy

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F(gpu):
    import paper_2607_25161_amd as F
    return F


def _beads(F, n, L, seed, **kw):
    """n single beads on a jittered lattice (spacing at least 2.05a)."""
    m = int(np.ceil(n ** (1 / 3)))
    rng = np.random.default_rng(seed)
    h = L / m
    x = (np.stack(np.unravel_index(rng.permutation(m ** 3)[:n], (m, m, m)), 1) + 0.5) * h - L / 2
    x += (rng.random((n, 3)) - 0.5) * max(h - 2.05, 0.0)
    s = F.System(F.default_params(r_lub=0.0, **kw))
    s.init_box(L)
    s.init_aggregates(np.arange(n + 1), np.zeros((n, 3)), x, np.tile([1.0, 0, 0, 0], (n, 1)))
    return s, x, rng


@pytest.mark.parametrize("xi,tol", [(0.348, 1e-5), (0.5, 1e-8), (1.2, 1e-6)])
def test_polynomials_at_interval_edges(F, xi, tol):
    s, _, _ = _beads(F, 3, 40.0, 1, xi=xi, ewald_tol=tol)
    w = s.info().r_cut / 64
    r = np.array([0.3 * w, w * (1 - 1e-9), w * (1 + 1e-9), 7.5 * w, 31 * w * (1 + 1e-12), 32 * w * (1 - 1e-12),
                  63 * w * (1 + 1e-9), 64 * w * (1 - 1e-9)])
    scale = np.array([rpy.mu_t(1, 1), rpy.mu_t(1, 1), rpy.mu_r(1, 1), rpy.mu_r(1, 1), rpy.mu_t(1, 1)])
    assert np.abs((s.real_functions(r) - pse.real_functions(r, 1.0, 1.0, xi)) / scale).max() < 1e-12


# lanes per row grow with the pairs per bead (1 to 64 here); 5,000 and 30,000 beads take one and
# several passes of rows per workgroup
@pytest.mark.parametrize("n,L,xi", [(1, 9.0, 0.6), (7, 30.0, 0.9), (129, 60.0, 0.6), (300, 32.0, 0.5), (257, 20.0, 0.35),
                                    (5000, 62.0, 0.4), (30000, 80.0, 0.45)])
def test_fp32_sum_within_single_precision(F, n, L, xi):
    s, _, rng = _beads(F, n, L, n, xi=xi, ewald_tol=1e-5)
    lam = rng.normal(size=6 * n)
    u64 = s.apply_mobility(lam, parts=1)
    u32 = s.apply_mobility(lam, parts=1, precision=F.FSD_MIXED)
    assert np.linalg.norm(u32 - u64) < 2e-6 * np.linalg.norm(u64)
    assert abs(lam @ u64) > 0
    mu = rng.normal(size=6 * n)  # the sum is symmetric
    assert abs(mu @ u64 - lam @ s.apply_mobility(mu, parts=1)) < 1e-12 * np.linalg.norm(mu) * np.linalg.norm(u64)
