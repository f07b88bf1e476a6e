"""Rounding of the FP32 real-space sum against the FP64 one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F(gpu):
    import paper_2607_25161_amd as F
    return F


# cutoffs and splitting parameters of the workloads; the sum of some tens to hundreds of pairs a bead, each
# with about ten roundings that do not add up, stays below 1.6 units of FP32 rounding of the sum
@pytest.mark.parametrize("strain", [None, 0.3])
@pytest.mark.parametrize("n,L,xi,tol", [(300, 20.3, 0.5, 1e-5), (1500, 34.7, 0.5, 1e-6), (4000, 48.1, 0.45, 1e-5),
                                        (10000, 65.3, 0.4, 1e-5), (20000, 82.3, 0.348, 1e-5)])
def test_rms_error(F, n, L, xi, tol, strain):
    rng = np.random.default_rng(n)
    m = int(np.ceil(n ** (1 / 3)))
    h = L / m
    x = (np.stack(np.unravel_index(rng.permutation(m ** 3)[:n], (m, m, m)), 1) + 0.5) * h - L / 2
    x += (rng.random((n, 3)) - 0.5) * (h - 2.05)
    s = F.System(F.default_params(xi=xi, ewald_tol=tol, r_lub=0.0))
    s.init_box(L)
    if strain:
        s.set_lees_edwards(True, strain)
    s.init_aggregates(np.arange(n + 1), np.zeros((n, 3)), x, np.tile([1.0, 0, 0, 0], (n, 1)))
    err = []
    for _ in range(3):
        lam = rng.normal(size=6 * n)
        u64 = s.apply_mobility(lam, parts=1)
        u32 = s.apply_mobility(lam, parts=1, precision=F.FSD_MIXED)
        err.append(np.linalg.norm(u32 - u64) / np.linalg.norm(u64))
    assert np.mean(err) < 1.6 * np.finfo(np.float32).eps, err
    s.close()
