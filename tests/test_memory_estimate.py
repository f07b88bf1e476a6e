"""fsd_estimate_bytes_on against the arrays it stands for: the spreading plan's slots by the support, and the
device memory that a system takes."""
import types

import numpy as np
import pytest


@pytest.fixture(scope="module")
def F():
    import paper_2607_25161_amd as F
    return F


def _slots(P, nbin, sheared):
    """Block slots of a bead: 8^3 blocks that its support can reach, wherever it starts."""
    reach = lambda points: min((7 + points - 1) // 8 + 1, nbin)
    return reach(P) ** 2 * reach(P + P // 2 if sheared else P)  # a sheared row starts up to P / 2 points aside


@pytest.mark.parametrize("sheared", [False, True])
@pytest.mark.parametrize("grid", [16, 64])
def test_estimate_follows_the_support(F, grid, sheared):
    def plan(P):  # records, places, sums; weights in two precisions, sheared rows' starts
        return 68 * _slots(P, grid // 8, sheared) + (12 * (P * P + P) + 2 * P if sheared else 36 * P)

    nb = 1000
    est = {P: F.estimate_bytes(F.default_params(grid=grid, support=P), nb, 100, 40.0, sheared) for P in (4, 10, 16, 21)}
    for P in (10, 16, 21):
        assert est[P] - est[4] >= nb * (plan(P) - plan(4))


def _beads(F, n, L, le, **kw):
    m = int(np.ceil(n ** (1 / 3)))
    x = (np.stack(np.unravel_index(np.random.default_rng(1).permutation(m ** 3)[:n], (m, m, m)), 1) + 0.5) * L / m - L / 2
    return types.SimpleNamespace(L=L, a=1.0, eta=1.0, xi=0.24, ewald_tol=1e-3, grid=64, r_lub=0.0, r_precond=0.0,
                                 gmres_tol=1e-5, offsets=np.arange(n + 1), x_body=np.zeros((n, 3)), com=x,
                                 quat=np.tile([1.0, 0, 0, 0], (n, 1)), force=np.zeros((n, 6)),
                                 grad_u=np.zeros((3, 3)), n_bead=n, n_agg=n, extra=kw)


@pytest.mark.gpu
@pytest.mark.parametrize("P", [10, 21])
@pytest.mark.parametrize("sheared", [False, True])
def test_estimate_covers_the_device_memory(gpu, F, P, sheared):
    import torch
    n, L = 30000, 95.0
    sus = _beads(F, n, L, sheared)

    def build():
        s = F.System.from_suspension(sus, lees_edwards=sheared, support=P)
        s.apply_mobility(np.zeros(6 * n))
        return s

    # code objects, and the scratch that each of the process's hardware queues gets at its first launches
    for s in [build() for _ in range(5)]:
        s.close()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    s = build()
    torch.cuda.synchronize()
    taken = before - torch.cuda.mem_get_info()[0]
    p = F.default_params(xi=0.24, ewald_tol=1e-3, grid=64, r_lub=0.0, r_precond=0.0, support=P)
    est = F.estimate_bytes(p, n, n, L, sheared)
    print("P", P, "sheared", sheared, "taken", taken, "estimate", est)
    s.close()
    assert 0 < taken <= est


@pytest.mark.gpu
@pytest.mark.parametrize("sheared", [False, True])
@pytest.mark.parametrize("grid", [0, 64])
def test_serving_estimate_is_what_a_batch_counts(gpu, F, sheared, grid):
    from paper_2607_25161_amd.serving import LibBackend, Request
    sus = _beads(F, 700, 30.0, sheared)
    sus.grid, sus.xi = grid, 0.0
    be = LibBackend(F, 1 << 34, 1, {}, lees_edwards=sheared)
    req = Request(rid=0, suspension=sus, n_steps=1, n_bead=700)
    slot = be.admit(req)
    assert be.used_bytes() == be.estimate(req)
    be.retire(slot)
