"""Two-step transforms: every side that has one, alone and inside the wave-space operator."""
import numpy as np
import pytest

from oracle import pse

pytestmark = pytest.mark.gpu

WAVE = [8, 16, 24, 32, 40, 48, 64, 72, 80, 96, 120, 128, 144, 160, 192, 240, 256]
OTHER = [27, 36, 45, 50, 54, 60, 75, 81, 90, 100, 108, 135, 150, 180]


@pytest.fixture(scope="module")
def F(gpu):
    import paper_2607_25161_amd as F
    return F


# FP64 rounding of a transform of n^3 points grows with log n: 1e-14 of the largest value
@pytest.mark.parametrize("n", WAVE + OTHER)
def test_3d_transform(F, n):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn(n, n, n, dtype=torch.complex128, device="cuda", generator=g)
    for sign in (-1, 1):
        y = x.clone()
        F.fft3d_noalloc(n, sign, y.data_ptr(), torch.cuda.current_stream().cuda_stream)
        ref = torch.fft.fftn(x) if sign < 0 else torch.fft.ifftn(x, norm="forward")
        assert float((y - ref).abs().max()) < 1e-14 * n ** 1.5 * 6


# Gaussians truncated below 1e-8 and multipliers resolved by every side (xi L / n <= 0.25)
@pytest.mark.parametrize("strain", [0.0, 0.37])
@pytest.mark.parametrize("n", [n for n in WAVE if n >= 40])
def test_wave_part(F, n, strain):
    rng = np.random.default_rng(n)
    L, nb, xi = 11.0, 5, 0.6
    s = F.System(F.default_params(xi=xi, grid=n, ewald_tol=1e-9, r_lub=0.0))
    s.init_box(L)
    if strain:
        s.set_lees_edwards(True, strain)
    s.init_aggregates(np.array([0, nb]), (rng.random((nb, 3)) - 0.5) * L, np.zeros((1, 3)), np.array([[1.0, 0, 0, 0]]))
    _, _, x = s.state(beads=True)
    lam = rng.normal(size=6 * nb)
    ref = pse.wave_mobility(x, L, 1.0, 1.0, xi, strain=strain) @ lam
    u = s.apply_mobility(lam, parts=2)
    assert np.abs(u - ref).max() < 1e-7 * np.abs(ref).max()
    u32 = s.apply_mobility(lam, parts=2, precision=F.FSD_MIXED)
    assert np.abs(u32 - u).max() < 1e-5 * np.abs(u).max()
    s.close()
