"""Rounding of the 3D transforms against 80-bit transforms of the same input."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F(gpu):
    import paper_2607_25161_amd as F
    return F


# rms error of a transform of n^3 points in units of 2^-53: about 0.6 sqrt(log2 n^3) for few-step transforms, a
# quarter allowed above it
@pytest.mark.parametrize("n", [20, 24, 36, 48, 60, 64, 96, 100, 120, 144])
def test_rms_error(F, n):
    import torch
    err = []
    for seed in range(3):
        r = np.random.default_rng(seed)
        x = r.normal(size=(n, n, n)) + 1j * r.normal(size=(n, n, n))
        ref = np.fft.fftn(x.astype(np.clongdouble))
        y = torch.tensor(x, device="cuda")
        F.fft3d_noalloc(n, -1, y.data_ptr(), torch.cuda.current_stream().cuda_stream)
        d = y.cpu().numpy() - ref
        err.append(float(np.sqrt((np.abs(d) ** 2).sum() / (np.abs(ref) ** 2).sum())))
    assert np.mean(err) < 0.75 * 2.0 ** -53 * np.sqrt(3 * np.log2(n))
