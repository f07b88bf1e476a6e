"""3D transforms on the sides of two register steps that no other workload takes, and on neighbours that have
no such steps."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F(gpu):
    import paper_2607_25161_amd as F
    return F


# FP64 rounding of a transform of n^3 points grows with log n: 1e-14 of the largest value
@pytest.mark.parametrize("n", [2, 3, 4, 5, 6, 9, 10, 12, 15, 18, 20, 25, 30, 125, 200, 225])
def test_3d_transform(F, n):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn(n, n, n, dtype=torch.complex128, device="cuda", generator=g)
    for sign in (-1, 1):
        y = x.clone()
        F.fft3d_noalloc(n, sign, y.data_ptr(), torch.cuda.current_stream().cuda_stream)
        ref = torch.fft.fftn(x) if sign < 0 else torch.fft.ifftn(x, norm="forward")
        assert float((y - ref).abs().max()) < 1e-14 * n ** 1.5 * 6
