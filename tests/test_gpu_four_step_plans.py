"""Four-step transforms of lengths whose half has no divisor up to 256 that leaves at
most 1024: a larger second factor (343 x 686, 375 x 625), or a first one above 1024
(1331 x 121). Tolerances: float64 1e-14, float32 4e-7 (float32 butterflies; some 40
roundings of 2^-24 in a random walk)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_1704_04362_amd.api")


@pytest.mark.parametrize("dtype,tol", [(np.float64, 1e-14), (np.float32, 4e-7)])
@pytest.mark.parametrize("n3, shape", [(235298, (3, 3)), (468750, (1, 1)), (470596, (2, 1)), (322102, (5, 2)),
                                       (449878, (1, 1))])
def test_four_step_plans(n3, shape, dtype, tol):
    x = np.random.default_rng(n3).standard_normal((*shape, n3)).astype(dtype)
    S = np.fft.rfft(x.astype(np.float64), axis=2).transpose(2, 0, 1)
    X = torch.from_numpy(x).cuda()
    re, im = api.tfft(X)
    got = re.cpu().numpy().astype(np.float64) + 1j * im.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(got - S) < tol * np.linalg.norm(S)
    sr, si = (torch.from_numpy(np.ascontiguousarray(v.astype(dtype))).cuda() for v in (S.real, S.imag))
    y = api.tifft(sr, si, n3).cpu().numpy()
    assert np.linalg.norm(y - x.astype(np.float64)) < tol * np.linalg.norm(x)
