"""Forward transforms against complex spectra, and inverse transforms of the oracle's
spectrum alone: the real and the imaginary parts and the sign of the exponent are
each pinned, at a length of every kernel (one tube a thread, packed registers, LDS,
dense products, four-step).

Tolerances: float64 1e-14; float32 4e-7, some 40 roundings of 2^-24 in a random
walk (the packed kernels and the four-step passes have float32 butterflies).
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_1704_04362_amd.api")

LENGTHS = [2, 3, 4, 5, 8, 10, 14, 16, 17, 18, 20, 21, 22, 23, 33, 34, 50, 64, 96, 100, 127, 128, 168, 202, 256, 258,
           1001, 1018, 1023, 2038, 3000, 4096, 10000, 65536]


@pytest.mark.parametrize("dtype,tol", [(np.float64, 1e-14), (np.float32, 4e-7)])
@pytest.mark.parametrize("n3", LENGTHS)
def test_complex_spectra(n3, dtype, tol):
    x = np.random.default_rng(n3).standard_normal((3, 5, n3)).astype(dtype)
    S = np.fft.rfft(x.astype(np.float64), axis=2).transpose(2, 0, 1)
    re, im = (v.cpu().numpy().astype(np.float64) for v in api.tfft(torch.from_numpy(x).cuda()))
    assert np.linalg.norm(re + 1j * im - S) < tol * np.linalg.norm(S)
    sr, si = (torch.from_numpy(np.ascontiguousarray(v.astype(dtype))).cuda() for v in (S.real, S.imag))
    y = api.tifft(sr, si, n3).cpu().numpy()
    assert np.linalg.norm(y - x.astype(np.float64)) < tol * np.linalg.norm(x)
