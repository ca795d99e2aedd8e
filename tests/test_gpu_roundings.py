"""Float32 tube transforms in LDS round no more often than one mixed-radix transform
of the whole tube in stages of 4, 2, 3, 5, 7, 11 and 13 that stores float32 values
after every stage: lengths of four times an odd number, whose packed half has a 2
left over, and inverses, whose division by the length is no rounding of its own."""
import math

import numpy as np
import pytest
import scipy.fft
import torch

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_1704_04362_amd.api")

# root mean square of the relative rounding error of a float32 value, over
# logarithmically spread values: 2^-24 sqrt(1/3 x 3/8 / ln 2); 2 % for the sample
ROUNDING = 1.02 * 2.0 ** -24 * math.sqrt(0.125 / math.log(2))


def stages(n):
    s = 0
    for p in (4, 2, 3, 5, 7, 11, 13):
        while n % p == 0:
            n //= p
            s += 1
    return s


@pytest.mark.parametrize("n", [308, 364, 484, 520, 572, 676, 924, 1372, 2000, 2156, 3696, 4004, 5324, 7436])
def test_float32_roundings(n):
    x = np.random.default_rng(n).standard_normal((1, 300, n)).astype(np.float32)
    S = scipy.fft.rfft(x.astype(np.float64), axis=2)
    re, im = (v.cpu().numpy().transpose(1, 2, 0) for v in api.tfft(torch.from_numpy(x).cuda()))
    most = ROUNDING * math.sqrt(stages(n))
    assert np.linalg.norm(re + 1j * im.astype(np.float64) - S) < most * np.linalg.norm(S)
    sr, si = (np.ascontiguousarray(v.astype(np.float32).transpose(2, 0, 1)) for v in (S.real, S.imag))
    y = scipy.fft.irfft((sr + 1j * si.astype(np.float64)).transpose(1, 2, 0), n=n, axis=2)
    back = api.tifft(torch.from_numpy(sr).cuda(), torch.from_numpy(si).cuda(), n).cpu().numpy()
    assert np.linalg.norm(back - y) < most * np.linalg.norm(y)
