"""Tube transforms of lengths with a prime factor above 13: dense products with the
roots of unity, compared with long double transforms over the sizes where the
kernel's blocks of outputs, terms and tubes begin and end, both ways separately."""
import math

import numpy as np
import pytest
import scipy.fft
import torch

from oracle import tensor as T

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_1704_04362_amd.api")


def bound(n, dtype):
    """A random walk of roundings of at most 2^-53 each: of the folding, the roots and
    the twiddles, of sums of up to 32 terms and of the blocks' sums (half of the
    steps weigh in, as partial sums grow evenly); float32 rounds its results once."""
    H = n // (2 if n % 2 else 4) + 1
    walk = 2.0 ** -53 * math.sqrt(3 + min(H, 32) / 2 + H / 64)
    return walk if dtype == np.float64 else walk + 2.0 ** -24


def rel(x, y):
    d = np.abs(x.astype(y.dtype) - y)
    return float(np.sqrt((d * d).sum() / (np.abs(y) ** 2).sum()))


CASES = [(n, t, np.float64) for n in (29, 31, 34, 37, 61, 62, 67, 122, 124, 127, 131, 134, 254, 262, 1018, 1021)
         for t in (1, 17, 65)]
CASES += [(n, t, np.float32) for n in (31, 62, 131, 499, 514) for t in (3, 130)]
CASES += [(67, 16449, np.float64), (131, 8257, np.float64), (134, 8225, np.float64), (262, 4130, np.float32),
          (2038, 9, np.float64), (2039, 9, np.float64), (4093, 5, np.float64), (8191, 5, np.float32)]


@pytest.mark.parametrize("n,tubes,dtype", CASES)
def test_dense_transforms(n, tubes, dtype):
    x = np.random.default_rng([n, tubes]).standard_normal((1, tubes, n)).astype(dtype)
    S = scipy.fft.rfft(x.astype(np.longdouble), axis=2)
    re, im = (v.cpu().numpy() for v in api.tfft(torch.from_numpy(x).cuda()))
    got = (re.astype(np.longdouble) + 1j * im.astype(np.longdouble)).transpose(1, 2, 0)
    assert rel(got, S) < bound(n, dtype)
    assert not im[0].any() and (n % 2 or not im[-1].any())
    # the inverse of the spectrum as stored, whose first (and last) slices are real
    sr, si = (np.ascontiguousarray(v.astype(dtype).transpose(2, 0, 1)) for v in (S.real, S.imag))
    y = scipy.fft.irfft((sr + 1j * si.astype(np.longdouble)).transpose(1, 2, 0), n=n, axis=2)
    si[0] = 7.0  # dropped
    if n % 2 == 0:
        si[-1] = -3.0
    back = api.tifft(torch.from_numpy(sr).cuda(), torch.from_numpy(si).cuda(), n).cpu().numpy()
    assert rel(back, y) < bound(n, dtype)


@pytest.mark.parametrize("n3", [31, 62, 134])
def test_dense_transforms_of_picked_slices(n3):
    g = np.random.default_rng(n3)
    A, B = g.standard_normal((5, 40, n3)), g.standard_normal((40, 19, n3))
    picks = api.tsample("norm2", 23, mode="iid", seed=4, A=torch.from_numpy(A).cuda())
    Z = api.tprod(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), picks=picks, prec="f64").cpu().numpy()
    idx, sc = (v.numpy() for v in picks.host())
    ref = T.tprod_fft(A[:, idx] * sc[None, :, None], B[idx] * sc[:, None, None])
    assert T.rel_fro(Z, ref) < 1e-14
