"""GPU parity of the randomized t-SVD over the widths of its small eigenproblems
(r + p = 1, even and odd ones, 31 and 32: the eight-wavefront solver; 33: the
other one).

Tolerance: an eigenvalue of B^H B is exact to about 2^-53 of the largest times
the width, so a singular value above 1e-2 of the largest (the inputs are of
exact rank with comparable singular values) to 33 x 1e-16 / 1e-4 < 1e-10.
"""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import tensor as T

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_1704_04362_amd.api")


@pytest.mark.parametrize("r,p", [(1, 0), (1, 1), (2, 1), (3, 4), (7, 0), (16, 14), (15, 16), (20, 12), (23, 10)])
def test_tsvd_rand_by_width(r, p):
    A = T.tprod_fft(W.gaussian((60, r, 6), seed=r), W.gaussian((r, 56, 6), seed=p + 50))
    U, S, V, Z = api.tsvd_rand_factors(torch.from_numpy(np.ascontiguousarray(A)).cuda(), r, p=p, q=1, seed=3)
    S = S.cpu().numpy()
    for k, H in enumerate(T.half_spectrum(A)):
        sv = np.linalg.svd(H, compute_uv=False)[:r]
        assert np.abs(S[k] - sv).max() < 1e-10 * sv[0]
    assert T.rel_fro(Z.cpu().numpy(), A) < 1e-10
    for Q in (U, V):
        G = T.half_spectrum(Q.cpu().numpy())
        assert max(np.abs(g.conj().T @ g - np.eye(r)).max() for g in G) < 1e-10
