"""GPU parity of the lateral slice norms where their kernel's split changes:
tubes that are no multiple of a 16-byte piece, short tubes (several times 32 of
them a workgroup), partial blocks of rows and of tubes, a run that ends inside
a piece.

Tolerance: sums of n1 n3 squares in float64, each addition rounding by 2^-53
of a partial sum that is at most the result: n1 n3 2^-53, at most 5e-13 here.
"""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_1704_04362_amd.api")


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("shape", [(1, 1, 1), (17, 1025, 1), (16, 515, 2), (33, 401, 3), (5, 257, 4), (15, 193, 5),
                                   (31, 65, 30), (18, 33, 64), (3, 31, 101), (16, 5, 255)])
def test_lateral_norms_by_tube_length(shape, dtype):
    A = W.gaussian(shape, seed=shape[1]).astype(dtype)
    want = (A.astype(np.float64) ** 2).sum(axis=(0, 2))
    got = api.slice_norms(torch.from_numpy(A).cuda()).cpu().numpy()
    assert np.abs(got / want - 1).max() < 5e-13
