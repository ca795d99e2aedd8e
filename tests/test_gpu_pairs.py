"""GPU parity of the pair step of the block Jacobi (Gram matrix, inner sweep and
rotations of two 16-row blocks) at the edges of its tiles: partial and empty row
blocks (16 rows), partial groups of 16 and tiles of 32 columns, odd column
counts, and one to several round-robin rounds.

Tolerance: a converged pair has inner products below 1e-6 of the larger squared
row norm, and rows are rounded to float32 (6e-8) once per rotation, about a
dozen sweeps of them at random: 1e-5 of ||M|| bounds both.
"""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import decomp as D

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_1704_04362_amd.api")


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("n1,n2", [(2, 2), (2, 3), (15, 16), (16, 33), (17, 31), (33, 34), (48, 65), (63, 15), (50, 129)])
@pytest.mark.parametrize("n3", [1, 4, 9])
def test_thresholding_at_tile_edges(n1, n2, n3):
    M = W.gaussian((n1, n2, n3), seed=31 * n1 + n2, salt=n3).astype(np.float32)
    tau = 0.5 * float(np.sqrt(n3 * max(n1, n2)))
    L, ranks, unc = api.tsvt(dev(M), tau, with_unconverged=True)
    ref, rr = D.tsvt(M, tau)
    assert np.linalg.norm(L.cpu().numpy() - ref) < 1e-5 * np.linalg.norm(M)
    assert np.array_equal(ranks.cpu().numpy(), rr) and int(unc) == 0
