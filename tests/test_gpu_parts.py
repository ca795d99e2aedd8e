"""GPU parity of products with few output tiles, whose contraction is cut into
parts: lengths around the shortest that is cut (256), parts of unequal length,
picks whose count (read on the device) leaves parts empty; tube lengths with
pre-split operands (8) and without (5); narrow results (at most 64 columns).

Tolerances: float32 1e-5, the bound stated for the t-product; bf16x3 1.3e-5
and bf16 1e-2 (2^-16 and 2^-8 dropped per product).
"""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import decomp as D
from oracle import tensor as T

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_1704_04362_amd.api")

TOL = {"f32": 1e-5, "bf16x3": 1.3e-5, "bf16": 1e-2}


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("prec", sorted(TOL))
@pytest.mark.parametrize("n3", [5, 8])
@pytest.mark.parametrize("n1,n2,n4", [(65, 255, 66), (65, 256, 66), (129, 545, 127), (70, 2049, 300),
                                      (70, 300, 33), (129, 1030, 64), (33, 257, 1)])
def test_products_in_parts(n1, n2, n4, n3, prec):
    A = W.gaussian((n1, n2, n3), seed=n2).astype(np.float32)
    B = W.gaussian((n2, n4, n3), seed=n2 + 1).astype(np.float32)
    C = api.tprod(dev(A), dev(B), prec=prec).cpu().numpy()
    assert T.rel_fro(C, T.tprod_fft(A.astype(np.float64), B.astype(np.float64))) < TOL[prec]


@pytest.mark.parametrize("prec", ["f32", "bf16x3"])
@pytest.mark.parametrize("n3", [5, 8])
@pytest.mark.parametrize("c", [3, 40, 300])
def test_rtproducts_in_parts_of_the_live_count(c, n3, prec):
    A = W.gaussian((66, 1500, n3), seed=7).astype(np.float32)
    B = W.gaussian((1500, 67, n3), seed=8).astype(np.float32)
    picks = api.tsample("norm2", c, mode="bernoulli", seed=4, A=dev(A))
    Z = api.tprod(dev(A), dev(B), picks=picks, prec=prec).cpu().numpy()
    idx, sc = picks.host()
    assert T.rel_fro(Z, D.rtprod(A, B, idx.numpy(), sc.numpy())) < TOL[prec]
