"""Narrow sampled products (at most 64 columns) in parts whose count of picks is read
on the device: few picks of many slots leave parts short or empty. Tolerances as in
test_gpu_parts.py."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import decomp as D
from oracle import tensor as T

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_1704_04362_amd.api")

TOL = {"f32": 1e-5, "bf16x3": 1.3e-5}


@pytest.mark.parametrize("prec", sorted(TOL))
@pytest.mark.parametrize("n4", [1, 20, 33, 64])
@pytest.mark.parametrize("c", [3, 40, 300, 1400])
def test_narrow_rtproducts_in_parts_of_the_live_count(c, n4, prec):
    A = W.gaussian((70, 1500, 5), seed=7).astype(np.float32)
    B = W.gaussian((1500, n4, 5), seed=8).astype(np.float32)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    picks = api.tsample("norm2", c, mode="bernoulli", seed=4, A=dev(A))
    Z = api.tprod(dev(A), dev(B), picks=picks, prec=prec).cpu().numpy()
    idx, sc = picks.host()
    assert T.rel_fro(Z, D.rtprod(A, B, idx.numpy(), sc.numpy())) < TOL[prec]
