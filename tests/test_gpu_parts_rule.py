"""Products of pre-split operands on both sides of the rule that cuts a contraction
into parts: lengths around those from which parts pay for summing their planes, by
precision and by number of output tiles. Tolerances as in test_gpu_parts.py."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import tensor as T

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_1704_04362_amd.api")

TOL = {"bf16x3": 1.3e-5, "bf16": 1e-2}


@pytest.mark.parametrize("prec", sorted(TOL))
@pytest.mark.parametrize("n1,n2,n4,n3", [(40, 223, 40, 4), (40, 256, 40, 4), (40, 289, 40, 4), (40, 321, 40, 4),
                                         (9, 640, 9, 1), (9, 1030, 9, 1), (300, 385, 260, 16), (512, 512, 512, 16),
                                         (512, 1024, 512, 16)])
def test_products_around_the_rule_for_parts(n1, n2, n4, n3, prec):
    A = W.gaussian((n1, n2, n3), seed=n2).astype(np.float32)
    B = W.gaussian((n2, n4, n3), seed=n2 + 1).astype(np.float32)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    C = api.tprod(dev(A), dev(B), prec=prec).cpu().numpy()
    assert T.rel_fro(C, T.tprod_fft(A.astype(np.float64), B.astype(np.float64))) < TOL[prec]
