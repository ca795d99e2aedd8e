"""GPU parity of the float64 per-slice products at the edges of their tiles (16,
32 and 64 rows and columns, 16-deep steps of the contraction), every pair of
operations, real and complex last slices.

Tolerance: a sum of 4 Kd products of unit-variance values rounds at 2^-53 of
its size once per product, sqrt(4 Kd) of them at random: 1e-14 sqrt(Kd) of the
result's norm is 45 times that.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_1704_04362_amd.api")

SHAPES = [(1, 1, 1, 1), (2, 16, 16, 4), (3, 17, 31, 15), (9, 33, 65, 16), (5, 64, 32, 48), (30, 65, 33, 17),
          (4, 130, 190, 33), (2, 700, 640, 5)]


@pytest.mark.parametrize("K,M,N,Kd", SHAPES)
@pytest.mark.parametrize("op_a,op_b", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("real_last", [False, True])
def test_f64_products_at_tile_edges(K, M, N, Kd, op_a, op_b, real_last):
    g = np.random.default_rng([K, M, N, Kd])
    A = g.standard_normal((K, Kd, M) if op_a else (K, M, Kd)) + 0j
    B = g.standard_normal((K, N, Kd) if op_b else (K, Kd, N)) + 0j
    A.imag = g.standard_normal(A.shape)
    B.imag = g.standard_normal(B.shape)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    re, im = api.spectrum_matmul((dev(A.real), dev(A.imag)), (dev(B.real), dev(B.imag)), op_a, op_b,
                                 real_last=real_last, prec="f64")
    for k in range(K):
        a, b = A[k], B[k]
        if k == 0 or (real_last and k == K - 1):
            a, b = a.real, b.real
        ref = (a.conj().T if op_a else a) @ (b.conj().T if op_b else b)
        got = re[k].cpu().numpy() + 1j * im[k].cpu().numpy()
        assert np.linalg.norm(got - ref) <= 1e-14 * np.sqrt(Kd) * np.linalg.norm(ref)


@pytest.mark.parametrize("K,N", [(1, 2 ** 29 + 70), (30, 2 ** 24 * 32 // 30 + 5)])
def test_f64_products_of_more_tiles_than_a_grid_row_holds(K, N):
    """2^24 tiles and a few more (a launch's x extent holds 2^32 work-items), in
    the round-robin order and in runs per XCD. Products of one term: exact."""
    a = torch.full((K, 1, 1), 3.0, dtype=torch.float64, device="cuda")
    b = torch.arange(K * N, dtype=torch.float64, device="cuda").view(K, 1, N)
    re, im = api.spectrum_matmul((a, a), (b, b), real_last=False, prec="f64")
    assert torch.equal(re[0], 3.0 * b[0]) and not im[0].any()
    if K > 1:  # (3 + 3i)(b + bi) = 6bi
        assert not re[1:].any() and torch.equal(im[1:], 6.0 * b[1:])
