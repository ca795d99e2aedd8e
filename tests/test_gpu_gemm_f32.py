"""GPU parity of the float32 per-slice products on the float32 matrix cores at
the edges of their two tile sizes (64 and 128 rows and columns, 16-deep steps of
the contraction), every pair of operations, real and complex last slices.

Tolerance: every one of Kd additions rounds by at most 2^-24 of its partial
sum, at random; the three-product form doubles the error: 2^-24 sqrt(Kd) x 4 of
the result's norm.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_1704_04362_amd.api")

SHAPES = [(1, 65, 65, 64), (3, 64, 128, 79), (2, 127, 129, 65), (5, 192, 193, 80), (9, 257, 66, 96),
          (40, 130, 129, 64), (33, 256, 256, 65), (2, 700, 640, 100)]


@pytest.mark.parametrize("K,M,N,Kd", SHAPES)
@pytest.mark.parametrize("op_a,op_b", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("real_last", [False, True])
def test_f32_products_at_tile_edges(K, M, N, Kd, op_a, op_b, real_last):
    g = np.random.default_rng([K, M, N, Kd])
    A = g.standard_normal((2, K, Kd, M) if op_a else (2, K, M, Kd)).astype(np.float32)
    B = g.standard_normal((2, K, N, Kd) if op_b else (2, K, Kd, N)).astype(np.float32)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    re, im = api.spectrum_matmul((dev(A[0]), dev(A[1])), (dev(B[0]), dev(B[1])), op_a, op_b, real_last=real_last,
                                 prec="f32")
    for k in range(K):
        real = k == 0 or (real_last and k == K - 1)
        a = A[0, k].astype(np.float64) + (0 if real else 1j * A[1, k])
        b = B[0, k].astype(np.float64) + (0 if real else 1j * B[1, k])
        ref = (a.conj().T if op_a else a) @ (b.conj().T if op_b else b)
        got = re[k].cpu().numpy() + 1j * im[k].cpu().numpy()
        assert np.linalg.norm(got - ref) <= 2.0 ** -24 * np.sqrt(Kd) * 4 * np.linalg.norm(ref)


def test_f32_products_of_rows_beyond_32_bit_tile_offsets():
    """Rows of 2^23 + 3 values (offsets in a tile of 64 bits), both operands read
    along the contraction; the reference in float64 on the same device, a block of the
    contraction at a time. Tolerance as above, over 2^23 additions."""
    Kd, M, N = 2 ** 23 + 3, 17, 66
    g = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda n: torch.randn((2, n, Kd), device="cuda", generator=g)  # noqa: E731
    a, b = (rnd(M), rnd(M)), (rnd(N), rnd(N))
    re, im = api.spectrum_matmul(a, b, 0, 1, real_last=False, prec="f32")
    ref = torch.zeros((2, 2, M, N), dtype=torch.float64, device="cuda")  # (re, im) per slice
    for k0 in range(0, Kd, 2 ** 20):
        ar, ai = (t[..., k0:k0 + 2 ** 20].double() for t in a)
        br, bi = (t[..., k0:k0 + 2 ** 20].double() for t in b)
        for k in range(2):  # A B^H; slice 0 is real
            ref[k, 0] += ar[k] @ br[k].T.contiguous()
            if k:
                ref[k, 0] += ai[k] @ bi[k].T.contiguous()
                ref[k, 1] += ai[k] @ br[k].T.contiguous() - ar[k] @ bi[k].T.contiguous()
    err = torch.stack((re.double(), im.double()), 1) - ref
    for k in range(2):
        assert err[k].norm() <= 2.0 ** -24 * Kd ** 0.5 * 4 * ref[k].norm()


@pytest.mark.parametrize("M", [64 * 65535, 64 * 65535 + 1])
@pytest.mark.parametrize("N", [20, 150])
def test_f32_products_of_very_many_rows(M, N):
    """As many rows as the grid holds in tiles of 64, and one more (tiles of 128).
    Either tile, and a product of the last rows alone, adds an output's products
    in the same order: the same bits; the vector kernel, whose complex products take
    four real ones, gives others."""
    g = torch.Generator(device="cuda").manual_seed(N)
    rnd = lambda *s: torch.randn(s, device="cuda", generator=g)  # noqa: E731
    a, b = (rnd(2, M, 64), rnd(2, M, 64)), (rnd(2, N, 64), rnd(2, N, 64))
    re, im = api.spectrum_matmul(a, b, 0, 1, real_last=False, prec="f32")
    for rows in (slice(0, 200), slice(M - 200, M)):
        few = api.spectrum_matmul(tuple(t[:, rows].contiguous() for t in a), b, 0, 1, real_last=False, prec="f32")
        assert torch.equal(re[:, rows], few[0]) and torch.equal(im[:, rows], few[1])
