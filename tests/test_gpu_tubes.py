"""GPU parity of the tube transforms over the tube lengths where their kernels
change: one thread per tube (3 to 23), the LDS stages with float64 (up to 256)
and float32 storage, Bluestein's transform (a prime factor above 13), odd and
even lengths, and fewer or more tubes than a workgroup takes.

Tolerances: float32 results round 2^-24 once per pass through float32 storage,
at most 8 passes in a transform (Bluestein: two transforms of at most 3 stages
and two products), so 8 x 6e-8 = 5e-7 bounds the relative Frobenius error of
one transform and twice that a round trip; float64 1e-14 (eps_64 times the
same count and the operations between).
"""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import decomp as D
from oracle import sampling as S
from oracle import tensor as T

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_1704_04362_amd.api")

TOL = {np.float32: 5e-7, np.float64: 1e-14}


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n3", [3, 14, 17, 23, 33, 34, 96, 127, 202, 256, 258, 1001, 1023, 2038, 3000, 4096])
def test_tube_transforms_by_length(n3, dtype):
    if dtype == np.float64 and n3 == 2038:
        n3 = 1018
    for n1, n2 in ((1, 1), (3, 13), (41, 53)):
        X = W.gaussian((n1, n2, n3), seed=n3, salt=n1).astype(dtype)
        re, im = api.tfft(dev(X))
        H = T.half_spectrum(X.astype(np.float64))
        assert T.rel_fro(re.cpu().numpy() + 1j * im.cpu().numpy(), H) < TOL[dtype]
        assert not im[0].any() and (n3 % 2 or not im[-1].any())
        assert T.rel_fro(api.tifft(re, im, n3).cpu().numpy(), X) < 2 * TOL[dtype]


@pytest.mark.parametrize("n3", [17, 80, 101, 600])
def test_tube_transforms_of_picked_slices(n3):
    """Picked, scaled slices (fewer live picks than slots) through these
    transforms: the rt-product against the oracle."""
    A = W.gaussian((9, 70, n3), seed=5)
    B = W.gaussian((70, 11, n3), seed=6)
    w = W.lognormal_weights(70, 3)
    picks = api.tsample("user", 20, mode="bernoulli", seed=2, w=dev(w))
    Z = api.tprod(dev(A), dev(B), picks=picks, prec="f64").cpu().numpy()
    idx, sc = S.sample_bernoulli(w, 20, seed=2)
    assert T.rel_fro(Z, D.rtprod(A, B, idx, sc)) < 1e-12


@pytest.mark.parametrize("n3, shape, dtype", [
    (8320, (1, 1), np.float32),      # 4160 = 20 x 208, one tube
    (10000, (3, 100), np.float32),   # 20 x 250: 256 slots a slice tile, a remainder
    (57122, (1, 9), np.float32),     # 169 x 169: odd pair count, no self-paired middle slice
    (262144, (1, 2), np.float32),    # 512 x 256
    (524288, (1, 1), np.float32),    # 1024 x 256, the longest
    (4100, (2, 65), np.float64),     # 41 is no radix: the direct kernel
    (4116, (2, 65), np.float64),     # 14 x 147
    (524288, (1, 3), np.float64),
])
def test_four_step_tiles(n3, shape, dtype):
    """Tile shapes of the four-step passes against float64 transforms on the
    host. float32: at most 8 roundings through float storage and float
    butterflies of at most log2(N) additions, relative error below
    2^-24 (8 + log2 n3) each way; float64 the same with 2^-53 and twice the
    count, for the host's own error."""
    X = W.gaussian((*shape, n3), seed=n3).astype(dtype)
    tol = 2.0 ** -24 * (8 + np.log2(n3)) if dtype == np.float32 else 2.0 ** -53 * 2 * (8 + np.log2(n3))
    if n3 == 4100:
        tol *= 16  # direct sums of 4100 terms
    re, im = api.tfft(dev(X))
    H = np.fft.rfft(X.astype(np.float64), axis=2).transpose(2, 0, 1)
    got = re.cpu().numpy().astype(np.float64) + 1j * im.cpu().numpy()
    assert got.shape == H.shape
    assert np.linalg.norm(got - H) < tol * np.linalg.norm(H)
    assert not im[0].any() and not im[-1].any()
    Y = api.tifft(re, im, n3).cpu().numpy().astype(np.float64)
    assert np.linalg.norm(Y - X) < 2 * tol * np.linalg.norm(X)


@pytest.mark.parametrize("prec,tol", [("f64", 1e-12), ("f32", 1e-5)])
@pytest.mark.parametrize("n3", [1, 2, 3, 5, 16, 23, 64, 168, 24])
def test_products_with_both_operands_in_one_launch(n3, prec, tol):
    """Both operands of a product transformed by one launch (lengths with a
    tube a thread): operands of one tube, of less and more than a workgroup, a
    sampled one. Tolerances: those of the t-product."""
    dtype = np.float64 if prec == "f64" else np.float32
    for n1, n2, n4 in ((1, 1, 1), (1, 70, 3), (9, 13, 31)):
        A = W.gaussian((n1, n2, n3), seed=n3).astype(dtype)
        B = W.gaussian((n2, n4, n3), seed=n3 + 1).astype(dtype)
        C = api.tprod(dev(A), dev(B), prec=prec).cpu().numpy()
        assert T.rel_fro(C, T.tprod_fft(A.astype(np.float64), B.astype(np.float64))) < tol
    picks = api.tsample("uniform", 7, mode="iid", seed=1, n=13)
    Z = api.tprod(dev(A), dev(B), picks=picks, prec=prec).cpu().numpy()
    idx, sc = picks.host()
    assert T.rel_fro(Z, D.rtprod(A, B, idx.numpy(), sc.numpy())) < tol


def test_product_of_operands_of_more_tubes_together_than_a_launch_holds():
    """2^32 tubes in both operands (20 GB; a launch holds 2^32 work-items): two
    launches. Whole numbers small enough for exact float32 products and sums."""
    n2 = 40_000_000
    A = torch.zeros((64, n2, 1), dtype=torch.float32, device="cuda")
    B = torch.zeros((n2, 64, 1), dtype=torch.float32, device="cuda")
    at = torch.randint(n2, (1000,), generator=torch.Generator().manual_seed(1)).unique().cuda()
    A[:, at] = torch.arange(64 * len(at), device="cuda").remainder(7).float().view(64, -1, 1)
    B[at] = torch.arange(len(at) * 64, device="cuda").remainder(5).float().view(-1, 64, 1)
    C = api.tprod(A, B, prec="f32")
    ref = A[:, at, 0].cpu().double() @ B[at, :, 0].cpu().double()
    api._WS_CACHE.clear()  # (41 GB)
    assert torch.equal(C[..., 0].cpu().double(), ref)


@pytest.mark.parametrize("n3", [499, 998])
def test_scaled_slices_enter_bluesteins_transform_unrounded(n3):
    """Impulses of 1 to 1.02 times a scale just below 1 + 2^-24: rounded to float32
    before the chirp, every scaled value falls back to the impulse, 2^-24 of it,
    and a product of two twice that (at position 7, whose chirp is no power of two
    times 1: the rounding after it is another for every value). The roundings of the transforms and products
    differ from slice to slice and from output to output: their mean over 64 x 64
    outputs of 250 slices or more is a hundredth of 2^-24."""
    s = 1.0 + 0.98 * 2.0 ** -24
    g = np.random.default_rng(n3)
    A, B = np.zeros((64, 1, n3), np.float32), np.zeros((1, 64, n3), np.float32)
    A[:, 0, 7], B[0, :, 7] = 1 + 0.02 * g.random(64), 1 + 0.02 * g.random(64)
    picks = api.Picks(1, "cuda")
    picks.idx.zero_()
    picks.scale.fill_(s)
    picks.count.fill_(1)
    Z = api.tprod(dev(A), dev(B), picks=picks, prec="f32").cpu().numpy().astype(np.float64)
    ref = np.outer(A[:, 0, 7].astype(np.float64), B[0, :, 7].astype(np.float64)) * s * s
    assert abs(np.mean(Z[:, :, 14] / ref - 1)) < 2.0 ** -24
