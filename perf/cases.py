"""Performance cases of the t-product library: the calls a program makes on
its public entry points, over the sizes the library is used at.

listed() names the cases, draw() gives further ones of the same ranges,
prepare() builds what a program holds before the call (inputs on the GPU, the
network of the learned proposal), run() makes one pass, work() counts the
bytes and operations a pass cannot do without, and exact() gives the same
results in float64 from plain torch and numpy.
"""
import math

import numpy as np
import torch

from paper_1704_04362_amd import api

PRECS = ("f64", "f32", "bf16x3")


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # the smallest exact pair: a program that multiplies many small
        # float64 tensors one after the other, bound by launches and the host
        {"name": "tprod_small_f64", "kind": "tprod", "n1": 64, "n2": 48, "n4": 32, "n3": 16, "prec": "f64"},
        # double precision data at its default precision, ragged sides and a
        # tube length without a power of two
        {"name": "tprod_f64", "kind": "tprod", "n1": 257, "n2": 380, "n4": 201, "n3": 60, "prec": "f64"},
        # float32 data at its default precision: ragged sides, the tube
        # length of an 80-frame video
        {"name": "tprod_f32", "kind": "tprod", "n1": 301, "n2": 777, "n4": 259, "n3": 80, "prec": "f32"},
        # the t-product workload of the benchmark
        {"name": "tprod_bf16x3", "kind": "tprod", "n1": 512, "n2": 2048, "n4": 512, "n3": 64, "prec": "bf16x3"},
        # its randomized product: squared-norm picks, then the sampled product
        {"name": "rtprod", "kind": "rtprod", "n1": 512, "n2": 2048, "n4": 512, "n3": 64, "c": 256, "prec": "bf16x3"},
        # the randomized Gram product of a very long tensor (l = r ln r of
        # 10^5 slices, five frames)
        {"name": "rtprod_tall", "kind": "rtprod", "n1": 300, "n2": 100000, "n4": 300, "n3": 5, "c": 1700,
         "prec": "bf16x3"},
        # transforms both ways at the shape of the smaller imaging data set
        {"name": "transforms_2000", "kind": "transforms", "n1": 122, "n2": 120, "n3": 2000, "prec": "f32"},
        # and at the tube length of the larger one, on a part of its pixels
        {"name": "transforms_500000", "kind": "transforms", "n1": 24, "n2": 24, "n3": 500000, "prec": "f32"},
        # t-CUR with exact leverage scores on both sides (range finder on the
        # whole tensor), the benchmark's low-rank tensor
        {"name": "tcur_lev", "kind": "tcur", "n1": 1024, "n2": 1024, "n3": 128, "r": 20, "c": 60, "cols": "lev",
         "prec": "bf16x3"},
        # t-CUR of the imaging data: uniform columns, rows by leverage of C,
        # a thousand Fourier slices of small sides
        {"name": "tcur_2000", "kind": "tcur", "n1": 122, "n2": 120, "n3": 2000, "r": 5, "c": 45, "cols": "uniform",
         "prec": "f32"},
        # ADMM iterations of tensor completion (half of the entries observed)
        {"name": "complete", "kind": "complete", "n1": 256, "n2": 256, "n3": 100, "r": 15, "iters": 10},
        # a training step of the learned proposal, a batch of 16 tensors
        {"name": "mlp_step", "kind": "mlp", "T": 16, "n": 512},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _smooth(n, most=7):
    for p in (2, 3, 5, 7):
        while p <= most and n % p == 0:
            n //= p
    return n == 1


def _near_smooth(rng, lo, hi, even=False):
    """A length between lo and hi whose prime factors are 2, 3, 5 and 7 (what
    data sets are cut or padded to)."""
    n = _log_int(rng, lo, hi)
    while not (_smooth(n) and not (even and n % 2)):
        n -= 1
    return max(n, lo)


def _tube(rng, lo, hi):
    """A tube length: half of them any whole number, half smooth ones."""
    return _log_int(rng, lo, hi) if rng.random() < 0.5 else _near_smooth(rng, lo, hi)


def draw(rng):
    kind = rng.choice(["tprod", "tprod", "rtprod", "transforms", "transforms", "tcur", "complete", "mlp"])
    if kind in ("tprod", "rtprod"):
        prec = rng.choice(PRECS)
        cap = {"f64": 1.5e10, "f32": 5e10, "bf16x3": 1.3e11}[prec]
        tall = kind == "rtprod" and rng.random() < 0.4
        while True:
            n1, n4 = _log_int(rng, 16, 1024), _log_int(rng, 16, 1024)
            n2 = _log_int(rng, 10000, 100000) if tall else _log_int(rng, 16, 2048)
            n3 = _tube(rng, 3, 12) if tall else _tube(rng, 4, 200)
            big = max(n1, n4) * n2 * n3
            if _tprod_flops(n1, n2, n4, n3) <= cap and big <= 1.5e8:
                break
        case = {"kind": kind, "n1": n1, "n2": n2, "n4": n4, "n3": n3, "prec": prec}
        if kind == "rtprod":
            case["c"] = max(1, min(n2, _log_int(rng, 16, 2048)))
        return case
    if kind == "transforms":
        if rng.random() < 0.3:
            n3, total = _near_smooth(rng, 10000, 500000, even=True), 2.8e8
        else:
            n3, total = _tube(rng, 16, 2048), 3e7
        rows = _log_int(rng, 4, 160)
        cols = max(1, min(_log_int(rng, 4, 160), int(total / n3 / rows)))
        return {"kind": "transforms", "n1": rows, "n2": cols, "n3": n3, "prec": rng.choice(["f32", "f32", "f64"])
                if n3 <= 2048 else "f32"}
    if kind == "tcur":
        if rng.random() < 0.5:
            n1, n2, n3 = _log_int(rng, 200, 1024), _log_int(rng, 200, 1024), _near_smooth(rng, 16, 128)
        else:
            n1, n2, n3 = _log_int(rng, 64, 160), _log_int(rng, 64, 160), _near_smooth(rng, 200, 2000)
        r = rng.randint(3, 20)
        return {"kind": "tcur", "n1": n1, "n2": n2, "n3": n3, "r": r, "c": rng.randint(2 * r, 60),
                "cols": rng.choice(["uniform", "norm2"]), "prec": rng.choice(["f32", "bf16x3"])}
    if kind == "complete":
        return {"kind": "complete", "n1": _log_int(rng, 48, 256), "n2": _log_int(rng, 48, 256),
                "n3": _near_smooth(rng, 16, 100), "r": rng.randint(3, 15), "iters": rng.randint(5, 10)}
    return {"kind": "mlp", "T": rng.randint(1, 32), "n": _log_int(rng, 64, 1024)}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _gen(seed, salt=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + salt)
    return g


def _randn(g, *shape, dtype=torch.float32):
    return torch.randn(shape, generator=g, device="cuda", dtype=dtype)


def _low_rank(g, n1, n2, n3, r, noise):
    """A tensor of tubal rank r plus Gaussian noise of standard deviation
    `noise`, composed slice by slice in the Fourier domain."""
    f = torch.fft.rfft(_randn(g, n1, r, n3), dim=2).permute(2, 0, 1).contiguous()
    h = torch.fft.rfft(_randn(g, r, n2, n3), dim=2).permute(2, 0, 1).contiguous()
    A = torch.fft.irfft(torch.bmm(f, h).permute(1, 2, 0).contiguous(), n=n3, dim=2)
    return (A + noise * _randn(g, n1, n2, n3)).contiguous()


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    dtype = torch.float64 if case.get("prec") == "f64" else torch.float32
    state = {"case": case, "seed": int(seed)}
    if kind in ("tprod", "rtprod"):
        # lognormal scales on the contracted slices: the products whose
        # squared-norm probabilities are worth sampling by
        n1, n2, n4, n3 = case["n1"], case["n2"], case["n4"], case["n3"]
        a = torch.exp(_randn(g, n2, dtype=dtype))
        b = torch.exp(_randn(g, n2, dtype=dtype))
        state["A"] = (_randn(g, n1, n2, n3, dtype=dtype) * a[None, :, None]).contiguous()
        state["B"] = (_randn(g, n2, n4, n3, dtype=dtype) * b[:, None, None]).contiguous()
    elif kind == "transforms":
        state["X"] = _randn(g, case["n1"], case["n2"], case["n3"], dtype=dtype)
    elif kind == "tcur":
        state["A"] = _low_rank(g, case["n1"], case["n2"], case["n3"], case["r"], math.sqrt(1e-3))
    elif kind == "complete":
        L = _low_rank(g, case["n1"], case["n2"], case["n3"], case["r"], 0.1)
        state["mask"] = (torch.rand(L.shape, generator=g, device="cuda") < 0.5).to(torch.uint8)
        state["X"] = (L * state["mask"].to(L.dtype)).contiguous()
    else:
        T, n = case["T"], case["n"]
        w = [_randn(g, 17, 128) * math.sqrt(2 / 17), 0.01 * _randn(g, 128), _randn(g, 128, 128) * math.sqrt(2 / 128),
             0.01 * _randn(g, 128), _randn(g, 128) * math.sqrt(1 / 128), 0.01 * _randn(g, 1)]
        state["params"] = torch.cat([x.reshape(-1) for x in w]).contiguous()
        state["m"] = torch.zeros_like(state["params"])
        state["v"] = torch.zeros_like(state["params"])
        state["feat"] = _randn(g, T * n, 17)
        state["target"] = torch.exp(_randn(g, T, n))
        state["step"] = 0
    return state


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "tprod":
        return api.tprod(state["A"], state["B"], prec=case["prec"])
    if kind == "rtprod":
        picks = api.tsample("norm2", case["c"], mode="iid", seed=state["seed"], A=state["A"])
        Z = api.tprod(state["A"], state["B"], picks=picks, prec=case["prec"])
        return {"Z": Z, "idx": picks.idx, "scale": picks.scale}
    if kind == "transforms":
        re, im = api.tfft(state["X"])
        return {"re": re, "im": im, "x": api.tifft(re, im, case["n3"])}
    if kind == "tcur":
        cols = case["cols"]
        Z, c, l = api.tcur(state["A"], case["c"], case["c"], case["r"], col_kind=cols, row_kind="lev",
                           mode="uniform" if cols == "uniform" else "iid", row_mode="iid", seed=state["seed"],
                           prec=case["prec"])
        return {"Z": Z, "cols": c.idx, "rows": l.idx}
    if kind == "complete":
        L, E, Y, ranks = api.tcomplete(state["X"], state["mask"], iters=case["iters"])
        return {"L": L, "E": E, "Y": Y, "ranks": ranks}
    state["step"] += 1
    loss, grad = api.mlp_train_step(state["params"], state["m"], state["v"], state["step"], 2e-3, state["feat"],
                                    state["target"], want_grad=True)
    return {"loss": loss, "grad": grad, "params": state["params"], "m": state["m"], "v": state["v"]}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------

def _tprod_flops(n1, n2, n4, n3):
    """Slice products: 8 operations per complex multiply-add, 2 in the real
    slices (the first, and the last of an even tube length)."""
    K, real = n3 // 2 + 1, 2 if n3 % 2 == 0 else 1
    return (8 * (K - real) + 2 * real) * n1 * n2 * n4


def _fft_flops(tubes, n3):
    return 2.5 * tubes * n3 * math.log2(max(n3, 2))


def work(case):
    kind = case["kind"]
    n1, n2, n3 = case.get("n1", 0), case.get("n2", 0), case.get("n3", 1)
    el = 8 if case.get("prec") == "f64" else 4
    K = n3 // 2 + 1
    if kind == "tprod":
        n4 = case["n4"]
        return {"bytes": el * n3 * (n1 * n2 + n2 * n4 + n1 * n4),
                "flops": _tprod_flops(n1, n2, n4, n3) + _fft_flops(n1 * n2 + n2 * n4 + n1 * n4, n3)}
    if kind == "rtprod":
        n4, c = case["n4"], case["c"]
        return {"bytes": el * n3 * (n1 * n2 + min(c, n2) * n4 + n1 * n4),
                "flops": 2 * n1 * n2 * n3 + _tprod_flops(n1, c, n4, n3) + _fft_flops((n1 + n4) * c + n1 * n4, n3)}
    if kind == "transforms":
        return {"bytes": 2 * el * n1 * n2 * (n3 + 2 * K), "flops": 2 * _fft_flops(n1 * n2, n3)}
    if kind == "tcur":
        c, r = case["c"], case["r"]
        flops = _tprod_flops(n1, c, r, n3) + _tprod_flops(r, c, n2, n3) + _tprod_flops(n1, r, n2, n3)
        flops += _fft_flops(n1 * n2 + c * (n1 + n2), n3)
        if case["cols"] == "lev":  # the sketch, one power iteration and the projection of the range finder
            flops += 4 * _tprod_flops(n1, n2, r + 10, n3) + _fft_flops(n1 * n2, n3)
        read = n1 * n2 if case["cols"] in ("lev", "norm2") else c * (n1 + n2)
        return {"bytes": el * n3 * (read + n1 * n2), "flops": flops}
    if kind == "complete":
        s, t = min(n1, n2), max(n1, n2)
        # per iteration: a transform each way, one factorization of each slice
        # (its Gram matrix, the eigenproblem, the two products that shrink it)
        # and the elementwise update of L, E and Y
        it = 2 * _fft_flops(n1 * n2, n3) + K * 8 * (3 * s * s * t + 4 * s ** 3)
        return {"bytes": n1 * n2 * n3 * (5 + 12) + case["iters"] * n1 * n2 * n3 * 24, "flops": case["iters"] * it}
    rows, P = case["T"] * case["n"], 18945
    return {"bytes": 4 * rows * 18 + 4 * P * 8, "flops": 6 * rows * (17 * 128 + 128 * 128 + 128)}


# ---------------------------------------------------------------------------
# The same results in float64
# ---------------------------------------------------------------------------

def _spec(X):
    """Half spectrum, K x n1 x n2; the real slices exactly real."""
    S = torch.fft.rfft(X.double(), dim=2)
    return S.permute(2, 0, 1).contiguous()


def _unspec(S, n3):
    return torch.fft.irfft(S.permute(1, 2, 0).contiguous(), n=n3, dim=2)


def _words(n, seed, stream):
    """Word 0 of the Philox4x64-10 blocks at counters 0 .. n-1."""
    bits = np.random.Philox(counter=(1 << 256) - 1, key=np.array([seed, stream], dtype=np.uint64))
    return [int(v) for v in bits.random_raw(4 * n)[::4]]


def _iid(w, c, seed, stream):
    """c draws with replacement from whole-number weights floor(w 2^(B-e))."""
    w = [float(v) for v in w]
    n = len(w)
    top = 62 - max(0, math.ceil(math.log2(n)))
    e = math.frexp(max(w))[1]
    q = [math.floor(math.ldexp(v, top - e)) for v in w]
    sums = np.cumsum(np.array(q, dtype=np.int64))
    S = int(sums[-1])
    idx = [int(np.searchsorted(sums, (u * S) >> 64, side="right")) for u in _words(c, seed, stream)]
    return idx, [1 / math.sqrt(c * q[j] / S) for j in idx]


def _uniform(n, c, seed, stream):
    keys = _words(n, seed, stream)
    idx = sorted(sorted(range(n), key=lambda i: (keys[i], i))[:c])
    return idx, [math.sqrt(n / c)] * c


def _svd(M):
    """Slice SVDs on the host."""
    return torch.linalg.svd(M.cpu(), full_matrices=False)


def _exact_tcur(case, s):
    n1, n2, n3, r, c = case["n1"], case["n2"], case["n3"], case["r"], case["c"]
    A = s["A"]
    if case["cols"] == "uniform":
        ci, cs = _uniform(n2, c, s["seed"], 0)
    else:
        ci, cs = _iid(A.double().square().sum(dim=(0, 2)).tolist(), c, s["seed"], 0)
    t = lambda v: torch.tensor(v, dtype=torch.float64, device=A.device)  # noqa: E731
    C = _spec(A[:, ci]) * t(cs)[None, None, :]
    U = _svd(C)[0][:, :, :r]
    wk = torch.full((n3 // 2 + 1,), 2.0, dtype=torch.float64)
    wk[0] = 1.0
    if n3 % 2 == 0:
        wk[-1] = 1.0
    ri, rs = _iid(((U.real ** 2 + U.imag ** 2).sum(dim=2) * wk[:, None]).sum(dim=0).tolist(), c, s["seed"], 1)
    R = _spec(A[ri]) * t(rs)[None, :, None]
    u, d, vh = _svd(C[:, ri] * t(rs)[None, :, None])
    inv = torch.where(d[:, :r] > c * 2.2e-16 * d[:, :1], 1 / d[:, :r], torch.zeros_like(d[:, :r]))
    left = C @ (vh[:, :r].mH * inv[:, None, :]).to(C.device)
    right = u[:, :, :r].mH.contiguous().to(C.device) @ R
    return {"Z": _unspec(left @ right, n3), "cols": None, "rows": None}


def _exact_complete(case, s):
    X, W, n3 = s["X"].double().cpu(), s["mask"].cpu().bool(), case["n3"]
    L, E, Y, mu = torch.zeros_like(X), torch.zeros_like(X), torch.zeros_like(X), 1e-3
    for _ in range(case["iters"]):
        u, d, vh = _svd(_spec(X - E - Y / mu))
        L = _unspec((u * (d - 1 / mu).clamp_min(0)[:, None, :]) @ vh, n3)
        E = torch.where(W, torch.zeros_like(X), X - L - Y / mu)
        Y = Y + mu * (L + E - X)
        mu = min(1.1 * mu, 1e10)
    return {"L": L, "E": E, "Y": Y, "ranks": None}


def _exact_mlp(s):
    P = s["params"].double().requires_grad_()
    W1, b1, W2, b2, w3, b3 = torch.split(P, [17 * 128, 128, 128 * 128, 128, 128, 1])
    h = torch.relu(s["feat"].double() @ W1.view(17, 128) + b1)
    h = torch.relu(h @ W2.view(128, 128) + b2)
    q = s["target"].double()
    q = q / q.sum(dim=1, keepdim=True)
    logp = torch.log_softmax((h @ w3 + b3).view(q.shape), dim=1)
    loss = (q * (q.log() - logp)).sum(dim=1).mean()
    loss.backward()
    g = P.grad
    m, v = 0.1 * g, 0.001 * g * g
    new = P.detach() - 2e-3 * (m / 0.1) / ((v / 0.001).sqrt() + 1e-8)
    return {"loss": loss.detach().reshape(1), "grad": g, "params": new, "m": m, "v": v}


def exact(case, seed):
    kind = case["kind"]
    if kind == "tcur" and case["cols"] == "lev":
        return None  # the picks follow a randomized estimate
    if kind == "complete" and case["iters"] * (case["n3"] // 2 + 1) * min(case["n1"], case["n2"]) ** 2 > 1.5e7:
        return None  # minutes of dense SVDs on the host
    s = prepare(case, seed)
    if kind == "tprod":
        return _unspec(torch.bmm(_spec(s["A"]), _spec(s["B"])), case["n3"])
    if kind == "rtprod":
        w = s["A"].double().square().sum(dim=(0, 2)).tolist()
        idx, sc = _iid(w, case["c"], s["seed"], 0)
        d = torch.tensor(sc, dtype=torch.float64, device=s["A"].device)
        C, R = _spec(s["A"][:, idx]) * d[None, None, :], _spec(s["B"][idx]) * d[None, :, None]
        return {"Z": _unspec(torch.bmm(C, R), case["n3"]), "idx": None, "scale": d}
    if kind == "transforms":
        S = _spec(s["X"])
        return {"re": S.real.contiguous(), "im": S.imag.contiguous(), "x": s["X"].double()}
    if kind == "tcur":
        return _exact_tcur(case, s)
    if kind == "complete":
        return _exact_complete(case, s)
    return _exact_mlp(s)
