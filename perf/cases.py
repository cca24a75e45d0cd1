"""The calls that a user of this framework makes, as cases whose run time can be measured.

Each case goes through the package's public functions with inputs that are made on the GPU from a seed.  Sizes are those
of the tests and of bench.py (the paper's table workloads, the 64 x 48 latency workload, the 4096 x 4096 headline, the
512-matrix batch, Lorenz filter design, the 238-unknown Krylov system, the 512 x 768 image) or generic odd ones.
"""
from __future__ import annotations

import math

import torch

import paper_2605_01464_amd as qp

_CTX = None


def _ctx():
    """The context that a program keeps for all its calls."""
    global _CTX
    if _CTX is None:
        _CTX = qp.Context(0)
    return _CTX


# ----------------------------------------------------------------------------------------------------- cases
def listed():
    return [
        # the smallest solve: one matrix, where latency and launches are all there is
        dict(name="solve_f64_64x48", kind="solve", m=64, n=48, method="qhpi19", dtype="f64", precision="f64",
             scaling="power", stop="e1_rel", tol=1e-12, cond=0.0),
        # the paper's table workloads (Gaussian matrices, its absolute stop rule), small and medium
        dict(name="solve_f64_300x300_qrapid", kind="solve", m=300, n=300, method="qrapid", dtype="f64", precision="f64",
             scaling="frob", stop="dx_abs", tol=1e-10, cond=0.0),
        dict(name="solve_f64_1000x500_qsai", kind="solve", m=1000, n=500, method="qsai", dtype="f64", precision="f64",
             scaling="frob", stop="dx_abs", tol=1e-10, cond=0.0),
        # the headline: a large FP64 solve at condition 1e3
        dict(name="solve_f64_4096", kind="solve", m=4096, n=4096, method="qhpi19", dtype="f64", precision="f64",
             scaling="power", stop="guarded", tol=1e-6, cond=1e3),
        # a tall FP32 solve (least-squares shape)
        dict(name="solve_f32_2048x1536", kind="solve", m=2048, n=1536, method="qhpi19", dtype="f32", precision="f32",
             scaling="power", stop="guarded", tol=1e-6, cond=0.0),
        # the same headline matrix through the BF16 -> FP32 -> FP64 ladder
        dict(name="ladder_4096", kind="solve", m=4096, n=4096, method="qhpi19", dtype="f32", precision="mixed",
             scaling="power", stop="guarded", tol=1e-6, cond=1e3),
        # many small uneven matrices in one call
        dict(name="batched_512", kind="batched", count=512, lo=32, hi=256, method="qhpi19"),
        # Lorenz filter design with 401 taps (an odd size, a Toeplitz matrix, products with a single column)
        dict(name="filter_f64_401", kind="filter", taps=401, method="qsai"),
        # global GMRES on the 238-unknown system with three right-hand sides
        dict(name="krylov_gmres_238x3", kind="krylov", nx=14, ny=17, m=3, method="gmres", precond=False),
        # CUR reconstruction of a colour image from 60 rows and columns
        dict(name="cur_f64_512x768", kind="cur", m=512, n=768, rank=60, method="qhpi19", dtype="f64"),
        # one quaternion product of odd, unaligned sizes
        dict(name="qgemm_f32_1345x777x1001", kind="qgemm", m=1345, n=777, k=1001, dtype="f32", prec="f32"),
        # the scaling network's loss and gradient on a minibatch (forward and backward)
        dict(name="mlp_gradient_256", kind="mlp", batch=256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve64", "solve64", "solve64", "solve32", "solve32", "ladder", "batched", "filter", "krylov", "cur",
                       "qgemm", "mlp"])
    if kind == "solve64":
        m = _log_int(rng, 24, 2400)
        n = max(16, min(2400, int(m * math.exp(rng.uniform(-1.0, 1.0)))))
        return dict(kind="solve", m=m, n=n, method=rng.choice(["qhpi19", "qsai", "qrapid"]), dtype="f64", precision="f64",
                    scaling=rng.choice(["power", "frob"]), stop=rng.choice(["guarded", "dx_rel"]), tol=1e-7, cond=0.0)
    if kind == "solve32":
        m = _log_int(rng, 24, 3000)
        n = max(16, int(m * rng.uniform(0.35, 0.8)))
        if rng.random() < 0.5:
            m, n = n, m
        return dict(kind="solve", m=m, n=n, method=rng.choice(["qhpi19", "qsai", "qrapid", "ns"]), dtype="f32", precision="f32",
                    scaling="power", stop="guarded", tol=1e-6, cond=0.0)
    if kind == "ladder":
        n = _log_int(rng, 700, 4000)
        return dict(kind="solve", m=n, n=n, method=rng.choice(["qhpi19", "qrapid"]), dtype="f32",
                    precision=rng.choice(["mixed", "f32_f64finish"]) if n < 2600 else "mixed", scaling="power",
                    stop="guarded", tol=1e-6, cond=300.0)
    if kind == "batched":
        hi = _log_int(rng, 48, 256)
        return dict(kind="batched", count=_log_int(rng, 8, 512), lo=max(8, hi // 8), hi=hi, method=rng.choice(["qhpi19", "qsai"]))
    if kind == "filter":
        return dict(kind="filter", taps=_log_int(rng, 201, 1001), method=rng.choice(["qsai", "qhpi19"]))
    if kind == "krylov":
        return dict(kind="krylov", nx=rng.randint(6, 14), ny=rng.randint(7, 17), m=rng.choice([1, 3, 6, 9]),
                    method=rng.choice(["gmres", "fom"]), precond=rng.random() < 0.5)
    if kind == "cur":
        return dict(kind="cur", m=_log_int(rng, 200, 1000), n=_log_int(rng, 200, 1000), rank=rng.randint(20, 110),
                    method=rng.choice(["qhpi19", "qsai"]), dtype="f64")
    if kind == "qgemm":
        prec = rng.choice(["f64", "f32", "bf16", "bf16x3"])
        hi = 2000 if prec in ("f64", "f32") else 3500
        return dict(kind="qgemm", m=_log_int(rng, 24, hi), n=_log_int(rng, 24, hi), k=_log_int(rng, 24, hi),
                    dtype="f64" if prec == "f64" else "f32", prec=prec)
    return dict(kind="mlp", batch=_log_int(rng, 16, 1024))


# ----------------------------------------------------------------------------------------------------- inputs
def _gen(seed, device="cuda"):
    g = torch.Generator(device=device)
    g.manual_seed(seed)
    return g


def _randn(g, *shape):
    return torch.randn(*shape, dtype=torch.float64, device=g.device, generator=g)


def _qmul(a, b):
    """Elementwise Hamilton product of component tensors of shape (4, ...)."""
    return torch.stack([a[0] * b[0] - a[1] * b[1] - a[2] * b[2] - a[3] * b[3],
                        a[0] * b[1] + a[1] * b[0] + a[2] * b[3] - a[3] * b[2],
                        a[0] * b[2] - a[1] * b[3] + a[2] * b[0] + a[3] * b[1],
                        a[0] * b[3] + a[1] * b[2] - a[2] * b[1] + a[3] * b[0]])


def _with_cond(g, n, cond):
    """n x n, unit-variance components, singular values geometric from 1 to 1 / cond: orthonormal DCTs and diagonals of
    random unit quaternions on both sides of the diagonal."""
    i = torch.arange(n, dtype=torch.float64, device=g.device)
    dct = torch.cos(math.pi / n * (i[None, :] + 0.5) * i[:, None]) * math.sqrt(2.0 / n)
    dct[0] *= math.sqrt(0.5)

    def unit():
        q = _randn(g, 4, n)
        return q / q.square().sum(0).sqrt()

    s = cond ** (-i / (n - 1))
    s *= 2.0 * n / s.square().sum().sqrt()
    A = torch.zeros(4, n, n, dtype=torch.float64, device=g.device)
    A[0] = torch.diag(s)
    for _ in range(2):
        A = torch.stack([dct @ p for p in _qmul(unit()[:, :, None], A)])
        A = torch.stack([p @ dct for p in _qmul(A, unit()[:, None, :])])
    return A


def _solve_input(case, seed):
    g = _gen(seed)
    A = _with_cond(g, case["n"], case["cond"]) if case["cond"] else _randn(g, 4, case["m"], case["n"])
    return A if case["dtype"] == "f64" else A.float()


def _batch_input(case, seed):
    """Sizes uniform in [lo, hi] (the same for every seed), the two sides at least 5/4 apart, so that FP32 tells the
    results from their rounding; Gaussian planes, all matrices in one allocation and all results in another."""
    gs = _gen(4242, "cpu")
    size = torch.randint(case["lo"], case["hi"] + 1, (case["count"], 2), generator=gs).tolist()
    shapes = []
    for m, n in size:
        if max(m, n) < 1.25 * min(m, n):
            m, n = (m, max(1, int(0.8 * m))) if m >= n else (max(1, int(0.8 * n)), n)
        shapes.append((m, n))
    flat = torch.randn(sum(4 * m * n for m, n in shapes), device="cuda", generator=_gen(seed))
    out = torch.zeros_like(flat)
    As, Xs, at = [], [], 0
    for m, n in shapes:
        As.append(flat[at:at + 4 * m * n].view(4, m, n))
        Xs.append(out[at:at + 4 * m * n].view(4, n, m))
        at += 4 * m * n
    return As, Xs, out


def _filter_input(case, seed):
    """The Lorenz system sampled on [0, 40] from a slightly moved start, delayed by one time unit and seen through unit
    noise: the Toeplitz matrix of the observations and the target signal."""
    taps = case["taps"]
    n = 2 * (taps - 1)
    dt = 40.0 / n
    h = dt / 10
    g = _gen(seed, "cpu")
    u, v, w = (1.0 + 1e-3 * x for x in torch.randn(3, generator=g, dtype=torch.float64).tolist())

    def f(u, v, w):
        return 10.0 * (v - u), u * (28.0 - w) - v, u * v - 8.0 / 3.0 * w

    ref = [(u, v, w)]
    for _ in range(n):
        for _ in range(10):
            a = f(u, v, w)
            b = f(u + 0.5 * h * a[0], v + 0.5 * h * a[1], w + 0.5 * h * a[2])
            c = f(u + 0.5 * h * b[0], v + 0.5 * h * b[1], w + 0.5 * h * b[2])
            d = f(u + h * c[0], v + h * c[1], w + h * c[2])
            u, v, w = (x + h / 6.0 * (p + 2.0 * q + 2.0 * r + s) for x, p, q, r, s in zip((u, v, w), a, b, c, d))
        ref.append((u, v, w))
    ref = torch.tensor(ref, dtype=torch.float64).T.contiguous()
    k = torch.arange(n + 1)
    x = torch.zeros(4, n + 1, dtype=torch.float64)
    x[1:] = ref[:, (k - int(round(1.0 / dt))).clamp(min=0)] + torch.randn(3, n + 1, generator=g, dtype=torch.float64)
    p = taps - 1
    i = torch.arange(taps)
    s = torch.zeros(4, taps, 1, dtype=torch.float64)
    s[1:, :, 0] = ref[:, p:2 * p + 1]
    return x[:, p + i[:, None] - i[None, :]].contiguous().cuda(), s.cuda()


def _krylov_input(case, seed):
    """A five-point finite-volume operator with log-normal transmissibilities, a skew part on its edges and a small
    diagonal, times 1 - i + 2 j + 1.5 k; right-hand sides uniform in [0, 1)."""
    nx, ny = case["nx"], case["ny"]
    n = nx * ny
    g = _gen(seed, "cpu")
    node = torch.arange(n).view(nx, ny)
    a = torch.cat([node[:-1].reshape(-1), node[:, :-1].reshape(-1)])
    b = torch.cat([node[1:].reshape(-1), node[:, 1:].reshape(-1)])
    t = torch.randn(len(a), generator=g, dtype=torch.float64).mul(2.0).exp()
    u = 0.5 * t * torch.randn(len(a), generator=g, dtype=torch.float64)
    S = torch.zeros(n, n, dtype=torch.float64)
    S.index_put_((a, a), t, accumulate=True)
    S.index_put_((b, b), t, accumulate=True)
    S[a, b] = u - t
    S[b, a] = -u - t
    S += 1e-3 * t.mean() * torch.eye(n, dtype=torch.float64)
    A = torch.stack([S, -S, 2.0 * S, 1.5 * S]).cuda()
    return A, torch.rand(4, n, case["m"], generator=g, dtype=torch.float64).cuda()


def _image_input(case, seed):
    """A smooth colour image (40 separable patterns) with fine texture, as a pure quaternion matrix, and the sampled
    rows and columns."""
    m, n = case["m"], case["n"]
    g = _gen(seed, "cpu")
    y = torch.linspace(0, 1, m, dtype=torch.float64)
    x = torch.linspace(0, 1, n, dtype=torch.float64)

    def smooth(t, k):
        f = torch.zeros_like(t)
        for _ in range(3):
            c, w, ph = torch.randn(1, generator=g).item(), torch.rand(1, generator=g).item(), torch.rand(1, generator=g).item()
            f = f + c * torch.sin(2 * math.pi * ((0.2 + w * (0.8 + 0.25 * k)) * t + ph))
        return f

    img = torch.zeros(4, m, n, dtype=torch.float64)
    for k in range(40):
        img[1:] += (torch.randn(3, 1, 1, generator=g, dtype=torch.float64) / (1.0 + k)) * (smooth(y, k)[:, None] * smooth(x, k)[None, :])
    img[1:] *= 0.35 / img[1:].abs().amax(dim=(1, 2), keepdim=True)
    img[1:] += 0.5 + 0.02 * torch.randn(3, m, n, generator=g, dtype=torch.float64)
    rows = torch.randperm(m, generator=g)[:case["rank"]].sort().values.int()
    cols = torch.randperm(n, generator=g)[:case["rank"]].sort().values.int()
    return img.cuda(), rows.cuda(), cols.cuda()


def _qgemm_input(case, seed):
    g = _gen(seed)
    dt = torch.float64 if case["dtype"] == "f64" else torch.float32
    return _randn(g, 4, case["m"], case["k"]).to(dt), _randn(g, 4, case["k"], case["n"]).to(dt)


def _mlp_input(case, seed):
    """Feature rows as matrices of 64 to 512 rows and columns give them, targets, and a network's parameters with the
    mean and spread of its ten inputs behind them."""
    g = _gen(seed, "cpu")

    def rnd(*shape):
        return torch.rand(*shape, generator=g, dtype=torch.float64)

    b = case["batch"]
    m, n = (64 + (448 * rnd(b)).floor() for _ in range(2))
    s1 = (rnd(b) * 4).exp()
    fro = (s1 * torch.minimum(m, n) * (0.02 + 0.5 * rnd(b))).sqrt()
    raw = torch.stack([s1, s1 * (0.9 + 0.1 * rnd(b)), fro, (s1 * m).sqrt() * (0.3 + 0.7 * rnd(b)),
                       (s1 * n).sqrt() * (0.3 + 0.7 * rnd(b)), m, n], dim=1)
    target = 0.2 + 0.4 * rnd(b)
    w = [torch.randn(i, o, generator=g, dtype=torch.float64) / math.sqrt(i) for i, o in ((10, 64), (64, 64), (64, 1))]
    bias = [0.1 * torch.randn(o, generator=g, dtype=torch.float64) for o in (64, 64, 1)]
    z = _features64(raw)
    flat = torch.cat([t.reshape(-1) for pair in zip(w, bias) for t in pair] + [z.mean(0), z.std(0)]).float()
    return raw, target, flat


def prepare(case, seed):
    kind, ctx = case["kind"], _ctx()
    st = {"case": case, "ctx": ctx}
    if kind == "solve":
        st["A"] = _solve_input(case, seed)
        st["out_dtype"] = torch.float32 if case["precision"] == "f32" else torch.float64
    elif kind == "batched":
        As, Xs, st["out"] = _batch_input(case, seed)
        st["args"] = qp.BatchArgs(As, Xs)
    elif kind == "filter":
        st["X"], st["s"] = _filter_input(case, seed)
    elif kind == "krylov":
        st["A"], st["B"] = _krylov_input(case, seed)
        # the preconditioner that a program keeps for its operator: four QSAI updates
        st["M"] = qp.solve(ctx, st["A"], "qsai", tol=0.0, max_iter=4, stop="dx_rel")[0] if case["precond"] else None
    elif kind == "cur":
        st["A"], st["rows"], st["cols"] = _image_input(case, seed)
    elif kind == "qgemm":
        st["A"], st["B"] = _qgemm_input(case, seed)
    else:
        raw, target, flat = _mlp_input(case, seed)
        st["ctx"] = qp.Context(0)  # the network belongs to its context
        if qp.qpinv_mlp_set_params(st["ctx"].handle, flat.tolist()) < 0:
            raise RuntimeError("mlp_set_params")
        st["raw"], st["target"] = raw.cuda(), target.cuda()
        st["grad"] = torch.zeros(qp.qpinv_mlp_num_params(), device="cuda")
    return st


def run(st):
    case, ctx = st["case"], st["ctx"]
    kind = case["kind"]
    if kind == "solve":
        return qp.solve(ctx, st["A"], case["method"], scaling=case["scaling"], tol=case["tol"], stop=case["stop"],
                        precision=case["precision"], out_dtype=st["out_dtype"])[0]
    if kind == "batched":
        qp.solve_batched(ctx, st["args"], case["method"], tol=1e-6, stop="guarded")
        return st["out"]
    if kind == "filter":
        h, s_hat, _ = qp.filter_design(ctx, st["X"], st["s"], case["method"])
        return [h, s_hat]
    if kind == "krylov":
        return qp.gl_krylov(ctx, st["A"], st["B"], case["method"], M=st["M"], tol=1e-6, max_iter=3000)[0]
    if kind == "cur":
        X, U, _ = qp.cur_reconstruct(ctx, st["A"], st["rows"], st["cols"], case["method"])
        return [X, U]
    if kind == "qgemm":
        return qp.qgemm(ctx, st["A"], st["B"], gemm_prec=case["prec"])
    status, loss = qp.qpinv_mlp_gradient(ctx.handle, st["raw"], st["target"], st["grad"])
    if status:
        raise RuntimeError(qp.qpinv_strerror(status))
    return [st["grad"], loss]


# ----------------------------------------------------------------------------------------------------- work
_PRODUCTS = {"ns": (1, 0, 1), "qsai": (1, 4, 1), "qhpi19": (1, 5, 1), "qrapid": (6, 2, 8)}  # m n s, s^3, m n s products
_ORDER = {"ns": 2, "qsai": 10, "qhpi19": 19, "qrapid": 52}


def _product(m, n, k):
    """Real operations of one quaternion product: eight real products (the bilinear rank of the Hamilton product)."""
    return 16.0 * m * n * k


def _solve_flops(m, n, method, cond=0.0):
    """Updates that a spectrum between 1 and 1 / cond needs from alpha = 1 / sigma_1^2, times the products of one."""
    s, o = min(m, n), max(m, n)
    if not cond:
        r = math.sqrt(s / o)
        cond = min((1 + r) / max(1 - r, 1e-9), 4.0 * s)
    updates = math.ceil(math.log(37.0 * cond * cond) / math.log(_ORDER[method]))
    a, b, c = _PRODUCTS[method]
    return updates * ((a + c) * _product(s, s, o) + b * _product(s, s, s))


def work(case):
    kind = case["kind"]
    if kind == "solve":
        m, n = case["m"], case["n"]
        size = 8 if case["dtype"] == "f64" else 4
        out = 4 if case["precision"] == "f32" else 8
        return {"bytes": 4.0 * m * n * (size + out), "flops": _solve_flops(m, n, case["method"], case["cond"])}
    if kind == "batched":
        mean = 0.5 * (case["lo"] + case["hi"])
        return {"bytes": 32.0 * case["count"] * mean * mean,
                "flops": case["count"] * _solve_flops(int(1.15 * mean), int(0.75 * mean), case["method"])}
    if kind == "filter":
        t = case["taps"]
        return {"bytes": 8.0 * 4 * (t * t + 3 * t), "flops": _solve_flops(t, t, case["method"], 1e3) + 2 * _product(t, 1, t)}
    if kind == "krylov":
        n, m = case["nx"] * case["ny"], case["m"]
        steps = 380 if case["precond"] else 5 * n
        basis = 4.0 * n * m * steps * steps  # two passes of projection and update over a basis that grows
        return {"bytes": 8.0 * 4 * (n * n + 2 * n * m), "flops": steps * _product(n, m, n) + 4.0 * basis}
    if kind == "cur":
        m, n, r = case["m"], case["n"], case["rank"]
        flops = sum(_solve_flops(r, o, case["method"], 1e3) for o in (m, n))
        flops += _product(m, r, n) + _product(r, r, m) + _product(m, r, r) + _product(m, n, r)
        return {"bytes": 8.0 * 4 * (2 * m * n + r * r), "flops": flops}
    if kind == "qgemm":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": 4.0 * (8 if case["dtype"] == "f64" else 4) * (m * k + k * n + m * n), "flops": _product(m, n, k)}
    b = case["batch"]
    return {"bytes": 8.0 * 8 * b + 4.0 * 2 * 4945, "flops": 6.0 * b * (10 * 64 + 64 * 64 + 64)}


# ----------------------------------------------------------------------------------------------------- 64-bit results
def _adjoint(A):
    """The 2m x 2n complex matrix of a quaternion matrix (4, m, n)."""
    a, b = torch.complex(A[0], A[1]), torch.complex(A[2], A[3])
    return torch.cat([torch.cat([a, b], 1), torch.cat([-b.conj(), a.conj()], 1)], 0)


def _planes(C):
    m, n = C.shape[0] // 2, C.shape[1] // 2
    a = 0.5 * (C[:m, :n] + C[m:, n:].conj())
    b = 0.5 * (C[:m, n:] - C[m:, :n].conj())
    return torch.stack([a.real, a.imag, b.real, b.imag])


def _pinv(A):
    """Pseudoinverse of a full-rank quaternion matrix in 64 bits: inverse of the complex matrix, or its QR factors."""
    if A.shape[1] < A.shape[2]:
        conj = torch.tensor([1.0, -1, -1, -1], dtype=A.dtype).view(4, 1, 1)
        return conj * _pinv((conj * A).transpose(1, 2)).transpose(1, 2)
    C = _adjoint(A)
    if C.shape[0] == C.shape[1]:
        return _planes(torch.linalg.inv(C))
    Q, R = torch.linalg.qr(C)
    return _planes(torch.linalg.solve_triangular(R, Q.conj().T, upper=True))


def _mul(A, B):
    """Hamilton product of matrices of planes."""
    p = [[A[i] @ B[j] for j in range(4)] for i in range(4)]
    return torch.stack([p[0][0] - p[1][1] - p[2][2] - p[3][3], p[0][1] + p[1][0] + p[2][3] - p[3][2],
                        p[0][2] - p[1][3] + p[2][0] + p[3][1], p[0][3] + p[1][2] - p[2][1] + p[3][0]])


def _features64(raw):
    s1, s1p, fro, n1, ni, m, n = raw.T
    mn, mx = torch.minimum(m, n), torch.maximum(m, n)
    return torch.stack([m.log(), n.log(), (mn / mx).log(), (fro * fro / s1).log(), (n1 * ni / s1).log(), (n1 / ni).log(),
                        (fro * fro / (s1 * mn)).log(), s1p / s1, (n1 / (m * s1).sqrt()).log(), (ni / (n * s1).sqrt()).log()], dim=1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve":
        return _pinv(_solve_input(case, seed).cpu().double())
    if kind == "batched":
        As, _, _ = _batch_input(case, seed)
        out = []
        for A in As:  # conditions below 20: the normal equations lose nothing that FP32 results could show
            A = A.cpu().double()
            C = _adjoint(A)
            H = C.conj().T
            X = torch.linalg.solve(H @ C, H) if C.shape[0] >= C.shape[1] else torch.linalg.solve(C @ H, C).conj().T
            out.append(_planes(X).reshape(-1))
        return torch.cat(out)
    if kind == "filter":
        X, s = (t.cpu() for t in _filter_input(case, seed))
        h = _mul(_pinv(X), s)
        return [h, _mul(X, h)]
    if kind == "krylov":
        A, B = (t.cpu() for t in _krylov_input(case, seed))
        return _planes(torch.linalg.solve(_adjoint(A), _adjoint(B)))
    if kind == "cur":
        A, rows, cols = (t.cpu() for t in _image_input(case, seed))
        C, R = A[:, :, cols.long()], A[:, rows.long(), :]
        U = _mul(_pinv(C), _mul(A, _pinv(R)))
        return [_mul(_mul(C, U), R), U]
    if kind == "qgemm":
        A, B = (t.cpu().double() for t in _qgemm_input(case, seed))
        return _mul(A, B)
    raw, target, flat = _mlp_input(case, seed)
    p = flat.double().requires_grad_(True)
    at, parts = 0, []
    for shape in ((10, 64), (64,), (64, 64), (64,), (64, 1), (1,), (10,), (10,)):
        size = math.prod(shape)
        parts.append(p[at:at + size].view(shape))
        at += size
    w1, b1, w2, b2, w3, b3, mean, std = parts
    z = (_features64(raw) - mean.detach()) / std.detach()
    y = (torch.tanh(torch.tanh(z @ w1 + b1) @ w2 + b2) @ w3 + b3)[:, 0]
    loss = (y - target).square().mean()
    loss.backward()
    return [p.grad[:-20].clone(), loss.item()]
