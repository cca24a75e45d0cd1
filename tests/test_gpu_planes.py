"""Solves of matrices whose planes are of very different size: every plane of one Newton-Schulz update X_1 = (2I - X_0 A) X_0 keeps the
direct form's bound, which has the terms of that plane alone, and planes that a complex subalgebra leaves zero are zero."""
import numpy as np
import pytest

from conftest import to_dev, to_np

pytestmark = pytest.mark.gpu

STRONG = {"s": (0,), "x": (1,), "sx": (0, 1), "sy": (0, 2), "sz": (0, 3), "yz": (2, 3), "xz": (1, 3)}


def _matrix(kind, eps, m, n, dtype):
    rng = np.random.default_rng(1000 * m + n)
    A = rng.standard_normal((4, m, n))
    if kind == "block":  # rows and columns that nothing couples to the rest, weak in planes x and z
        h, w = m // 2, n // 2
        A[:, :h, w:] = 0.0
        A[:, h:, :w] = 0.0
        A[1, :h] *= eps
        A[3, :h] *= eps
    else:
        for p in range(4):
            if p not in STRONG[kind]:
                A[p] *= eps
    return A.astype(np.float32).astype(np.float64) if dtype == "f32" else A


def _terms(A, B):
    """Per plane p, sum over q of |A_q| |B_{p^q}|: the terms of the Hamilton product's plane."""
    A, B = np.abs(A), np.abs(B)
    return np.stack([sum(A[q] @ B[p ^ q] for q in range(4)) for p in range(4)])


def _mul(A, B):
    s = [(1, -1, -1, -1), (1, 1, 1, -1), (1, -1, 1, 1), (1, 1, -1, 1)]
    return np.stack([sum(s[p][q] * (A[q] @ B[p ^ q]) for q in range(4)) for p in range(4)])


def _start(A, alpha):
    return alpha * np.array([1.0, -1.0, -1.0, -1.0]).reshape(4, 1, 1) * A.transpose(0, 2, 1)


def _check(A, X1, X0, dtype):
    u = 2.0 ** -53 if dtype == "f64" else 2.0 ** -24
    _, m, n = A.shape
    k1, k2 = max(m, n), min(m, n)
    left = m > n
    pair = (lambda T, X: (T, X)) if left else (lambda T, X: (X, T))
    T = -_mul(*((X0, A) if left else (A, X0)))
    T[0] += 2.0 * np.eye(k2)
    ref = _mul(*pair(T, X0))
    # a plane's 4 K products and additions and its epilogue, X_0 and T rounded once; the host's own sums in FP64
    eT = (4 * k1 + 12) * (u + 2.0 ** -53) * _terms(*((X0, A) if left else (A, X0))) + 2 * u * np.abs(T)
    bound = 1.01 * (_terms(*pair(eT, X0)) + (4 * k2 + 12) * (u + 2.0 ** -53) * _terms(*pair(T, X0)))
    err = np.abs(X1 - ref)
    for p in range(4):
        assert np.all(err[p] <= bound[p] + 1e-38), (p, float((err[p] / (bound[p] + 1e-38)).max()))


CASES = [("s", 1e-3), ("s", 1e-6), ("x", 1e-6), ("sx", 1e-6), ("sy", 1e-4), ("sy", 0.0), ("sz", 0.0), ("xz", 1e-5), ("yz", 1e-5),
         ("block", 1e-5), ("block", 0.0)]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("m,n", [(33, 40), (300, 160), (1040, 1030)])
@pytest.mark.parametrize("kind,eps", CASES)
def test_weak_planes_keep_their_digits(qctx, dtype, m, n, kind, eps):
    import paper_2605_01464_amd as q

    A = _matrix(kind, eps, m, n, dtype)
    alpha = 1.0 / np.sum(A * A)
    X, info = q.solve(qctx, to_dev(A, dtype), "ns", scaling="given", alpha=alpha, tol=0.0, max_iter=1, stop="guarded",
                      precision=dtype)
    assert info["iters"] == 1
    _check(A, to_np(X), _start(A, alpha), dtype)


@pytest.mark.parametrize("cfg", [0, 3, 5, 6, 7])
def test_weak_planes_in_a_batch(qctx, cfg):
    import paper_2605_01464_amd as q

    As = [_matrix(kind, eps, m, n, "f32") for kind, eps in CASES for m, n in ((17, 16), (70, 33), (40, 130))]
    alphas = [1.0 / np.sum(A * A) for A in As]
    qctx.set("batched_cfg", cfg)
    try:
        Xs, infos = q.solve_batched(qctx, [to_dev(A, "f32") for A in As], "ns", 2, scaling="given", alphas=alphas, tol=0.0,
                                    max_iter=1, stop="dx_rel", check=False)
    finally:
        qctx.set("batched_cfg", -1)
    for A, a, X, info in zip(As, alphas, Xs, infos):
        assert info["iters"] == 1
        _check(A, to_np(X), _start(A, a), "f32")


def _forms(q, ctx, A, dtype):
    ctx.set("small_path", 0)
    ctx.set("gemm_timing", 1)
    q.qpinv_gemm_stats(ctx.handle)
    try:
        q.solve(ctx, to_dev(A, dtype), "ns", tol=0.0, max_iter=1, stop="guarded", precision=dtype)
        _, rows = q.qpinv_gemm_stats(ctx.handle)
    finally:
        ctx.set("small_path", 1)
        ctx.set("gemm_timing", 0)
    return {"x8_" in q.qpinv_tile_config_name(r["prec"], r["cfg"]) for r in rows}


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_rule(qctx, dtype):
    """Both sides of the lines: 1/5 over the matrix and 1/16 in a row, and the matrices that stay exact in either form."""
    import paper_2605_01464_amd as q

    A = np.sign(np.random.default_rng(3).standard_normal((4, 70, 300)))  # elements of +-1: exact plane norms
    for pair in ((1, 2), (1, 3), (2, 3)):
        for f, eight in ((0.21, True), (0.19, False)):
            B = A.copy()
            B[list(pair)] *= f
            assert _forms(q, qctx, B, dtype) == {eight}, (pair, f)
    for f, eight in ((0.07, True), (0.06, False)):
        B = A.copy()
        B[2:, 41] *= f
        assert _forms(q, qctx, B, dtype) == {eight}, f
    for keep, eight in (((0,), True), ((2,), True), ((0, 1), True), ((2, 3), True), ((0, 2), False), ((1, 2), False)):
        B = np.zeros_like(A)
        B[list(keep)] = A[list(keep)]
        assert _forms(q, qctx, B, dtype) == {eight}, keep
    B = np.zeros_like(A)  # a plane whose squares underflow is not a zero plane
    B[0], B[2] = A[0], A[2] * (1e-170 if dtype == "f64" else 1e-30)
    assert _forms(q, qctx, B, dtype) == {False}


@pytest.mark.parametrize("dtype,m,n", [("f64", 21, 671), ("f64", 116, 473), ("f64", 173, 370), ("f32", 5, 760), ("f32", 64, 661)])
def test_largest_allocation_free_shapes(qctx, dtype, m, n):
    """Shapes whose workspace bound just fits the allocation-free scratch: looking at the planes takes none of it."""
    import torch

    import paper_2605_01464_amd as q

    qctx.set("autotune", 0)
    A = to_dev(np.random.default_rng(m).standard_normal((4, m, n)), dtype)
    X = torch.empty((4, n, m), dtype=A.dtype, device="cuda")
    info = q.solve_noalloc(qctx, A, X, "qhpi19", precision=dtype, check=False)
    assert info["status"] == q.OK
    assert torch.equal(X, q.solve(qctx, A, "qhpi19", precision=dtype)[0])


@pytest.mark.parametrize("m,n", [(209716, 16), (16, 209716)])
def test_rows_beyond_the_scratch(qctx, m, n):
    """More rows than the products' scratch holds sums for."""
    import torch

    import paper_2605_01464_amd as q

    A = torch.randn(4, m, n, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(4))
    X, info = q.solve(qctx, A, "qhpi19", tol=1e-9)
    assert info["status"] == q.OK
    P = [[X[i] @ A[j] if m > n else A[i] @ X[j] for j in range(4)] for i in range(4)]
    I = torch.stack([P[0][0] - P[1][1] - P[2][2] - P[3][3], P[0][1] + P[1][0] + P[2][3] - P[3][2],
                     P[0][2] - P[1][3] + P[2][0] + P[3][1], P[0][3] + P[1][2] - P[2][1] + P[3][0]])
    I[0] -= torch.eye(16, dtype=torch.float64, device="cuda")
    assert I.abs().max().item() <= 1e-11


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("keep", [(0,), (2,), (0, 1), (2, 3)])
def test_given_start_with_other_planes(qctx, dtype, keep):
    """A matrix that the form itself keeps exact, from a start whose other planes are weak: they keep their digits too."""
    import paper_2605_01464_amd as q

    dt = np.float32 if dtype == "f32" else np.float64
    A = _matrix("s", 1.0, 90, 70, dtype)
    A[[p for p in range(4) if p not in keep]] = 0.0
    X0 = _start(A, 1.0 / np.sum(A * A)) + 1e-7 * np.random.default_rng(8).standard_normal((4, 70, 90)) * np.array(
        [float(p not in keep) for p in range(4)]).reshape(4, 1, 1)
    X0 = X0.astype(dt).astype(np.float64)
    X, info = q.solve(qctx, to_dev(A, dtype), "ns", scaling="x0", tol=0.0, max_iter=1, stop="guarded", precision=dtype,
                      X=to_dev(X0, dtype))
    assert info["iters"] == 1
    _check(A, to_np(X), X0, dtype)
