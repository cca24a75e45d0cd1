"""The eight-product form of the solvers' FP64 and FP32 products: one Newton-Schulz update X_1 = (2I - X_0 A) X_0 from a given
alpha, element by element against the host in FP64, at the edges of its tiles (16 x 16 in registers, 32 x 32 and 64 x 64
through LDS, the K step of 8 or 16 and its remainders) and of its rule."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _mul(A, B):
    p = [[A[i] @ B[j] for j in range(4)] for i in range(4)]
    return np.stack([p[0][0] - p[1][1] - p[2][2] - p[3][3], p[0][1] + p[1][0] + p[2][3] - p[3][2],
                     p[0][2] - p[1][3] + p[2][0] + p[3][1], p[0][3] + p[1][2] - p[2][1] + p[3][0]])


def _one_update(q, ctx, A, alpha, dtype):
    from conftest import to_dev, to_np

    ctx.set("small_path", 0)
    ctx.set("gemm_timing", 1)
    q.qpinv_gemm_stats(ctx.handle)
    try:
        X, info = q.solve(ctx, to_dev(A, dtype), "ns", scaling="given", alpha=alpha, tol=0.0, max_iter=1, stop="guarded",
                          precision=dtype)
        _, rows = q.qpinv_gemm_stats(ctx.handle)
    finally:
        ctx.set("small_path", 1)
        ctx.set("gemm_timing", 0)
    assert info["iters"] == 1
    return to_np(X), {q.qpinv_tile_config_name(r["prec"], r["cfg"]) for r in rows}


# square sizes around each tile's range, long and short K (the residual's side is the smaller dimension); the last two have
# smaller tiles over the rows of the last round
SHAPES = [(1, 1), (2, 1), (15, 17), (16, 16), (33, 31), (129, 7), (9, 260), (65, 640), (701, 690), (1030, 1001), (2060, 40),
          (1100, 1090), (1043, 1300)]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("m,n", SHAPES)
def test_one_update_elementwise(qctx, dtype, m, n):
    import paper_2605_01464_amd as q

    rng = np.random.default_rng(77 * m + n)
    A = rng.standard_normal((4, m, n))
    A[:, : m // 2] *= rng.uniform(0.1, 10.0, size=(4, 1, 1))  # planes of different size
    if dtype == "f32":
        A = A.astype(np.float32).astype(np.float64)
    u = 2.0 ** -53 if dtype == "f64" else 2.0 ** -24
    alpha = 1.0 / np.sum(A * A)
    X1, names = _one_update(q, qctx, A, alpha, dtype)
    k1, k2 = max(m, n), min(m, n)  # K of the two products; below 16 the direct form is kept
    assert {"x8_" in name for name in names} == {k >= 16 for k in (k1, k2)}, names
    conj = np.array([1.0, -1.0, -1.0, -1.0]).reshape(4, 1, 1)
    X0 = alpha * conj * A.transpose(0, 2, 1)
    left = m > n
    s = min(m, n)
    P = _mul(X0, A) if left else _mul(A, X0)
    T = -P
    T[0] += 2.0 * np.eye(s)
    ref = _mul(T, X0) if left else _mul(X0, T)
    # |error| <= 3 gamma_{K + 8} sum_k (sum_p |a_p|) (sum_q |b_q|): an output is half the sum of four products plus a fifth,
    # each with K terms of one rounded sum of two elements a side
    a1, x1, t1 = (np.abs(M).sum(0) for M in (A, X0 * (1 + 2 * u), T))
    eT = 3 * (k1 + 12) * u * (x1 @ a1 if left else a1 @ x1) + 2 * u * np.abs(T).max(0)
    eT4 = 4 * eT
    bound = (eT4 @ x1 if left else x1 @ eT4) + 3 * (k2 + 12) * u * (t1 @ x1 if left else x1 @ t1)
    err = np.abs(X1 - ref).max(0)
    # the host's own FP64 evaluation has the direct form's bound
    host = 4 * 2.0 ** -53 * (k1 + k2 + 8) * ((t1 + (x1 @ a1 if left else a1 @ x1)) @ x1 if left else x1 @ (t1 + (a1 @ x1)))
    assert np.all(err <= bound + host), float((err / (bound + host)).max())
    # and in the norm it is no less accurate than the direct form's typical error
    assert np.linalg.norm(X1 - ref) <= 16 * u * np.sqrt(k1 + k2) * np.linalg.norm(ref)


@pytest.mark.parametrize("dtype,scale", [("f32", 2.0 ** 60), ("f32", 2.0 ** -60), ("f64", 2.0 ** 400)])
def test_extreme_norms_take_the_direct_form(qctx, dtype, scale):
    """A norm near the type's limits keeps the direct form, and the update scales with the matrix exactly."""
    import paper_2605_01464_amd as q

    A = np.random.default_rng(5).standard_normal((4, 70, 50)).astype(np.float32).astype(np.float64)
    alpha = 1.0 / np.sum(A * A)
    qctx.set("gemm_cfg_" + dtype, 1)
    try:
        X, _ = _one_update(q, qctx, A, alpha, dtype)
    finally:
        qctx.set("gemm_cfg_" + dtype, -1)
    ctx = qctx
    from conftest import to_dev, to_np

    ctx.set("small_path", 0)
    ctx.set("gemm_timing", 1)
    q.qpinv_gemm_stats(ctx.handle)
    try:
        Xs, _ = q.solve(ctx, to_dev(A * scale, dtype), "ns", scaling="given", alpha=alpha / scale ** 2, tol=0.0, max_iter=1,
                        stop="guarded", precision=dtype)
        _, rows = q.qpinv_gemm_stats(ctx.handle)
    finally:
        ctx.set("small_path", 1)
        ctx.set("gemm_timing", 0)
    assert all("x8_" not in q.qpinv_tile_config_name(r["prec"], r["cfg"]) for r in rows)
    u = 2.0 ** -53 if dtype == "f64" else 2.0 ** -24
    assert np.linalg.norm(to_np(Xs) * scale - X) <= 64 * u * np.linalg.norm(X)


def test_unaligned_input(qctx):
    """A caller's rows off 16-byte boundaries are copied once; the result is that of the same matrix on such boundaries."""
    import torch

    import paper_2605_01464_amd as q

    A = torch.from_numpy(np.random.default_rng(6).standard_normal((4, 141, 133))).cuda()
    padded = torch.zeros(4, 141, 136, dtype=torch.float64, device="cuda")
    padded[:, :, :133] = A
    X0, i0 = q.solve(qctx, padded[:, :, :133], "qhpi19")
    X1, i1 = q.solve(qctx, A, "qhpi19")
    assert i0["iters"] == i1["iters"] and torch.equal(X0, X1)
