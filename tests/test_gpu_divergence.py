"""Solves from a scaling outside (0, 2 / sigma_1^2) (Theorem 1): every path, stop rule and method ends as diverged, with a finite
iterate, also where the sums of an update turn into NaN before any of them is infinite.  (The guarded rule may stop earlier, at the
first rise of the relative change.)"""
import numpy as np
import pytest

from conftest import to_dev, to_np

pytestmark = pytest.mark.gpu

FACTORS = [2.5, 4.0, 20.0, 200.0, 3e4, 1e9]


def _inputs(m, n, deficient):
    A = np.random.default_rng(m + n).standard_normal((4, m, n))
    if deficient:
        A[:, :, n - n // 3:] = A[:, :, :n // 3]
    C = np.block([[A[0] + 1j * A[1], A[2] + 1j * A[3]], [-A[2] + 1j * A[3], A[0] - 1j * A[1]]])
    return A, 1.0 / np.linalg.norm(C, 2) ** 2


def _ended(q, stop, info):
    return (info["status"] == q.EDIVERGED and info["reason"] == "diverged") or (stop == "guarded" and info["reason"] == "rise")


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("stop", ["dx_abs", "dx_rel", "e1_rel", "guarded"])
@pytest.mark.parametrize("method,order", [("ns", None), ("qsai", None), ("qhpi19", None), ("qrapid", None), ("hpi", 7)])
@pytest.mark.parametrize("m,n", [(64, 48), (100, 130), (200, 170)])
def test_solve(qctx, dtype, stop, method, order, m, n):
    import paper_2605_01464_amd as q

    for deficient in (False, True):
        A, a = _inputs(m, n, deficient)
        for f in FACTORS:
            X, info = q.solve(qctx, to_dev(A, dtype), method, order, scaling="given", alpha=f * a, tol=1e-10, max_iter=200, stop=stop,
                              precision=dtype, check=False)
            assert _ended(q, stop, info), (f, deficient, info)
            assert np.isfinite(to_np(X)).all(), (f, deficient)


@pytest.mark.parametrize("cfg", [0, 1, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("stop", ["dx_rel", "guarded"])
def test_batch(qctx, cfg, stop):
    import paper_2605_01464_amd as q

    cases = [(m, n, d, f) for m, n in ((20, 17), (70, 33), (40, 130)) for d in (False, True) for f in FACTORS]
    ins = [_inputs(m, n, d) for m, n, d, _ in cases]
    for method in ("ns", "qsai", "qhpi19"):
        qctx.set("batched_cfg", cfg)
        try:
            Xs, infos = q.solve_batched(qctx, [to_dev(A, "f32") for A, _ in ins], method, scaling="given",
                                        alphas=[c[3] * a for c, (_, a) in zip(cases, ins)], tol=1e-6, max_iter=200, stop=stop,
                                        check=False)
        finally:
            qctx.set("batched_cfg", -1)
        for c, X, info in zip(cases, Xs, infos):
            assert _ended(q, stop, info), (method, c, info)
            assert np.isfinite(to_np(X)).all(), (method, c)
