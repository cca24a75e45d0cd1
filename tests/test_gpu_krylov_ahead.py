"""A Krylov run that ends after its first step queues no further ones."""
import numpy as np
import pytest

from conftest import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(60, 2), (300, 20)])
def test_no_step_beyond_the_first(qctx, n, m):
    import paper_2605_01464_amd as q

    rng = np.random.default_rng(n)
    A = rng.standard_normal((4, n, n)) / n
    A[0] += 2.0 * np.eye(n)
    Ad, Bd = to_dev(A, "f64"), to_dev(rng.standard_normal((4, n, m)), "f64")
    M, _ = q.solve(qctx, Ad, "qsai", tol=1e-12)
    qctx.set("gemm_timing", 1)
    q.qpinv_gemm_stats(qctx.handle)
    try:
        _, info = q.gl_krylov(qctx, Ad, Bd, M=M, tol=1e-6, max_iter=50)
        _, rows = q.qpinv_gemm_stats(qctx.handle)
    finally:
        qctx.set("gemm_timing", 0)
    assert info["status"] == q.OK and info["iters"] == 1
    # A X_0 and M R_0, the step's A V and M A V, and the residual of the stopping test and of the result
    assert sum(r["launches"] for r in rows) == 6
