"""Products of at most 16 columns against the host in FP64 and, bit for bit, against the 32 x 32 tile configuration whose sums they
keep; Krylov runs whose vectors are longer than the fused norm takes."""
import numpy as np
import pytest

import qsynth
from conftest import to_dev, to_np
from oracle import krylov as K
from oracle import quat as Q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,same", [("f64", 1), ("f32", 6)])
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (16, 16, 8), (17, 15, 129), (5, 3, 16), (238, 3, 238), (33, 16, 255), (50, 2, 0)])
def test_narrow_product(qctx, prec, same, m, n, k):
    import torch

    import paper_2605_01464_amd as q

    rng = np.random.default_rng(1000 * m + 10 * n + k)
    A, B, C0 = (rng.standard_normal(s) for s in ((4, m, k), (4, k, n), (4, m, n)))
    Ad, Bd = to_dev(A, prec), to_dev(B, prec)
    C, D = to_dev(C0, prec), to_dev(C0, prec)
    q.qgemm(qctx, Ad, Bd, C, alpha=1.5, beta=-0.5, gamma=2.0)
    q.qgemm(qctx, Ad, Bd, D, alpha=1.5, beta=-0.5, gamma=2.0, cfg=same)
    assert torch.equal(C, D)
    ref = 1.5 * Q.qmul(to_np(Ad), to_np(Bd)) - 0.5 * to_np(to_dev(C0, prec))
    ref[0] += 2.0 * np.eye(m, n)
    u = 2.0 ** -53 if prec == "f64" else 2.0 ** -24
    S = np.abs(to_np(Ad)).sum(0) @ np.abs(to_np(Bd)).sum(0)
    assert np.all(np.abs(to_np(C) - ref) <= (4 * k + 8) * u * (1.5 * S + 0.5 * np.abs(C0) + 2.0) + 1e-30)


def test_krylov_long_vectors(qctx):
    """4 n m = 18480 doubles: the norm has a kernel of its own."""
    import paper_2605_01464_amd as q

    d = qsynth.krylov_instance(110, grid=(6, 7), seed=713)
    ref = K.solve(d["A"], d["B"], "gmres", tol=0.0, max_iter=6)
    X, info = q.gl_krylov(qctx, to_dev(d["A"], "f64"), to_dev(d["B"], "f64"), method="gmres", tol=0.0, max_iter=6, history=True)
    assert info["iters"] == 6
    assert np.allclose(info["history"], ref["history"], rtol=1e-8, atol=0.0)
    assert Q.fro(to_np(X) - ref["X"]) <= 1e-8 * Q.fro(ref["X"])
