"""Krylov runs on both sides of the lengths at which the basis update changes its kernel (4 n m = 16384 and 2^18 doubles), with a
length off the workgroups' 256 elements, against the oracle at a fixed number of steps."""
import numpy as np
import pytest

import qsynth
from conftest import to_dev, to_np
from oracle import krylov as K
from oracle import quat as Q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [97, 98, 1560, 1561])
def test_lengths(qctx, m):
    import paper_2605_01464_amd as q

    d = qsynth.krylov_instance(m, grid=(6, 7), seed=714)  # n = 42
    ref = K.solve(d["A"], d["B"], "gmres", tol=0.0, max_iter=5)
    X, info = q.gl_krylov(qctx, to_dev(d["A"], "f64"), to_dev(d["B"], "f64"), method="gmres", tol=0.0, max_iter=5, history=True)
    assert info["iters"] == 5
    assert np.allclose(info["history"], ref["history"], rtol=1e-8, atol=0.0)
    assert Q.fro(to_np(X) - ref["X"]) <= 1e-8 * Q.fro(ref["X"])
