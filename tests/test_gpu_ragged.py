"""Products of odd sizes and strides in every tile configuration: against the host in FP64, and bit for bit against the same
operands on 16-byte boundaries where the sizes are whole tiles."""
import numpy as np
import pytest

from conftest import to_np
from oracle import quat as Q

pytestmark = pytest.mark.gpu
CONFIGS = {"f32": 9, "f64": 7}


def strided(x, ld, prec):
    """x as a view of a buffer with row stride ld whose other elements are NaN."""
    import torch

    dt = torch.float64 if prec == "f64" else torch.float32
    buf = torch.full((4, x.shape[1], ld), float("nan"), dtype=dt, device="cuda")
    buf[:, :, :x.shape[2]] = torch.from_numpy(x)
    return buf[:, :, :x.shape[2]]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (65, 67, 33), (31, 129, 17), (130, 66, 5), (128, 128, 150), (64, 20, 32)])
def test_odd_strides(qctx, prec, m, n, k):
    import paper_2605_01464_amd as q

    rng = np.random.default_rng(100 * m + 10 * n + k)
    dt = np.float64 if prec == "f64" else np.float32
    A, B, C0 = (rng.standard_normal(s).astype(dt) for s in ((4, m, k), (4, k, n), (4, m, n)))
    ref = 1.5 * Q.qmul(A.astype(np.float64), B.astype(np.float64)) - 0.5 * C0.astype(np.float64)
    ref[0] += 2.0 * np.eye(m, n)
    u = 2.0 ** -53 if prec == "f64" else 2.0 ** -24
    S = np.abs(A).sum(0).astype(np.float64) @ np.abs(B).sum(0).astype(np.float64)
    bound = (4 * k + 8) * u * (1.5 * S + 0.5 * np.abs(C0) + 2.0) + 1e-30
    for cfg in range(CONFIGS[prec]):
        for pad in (1, 2, 5):
            C = strided(C0, n + pad, prec)
            q.qgemm(qctx, strided(A, k + pad, prec), strided(B, n + 2 * pad + 1, prec), C, alpha=1.5, beta=-0.5,
                    gamma=2.0, cfg=cfg)
            assert np.all(np.abs(to_np(C) - ref) <= bound), (cfg, pad)


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_odd_strides_same_bits(qctx, prec):
    import torch

    import paper_2605_01464_amd as q

    m, n, k = 128, 256, 144
    rng = np.random.default_rng(7)
    A, B = rng.standard_normal((4, m, k)), rng.standard_normal((4, k, n))
    for cfg in range(CONFIGS[prec]):
        C0 = q.qgemm(qctx, strided(A, k, prec), strided(B, n, prec), cfg=cfg)
        C1 = q.qgemm(qctx, strided(A, k + 3, prec), strided(B, n + 1, prec), cfg=cfg)
        assert torch.equal(C0, C1), cfg
