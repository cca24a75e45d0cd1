"""The operand loads of products off whole tiles give the same bits: 16-byte ones of aligned rows and element ones of odd strides,
on both sides of the line between them (one 32 x 32 tile per compute unit) and with NaN outside the matrices."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _view(x, ld, dt):
    import torch

    buf = torch.full((4, x.shape[1], ld), float("nan"), dtype=dt, device="cuda")
    buf[:, :, :x.shape[2]] = torch.from_numpy(x)
    return buf[:, :, :x.shape[2]]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("m,n,k", [(17, 18, 19), (33, 34, 130), (500, 500, 66), (510, 514, 70), (4100, 14, 9)])
def test_same_bits(qctx, prec, m, n, k):
    import torch

    import paper_2605_01464_amd as q

    rng = np.random.default_rng(m + n + k)
    A, B = rng.standard_normal((4, m, k)), rng.standard_normal((4, k, n))
    dt = torch.float64 if prec == "f64" else torch.float32
    even = lambda c: (c + 3) // 4 * 4  # noqa: E731
    C = q.qgemm(qctx, _view(A, even(k), dt), _view(B, even(n), dt))
    D = q.qgemm(qctx, _view(A, even(k) + 1, dt), _view(B, even(n) + 3, dt))
    assert torch.isfinite(C).all() and torch.equal(C, D)
