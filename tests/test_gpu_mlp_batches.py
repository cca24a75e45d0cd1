"""The network's gradient and loss at minibatch sizes around the kernels' sample groups and batch quarters, with and without
an index, against FP64 backpropagation."""
import numpy as np
import pytest

from oracle import mlp as OM
from test_gpu_learned import random_raw, set_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 2, 3, 4, 5, 7, 255, 1024])
def test_gradient_batches(qctx, batch):
    import torch

    import paper_2605_01464_amd as q

    rng = np.random.default_rng(100 + batch)
    theta, mean, std = set_params(q, qctx, rng)
    raw, tgt = random_raw(rng, batch), rng.standard_normal(batch)
    grad = torch.empty(OM.NPARAM, dtype=torch.float32, device="cuda")
    st, loss = q.qpinv_mlp_gradient(qctx.handle, torch.from_numpy(raw).cuda(), torch.from_numpy(tgt).cuda(), grad)
    assert st == q.OK
    lo, go = OM.loss_and_grad(theta, (OM.transform(raw) - mean) / std, tgt)
    assert loss == pytest.approx(lo, rel=1e-4)
    assert np.linalg.norm(grad.double().cpu().numpy() - go) <= 1e-4 * np.linalg.norm(go)


def test_train_step_takes_the_indexed_rows(qctx):
    import torch

    import paper_2605_01464_amd as q

    rng = np.random.default_rng(9)
    theta, mean, std = set_params(q, qctx, rng)
    raw, tgt = random_raw(rng, 50), rng.standard_normal(50)
    idx = rng.permutation(50)[:21].astype(np.int32)
    st, loss = q.qpinv_mlp_train_step(qctx.handle, torch.from_numpy(raw).cuda(), torch.from_numpy(tgt).cuda(),
                                      torch.from_numpy(idx).cuda(), 21, 1e-3)
    assert st == q.OK
    lo, go = OM.loss_and_grad(theta, (OM.transform(raw[idx]) - mean) / std, tgt[idx])
    assert loss == pytest.approx(lo, rel=1e-4)
    _, vals = q.qpinv_mlp_get_params(qctx.handle)
    # Adam's first step moves every parameter by lr against the sign of its gradient
    moved = np.asarray(vals[:OM.NPARAM]) - theta
    big = np.abs(go) > 1e-3 * np.abs(go).max()
    assert np.all(np.sign(moved[big]) == -np.sign(go[big])) and np.all(np.abs(moved[big]) <= 1.01e-3)
