"""The tolerance network's matrix kernels at the edges of their tiles: batches
around 16, 64 and a full launch, with samples outside the caller's arrays.

Tolerance: gradients as FP32 sums of the batch, 1e-4 of the largest entry, as
derived for the full-size check."""

import numpy as np
import pytest

import synth
from oracle import mlp
from tests.gpu_util import torch_gpu

pytestmark = pytest.mark.gpu


def _net(seed):
    theta = synth.mlp_init(seed).astype(np.float32)
    theta[-65:-1] *= 8.0
    return theta


def _features(rng, n):
    return np.stack([rng.uniform(1, 12, n), rng.uniform(0, 1, n), rng.uniform(-3.1, 3.1, n),
                     rng.uniform(-1, 1, n), rng.uniform(-0.7, 0.7, n), rng.uniform(0, 6.9, n)],
                    axis=1).astype(np.float32)


@pytest.mark.parametrize("batch", [1, 15, 16, 17, 63, 64, 65, 129, 16385])
def test_gradient_tile_edges(batch):
    from paper_2603_18401_amd import learned_eps as L
    torch = torch_gpu()
    rng = np.random.default_rng(batch)
    theta = _net(3)
    X = _features(rng, 4 * batch + 64)
    f = mlp.forward(theta.astype(np.float64), X.astype(np.float64))
    ok = (np.abs(f["a1"]).min(axis=1) > 1e-3) & (np.abs(f["a2"]).min(axis=1) > 1e-3)
    rows = np.nonzero(ok)[0]
    rows = np.resize(rows, batch)  # repeated if too few lie clear of the kinks
    y = (f["yhat"][rows] + rng.choice([-0.5, 0.5], batch)).astype(np.float32)
    slots = np.arange(batch, dtype=np.int32)
    fidx = rows.astype(np.int64)
    # one slot outside the targets and one feature row outside the features
    # contribute nothing, but count in the mean
    live = np.ones(batch, bool)
    if batch > 15:
        slots[7], fidx[11] = batch + 5, len(X)
        live[[7, 11]] = False
    dev = torch.device("cuda:0")
    g = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    tr = L.Trainer(theta, dev, q=0.9)
    grad, loss = tr.grad(g(X), g(y), g(slots), feat_index=g(fidx))
    got = grad.cpu().numpy().astype(np.float64)
    rl, rg = mlp.loss_and_grad(theta.astype(np.float64), X[rows[live]].astype(np.float64),
                               y[live].astype(np.float64), 0.9)
    rl, rg = rl * live.sum() / batch, rg * live.sum() / batch
    assert abs(float(loss.item()) - rl) <= 1e-5 * abs(rl)
    assert np.abs(got - rg).max() <= 1e-4 * np.abs(rg).max()
    again = tr.grad(g(X), g(y), g(slots), feat_index=g(fidx))[0].cpu().numpy()
    assert np.array_equal(got, again.astype(np.float64))
