"""The tolerance network's matrix kernels at the edges of their tiles: batches
and keypoint counts around 16, 64 and a full launch, samples outside the
caller's arrays, and inputs that the split into BF16 parts cannot hold.

Tolerances: gradients as FP32 sums of the batch, 1e-4 of the largest entry;
inference 1e-5 relative + 5e-5 px (64-term FP32 dot products of O(1-10)
terms); both as derived for the full-size checks."""

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


@pytest.mark.parametrize("n", [1, 15, 17, 63, 64, 65, 257, 768 * 256 + 1])
def test_inference_tile_edges(n):
    from paper_2603_18401_amd import learned_eps as L
    torch = torch_gpu()
    theta = _net(5)
    X = _features(np.random.default_rng(n), n)
    dev = torch.device("cuda:0")
    got = L.infer(torch.from_numpy(X).to(dev), torch.from_numpy(theta).to(dev)).cpu().numpy()
    ref = mlp.infer_bf16(theta, X)
    assert np.all(np.abs(got - ref) <= 1e-5 * ref + 5e-5), np.abs(got - ref).max()


def _plain(theta, X):
    """The network left to right in FP32, max(NaN, 0) = 0."""
    u = theta.view(np.uint32)
    t = ((u + 0x7FFF + ((u >> 16) & 1)) & np.uint32(0xFFFF0000)).view(np.float32)
    w1, b1, w2, b2 = t[:384].reshape(64, 6), t[384:448], t[448:4544].reshape(64, 64), t[4544:4608]
    w3, b3 = t[4608:4672], t[4672]
    out = np.empty(len(X), np.float32)
    with np.errstate(all="ignore"):
        for k, x in enumerate(X.astype(np.float32)):
            a = b1.copy()
            for c in range(6):
                a = a + w1[:, c] * x[c]
            h = np.fmax(a, np.float32(0))
            a = b2.copy()
            for c in range(64):
                a = a + w2[:, c] * h[c]
            z = np.float64(b3)
            for c in range(64):
                z = z + np.float64(w3[c]) * np.fmax(a[c], np.float32(0))
            sp = np.fmax(z, 0) + np.log1p(np.exp(-np.abs(z)))
            out[k] = np.fmin(np.fmax(sp, 0.5), 8.0)
    return out


@pytest.mark.parametrize("what", ["features", "weights"])
def test_inference_of_what_a_split_cannot_hold(what):
    from paper_2603_18401_amd import learned_eps as L
    torch = torch_gpu()
    theta = _net(6)
    X = _features(np.random.default_rng(1), 200)
    if what == "features":
        X[3, 5], X[70, 0], X[71, 1], X[130, 2], X[199, 0] = np.inf, np.nan, -np.inf, 1e20, 3e38
    else:
        theta[448 + 77] = np.inf
        theta[4544 + 9] = np.nan
    dev = torch.device("cuda:0")
    got = L.infer(torch.from_numpy(X).to(dev), torch.from_numpy(theta).to(dev)).cpu().numpy()
    ref = _plain(theta, X)
    assert np.all(np.abs(got - ref) <= 1e-5 * ref + 5e-5), np.abs(got - ref).max()
