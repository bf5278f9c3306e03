"""Keypoints that crowd into a small part of the angles seen from the epipole:
the query sort puts hundreds of them into one of its 2048 groups, and the
tiles must still hold queries that are neighbours in angle.  Candidates and
matches against the oracle; the counter of scanned records tells whether the
windows follow the queries."""

import numpy as np
import pytest

import oracle
from tests.gpu_util import torch_gpu

pytestmark = pytest.mark.gpu

W, H = 6048, 4032


def _F(ex, ey):
    """Pure translation: lines through the epipole (ex, ey)."""
    e = np.array([ex, ey, 1.0])
    e /= np.linalg.norm(e)
    return np.array([[0, -e[2], e[1]], [e[2], 0, -e[0]], [-e[1], e[0], 0]])


def _points(rng, kind, n):
    c = np.array([W - 500.0, H / 2])
    if kind == "cluster":
        return c + 40.0 * rng.standard_normal((n, 2))
    if kind == "two":  # two clusters and a few points anywhere
        p = c + 12.0 * rng.standard_normal((n, 2))
        p[: n // 3] = np.array([800.0, 900.0]) + 25.0 * rng.standard_normal((n // 3, 2))
        p[n - n // 10:] = rng.random((n // 10, 2)) * [W, H]
        return p
    if kind == "rays":  # a few directions, each of many equal keys
        a = rng.integers(0, 7, n) * 0.01 + 0.3
        r = rng.integers(100, 2000, n)
        return np.stack([W / 2 - 500 + r * np.cos(a), H / 2 + r * np.sin(a)], 1)
    raise ValueError(kind)


# the last: whether the crowds fill groups of more than two tiles (or the tiles
# are small), so that the queries have to be in order
CASES = [("cluster", (300,), (900,), False), ("cluster", (1024, 1025), (1500, 700), False),
         ("cluster", (5000,), (5000,), True), ("two", (4000, 60, 2500), (3000, 400, 2500), True),
         ("two", (900,), (20000,), True), ("cluster", (700, 1300), (6000, 24000), True),
         ("rays", (3000,), (3000,), True), ("rays", (600, 700), (600, 700), True),
         ("cluster", (131072,), (300,), True)]


@pytest.mark.parametrize("kind,ms,ns,ordered", CASES)
def test_crowded_queries(kind, ms, ns, ordered):
    import paper_2603_18401_amd as E
    torch = torch_gpu()
    dev = torch.device("cuda:0")
    g = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    rng = np.random.default_rng(len(kind) + sum(ms))
    F = _F(W / 2 - 500, H / 2)
    kp1 = np.concatenate([_points(rng, kind, m) for m in ms]).astype(np.float32)
    kp2 = np.concatenate([_points(rng, kind, n) for n in ns]).astype(np.float32)
    d1, d2 = (rng.standard_normal((len(k), 128)).astype(np.float32) for k in (kp1, kp2))
    qb = np.concatenate([[0], np.cumsum(ms)]).astype(np.int64)
    kb = np.concatenate([[0], np.cumsum(ns)]).astype(np.int64)
    eps = 0.3
    ro, rc, _ = oracle.candidates_batch([F] * len(ms), kp1, kp2, eps, qb[:-1], list(ms), kb[:-1],
                                        list(ns))
    idx = E.Index([E.PairSpec(F, W, H, m, n) for m, n in zip(ms, ns)], g(kp2), eps=eps)
    offs, cols, best, bd, sd = idx.query_match(g(kp1), g(d1), g(d2))
    assert np.array_equal(offs.cpu().numpy(), ro) and np.array_equal(cols.cpu().numpy(), rc)
    scanned = idx.stats()["records_scanned"]
    want = [np.concatenate(v) for v in zip(*[
        oracle.match(d1[q0:q1], d2[k0:k1], ro[q0:q1 + 1] - ro[q0], rc[ro[q0]:ro[q1]])
        for q0, q1, k0, k1 in zip(qb, qb[1:], kb, kb[1:])])]
    for a, b in zip((best, bd, sd), want):
        assert np.array_equal(a.cpu().numpy().view(np.uint32), b.view(np.uint32))
    offs, cols = idx.query(g(kp1))  # the counting pass, and a match over its tiles
    assert np.array_equal(offs.cpu().numpy(), ro) and np.array_equal(cols.cpu().numpy(), rc)
    f1, f2 = g(d1), g(d2)
    got = idx.match(offs, cols, E.quantize(f1, "bf16"), E.quantize(f2, "bf16"), dtype="bf16",
                    desc1_f32=f1, desc2_f32=f2)
    for a, b in zip(got, want):
        assert np.array_equal(a.cpu().numpy().view(np.uint32), b.view(np.uint32))
    # a query scans the records that can meet the 16 queries around it; parts
    # of groups that cross from one workgroup (256 queries) to the next may stay
    # unsorted there
    if ordered:
        assert scanned <= 1.5 * sum(
            _least_scans(kp1[q0:q1], kp2[k0:k1], eps) for q0, q1, k0, k1 in
            zip(qb, qb[1:], kb, kb[1:]))


def _least_scans(kp1, kp2, eps):
    """Records scanned by queries in the order of their angles: every 16 of them
    scan the intervals that meet their span, wherever the groups of 16 start."""
    c = np.array([W / 2 - 500, H / 2])
    # (angles from a direction where no cluster lies)
    a1, a2 = ((np.arctan2(*(k.astype(float) - c).T[::-1]) + 1.0) % np.pi for k in (kp1, kp2))
    d = np.hypot(*(kp2.astype(float) - c).T)
    half = np.arcsin(np.minimum(1.0, eps / np.maximum(d, eps)))
    a1 = np.sort(a1)
    lo, hi = np.sort(a2 - half), np.sort(a2 + half)
    wrap = (a2 - half < 0) | (a2 + half > np.pi)  # (counted for every group)
    most = 0
    for o in range(16):
        at = np.concatenate([[0], np.arange(o, len(a1), 16), [len(a1)]])
        at = np.unique(at)
        first, last, size = a1[at[:-1]], a1[at[1:] - 1], np.diff(at)
        meets = np.searchsorted(lo, last, "right") - np.searchsorted(hi, first, "left")
        most = max(most, int((size * (meets + wrap.sum())).sum()))
    return most
