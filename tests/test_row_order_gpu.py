"""Rows leave the tile pass in ascending j whatever the window's size (edges of
its bitmap words, of a round of records and of the longest window kept) and
however its j are spread over the order's buckets.  Candidates and matches
against the oracle, bit by bit."""

import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import torch_gpu

pytestmark = pytest.mark.gpu


def _strip(m, n, order, seed):
    """Horizontal epipolar lines (infinite epipole); all keypoints in a strip of
    20 rows, so a tile's window is nearly all of image 2.  Rows hold 0 to all
    records."""
    p = synth.make_pair(1920, 1080, 1080.0, np.eye(3), [1.0, 0.0, 0.0], 8, 0, 0, seed,
                        float_desc=False)
    rng = np.random.default_rng(seed)
    kp1 = np.stack([rng.random(m) * 1900, 500 + 20 * rng.random(m)], 1).astype(np.float32)
    kp2 = np.stack([rng.random(n) * 1900, 500 + 20 * rng.random(n)], 1).astype(np.float32)
    if order == "raster":
        kp2 = kp2[np.argsort(kp2[:, 1], kind="stable")]
    elif order == "skewed":
        # 3000 keypoints far from the strip keep the j of the window's records
        # in one bucket, but for one at the end
        far = np.stack([rng.random(3000) * 1900, 5 + 100 * rng.random(3000)], 1)
        kp2 = np.concatenate([kp2[:-1], far.astype(np.float32), kp2[-1:]])
    return p.F, kp1, kp2


@pytest.mark.parametrize("order", ["random", "raster", "skewed"])
@pytest.mark.parametrize("n", [1, 2, 32, 33, 128, 129, 256, 257, 511, 513, 1023, 1024, 1025, 1300])
def test_rows_ascend(n, order):
    import paper_2603_18401_amd as E
    torch = torch_gpu()
    dev = torch.device("cuda:0")
    g = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    m = 70
    F, kp1, kp2 = _strip(m, n, order, n)
    nt = len(kp2)
    rng = np.random.default_rng(n)
    d1 = synth.pairs._unit_rows(rng.standard_normal((m, 128)))
    d2 = synth.pairs._unit_rows(rng.standard_normal((nt, 128)))
    f1, f2 = g(d1), g(d2)
    c1, c2 = E.quantize(f1, "bf16"), E.quantize(f2, "bf16")
    c8, s8 = E.quantize(f2, "fp8")
    e8 = E.rounding_error(f2, c8, "fp8", s8)
    for eps in (0.4, 2.0, 6.0):
        ro, rc, _ = oracle.candidates(F, kp1, kp2, eps)
        rb, rbd, rsd = oracle.match(d1, d2, ro, rc)
        idx = E.Index([E.PairSpec(F, 1920, 1080, m, nt)], g(kp2), eps=eps)
        offs, cols = [t.cpu().numpy() for t in idx.query(g(kp1))]
        assert np.array_equal(offs, ro) and np.array_equal(cols, rc)
        for got in (idx.query_match(g(kp1), f1, f2),
                    idx.query_match_bf16(g(kp1), c1, c2, f1, f2),
                    idx.query_match_fp8(g(kp1), c8, s8, e8, f1, f2)):
            offs, cols, b, bd, sd = [t.cpu().numpy() for t in got]
            assert np.array_equal(offs, ro) and np.array_equal(cols, rc)
            assert np.array_equal(b, rb)
            assert np.array_equal(bd.view(np.uint32), rbd.view(np.uint32))
            assert np.array_equal(sd.view(np.uint32), rsd.view(np.uint32))


@pytest.mark.parametrize("n", [60, 500, 900, 2500])
def test_rows_of_scanned_queries(n):
    """Queries whose line misses the epipole (a matrix of full rank) are scanned
    against all of image 2; their rows are sorted by their wavefront."""
    import paper_2603_18401_amd as E
    torch = torch_gpu()
    dev = torch.device("cuda:0")
    g = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    m = 130
    F, kp1, kp2 = _strip(m, n, "random", n)
    F = F + 1e-5 * np.abs(F).max() * np.eye(3)
    for eps in (0.5, 1.5, 4.0):
        ro, rc, _ = oracle.candidates(F, kp1, kp2, eps)
        idx = E.Index([E.PairSpec(F, 1920, 1080, m, n)], g(kp2), eps=eps)
        offs, cols = [t.cpu().numpy() for t in idx.query(g(kp1))]
        assert idx.stats()["scanned_queries"] > 0
        assert np.array_equal(offs, ro) and np.array_equal(cols, rc)


@pytest.mark.parametrize("n", [60, 900, 2500])
def test_left_over_rows_are_rebuilt_and_matched(n):
    """Scanned queries after a fused pass, without a wait in between: the rows
    and their matches, and in a buffer that is too small the rows as far as
    they go."""
    import paper_2603_18401_amd as E
    torch = torch_gpu()
    dev = torch.device("cuda:0")
    g = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    m = 130
    F, kp1, kp2 = _strip(m, n, "raster", n)
    F = F + 1e-5 * np.abs(F).max() * np.eye(3)
    rng = np.random.default_rng(n)
    d1 = synth.pairs._unit_rows(rng.standard_normal((m, 128)))
    d2 = synth.pairs._unit_rows(rng.standard_normal((n, 128)))
    f1, f2, k1 = g(d1), g(d2), g(kp1)
    c1, c2 = E.quantize(f1, "bf16"), E.quantize(f2, "bf16")
    for eps in (0.5, 4.0):
        ro, rc, _ = oracle.candidates(F, kp1, kp2, eps)
        rb, rbd, rsd = oracle.match(d1, d2, ro, rc)
        for room in (len(rc) + 3, max(1, len(rc) // 2)):
            idx = E.Index([E.PairSpec(F, 1920, 1080, m, n)], g(kp2), eps=eps)
            for bf16 in (False, True):
                offs = torch.empty(m + 1, dtype=torch.int64, device=dev)
                cols = torch.full((room,), -7, dtype=torch.int32, device=dev)
                kw = dict(row_offsets=offs, col_indices=cols, sync=False)
                out = (idx.query_match_bf16(k1, c1, c2, f1, f2, **kw) if bf16
                       else idx.query_match(k1, f1, f2, **kw))
                assert idx.stats()["scanned_queries"] > 0
                assert np.array_equal(offs.cpu().numpy(), ro)
                k = min(room, len(rc))
                assert np.array_equal(cols.cpu().numpy()[:k], rc[:k])
                assert np.all(cols.cpu().numpy()[k:] == -7)
                if room >= len(rc):
                    b, bd, sd = [t.cpu().numpy() for t in out[2:]]
                    assert np.array_equal(b, rb)
                    assert np.array_equal(bd.view(np.uint32), rbd.view(np.uint32))
                    assert np.array_equal(sd.view(np.uint32), rsd.view(np.uint32))
