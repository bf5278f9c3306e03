"""The angle sort at the edges of its tiles (1024 elements, 2-pass records,
one or two passes for the queries) and of the pairs' arcs of keys: the
candidate sets against the oracle, and the number of records scanned against
what a full sort by angle needs."""

import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import torch_gpu

pytestmark = pytest.mark.gpu

POSES = {
    "far": (synth.pairs._yaw(1e-4), [1.0, 0.0, 0.0]),
    "infinite": (np.eye(3), [1.0, 0.0, 0.0]),
    "vertical": (np.eye(3), [0.0, 1.0, 0.0]),
    "forward": (np.eye(3), [0.0, 0.0, 1.0]),
    "backward": (synth.pairs._yaw(3.0), [0.1, 0.05, -1.0]),
    "edge": (np.eye(3), [0.62, 0.1, 0.8]),   # the epipole near the image's right edge
    "oblique": (synth.pairs._yaw(12.0), [0.8, -0.5, 0.3]),
}


def _pair(pose, m, n, seed):
    R, C2 = POSES[pose]
    p = synth.make_pair(1920, 1080, 1080.0, R, C2, 8, 0, 0, seed, float_desc=False)
    rng = np.random.default_rng(seed)
    # some keypoints lie outside the image, beyond the pair's arc
    kp = [(rng.random((k, 2)) * [2100, 1300] - [90, 110]).astype(np.float32) for k in (m, n)]
    return p.F, kp[0], kp[1]


def _check(torch, E, pairs, eps):
    dev = torch.device("cuda:0")
    g = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    specs = [E.PairSpec(F, 1920, 1080, len(a), len(b)) for F, a, b in pairs]
    idx = E.Index(specs, g(np.concatenate([b for _, _, b in pairs])), eps=eps)
    offs, cols = idx.query(g(np.concatenate([a for _, a, _ in pairs])))
    offs, cols = offs.cpu().numpy(), cols.cpu().numpy()
    q = 0
    for F, a, b in pairs:
        ro, rc, _ = oracle.candidates(F, a, b, eps)
        assert np.array_equal(offs[q:q + len(a) + 1] - offs[q], ro)
        assert np.array_equal(cols[offs[q]:offs[q + len(a)]], rc)
        q += len(a)
    return idx.stats()


@pytest.mark.parametrize("m,n", [(1, 1), (63, 1023), (1024, 1024), (1025, 1025), (2048, 2049),
                                 (700, 5000), (5000, 700)])
def test_tile_edges(m, n):
    import paper_2603_18401_amd as E
    torch = torch_gpu()
    names = sorted(POSES)
    _check(torch, E, [_pair(names[k % len(names)], m, n, 10 * k + m) for k in range(3)], 3.0)
    # segments of one and of several tiles, and empty ones, in one batch
    _check(torch, E, [_pair("far", m, n, 1), _pair("edge", 0, 9, 2), _pair("forward", 90, 0, 3),
                      _pair("oblique", 3000, 40, 4), _pair("infinite", 20, 2100, 5)], 3.0)


@pytest.mark.parametrize("pose", sorted(POSES))
def test_arcs(pose):
    import paper_2603_18401_amd as E
    torch = torch_gpu()
    st = _check(torch, E, [_pair(pose, 4000, 4000, 77)], 2.0)
    # a tile of 64 queries spans 1/62 of the pair's records; its window adds
    # the tolerance on both sides, and the width classes round it up to twice:
    # a sort that missed the arc would scan half of the pair or all of it
    assert st["scanned_queries"] < 100
    assert st["records_scanned"] <= 4000 * 4000 * 0.1
    assert st["candidates"] <= st["angle_hits"] <= st["records_scanned"]


def test_two_pass_queries():
    import paper_2603_18401_amd as E
    torch = torch_gpu()
    _check(torch, E, [_pair("far", 131073, 50, 5), _pair("forward", 700, 60, 6)], 2.0)
    _check(torch, E, [_pair("oblique", 40, 131100, 7)], 0.5)


@pytest.mark.parametrize("m,n", [(70, 560), (70, 561), (70, 1121), (70, 2241), (9, 6000),
                                 (500, 5000), (1, 300)])
def test_uneven_pairs_take_smaller_tiles(m, n):
    """8, 16 and 32 image-2 keypoints per query are the edges of the rule:
    candidates and FP32 / BF16 matches equal the oracle's on both sides."""
    import paper_2603_18401_amd as E
    torch = torch_gpu()
    dev = torch.device("cuda:0")
    g = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    F, kp1, kp2 = _pair("oblique", m, n, m + n)
    rng = np.random.default_rng(n)
    d1 = synth.pairs._unit_rows(rng.standard_normal((m, 128)))
    d2 = synth.pairs._unit_rows(rng.standard_normal((n, 128)))
    for eps in (2.0, 12.0):
        ro, rc, _ = oracle.candidates(F, kp1, kp2, eps)
        rb, rbd, rsd = oracle.match(d1, d2, ro, rc)
        idx = E.Index([E.PairSpec(F, 1920, 1080, m, n)], g(kp2), eps=eps)
        f1, f2 = g(d1), g(d2)
        for got in (idx.query_match(g(kp1), f1, f2),
                    idx.query_match_bf16(g(kp1), E.quantize(f1, "bf16"), E.quantize(f2, "bf16"),
                                         f1, f2)):
            offs, cols, b, bd, sd = [t.cpu().numpy() for t in got]
            assert np.array_equal(offs, ro) and np.array_equal(cols, rc)
            assert np.array_equal(b, rb)
            assert np.array_equal(bd.view(np.uint32), rbd.view(np.uint32))
            assert np.array_equal(sd.view(np.uint32), rsd.view(np.uint32))
        offs, cols = idx.query(g(kp1))
        b, bd, sd = [t.cpu().numpy() for t in idx.match(offs, cols, f1, f2)]
        assert np.array_equal(b, rb) and np.array_equal(sd.view(np.uint32), rsd.view(np.uint32))
