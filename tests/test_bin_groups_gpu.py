"""Binary matches of calls with many queries (16 lanes per query from 32768 on):
rows of every length around the groups' rounds, ties and repeated candidates,
against the oracle, on both sides of the line."""

import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import torch_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [32767, 32768, 32783])
@pytest.mark.parametrize("ratio", [0.0, 0.9])
def test_rows_of_every_length(m, ratio):
    import paper_2603_18401_amd as E
    torch = torch_gpu()
    dev = torch.device("cuda:0")
    g = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    rng = np.random.default_rng(m)
    n = 500
    p = synth.make_pair(1920, 1080, 1080.0, np.eye(3), [1.0, 0.0, 0.0], 8, 0, 0, 1,
                        float_desc=False)
    b1 = rng.integers(0, 2**32, (m, 8), dtype=np.uint32)
    b2 = rng.integers(0, 2**32, (n, 8), dtype=np.uint32)
    b2[10:40] = b2[:30]  # equal distances: the lower j wins
    b1[:200] = b2[rng.integers(0, n, 200)]
    lens = rng.integers(0, 12, m)
    lens[:140] = np.arange(140)
    lens[-3:] = (0, 33, 1)
    cols = [np.sort(rng.choice(n, k, replace=False)) for k in lens]
    cols[9][1:4] = cols[9][0]  # a repeated candidate
    ro = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    rc = np.concatenate(cols).astype(np.int32)
    kp = lambda k: g((rng.random((k, 2)) * [1900, 1000]).astype(np.float32))  # noqa: E731
    idx = E.Index([E.PairSpec(p.F, 1920, 1080, m, n)], kp(n), eps=1.0)
    d1, d2 = g(b1.view(np.int32)), g(b2.view(np.int32))
    rb, rbd, rsd = oracle.match(b1, b2, ro, rc, ratio=ratio, binary=True)
    for queried in (False, True):  # rows in the caller's order, then in the tiles' order
        if queried:
            idx.query(kp(m))
        b, bd, sd = idx.match(g(ro), g(rc), d1, d2, dtype="bin256", ratio=ratio)
        assert np.array_equal(b.cpu().numpy(), rb)
        assert np.array_equal(bd.cpu().numpy(), rbd) and np.array_equal(sd.cpu().numpy(), rsd)
