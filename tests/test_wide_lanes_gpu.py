"""The wide rows' selection keeps three keys per lane: a row's entries are dealt
to four lanes, entries 4 g .. 4 g + 3 of every 16 to lane group g.  Rows whose
nearest candidates all belong to one lane, at the edges of the blocks of 64 and
the rounds of 256 entries, against the oracle, bit by bit."""

import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import torch_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [129, 192, 193, 256, 257, 513, 1100])
@pytest.mark.parametrize("near", [1, 2, 3, 4, 7])
def test_nearest_in_one_lane(n, near):
    import paper_2603_18401_amd as E
    torch = torch_gpu()
    dev = torch.device("cuda:0")
    g = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    m = 70
    rng = np.random.default_rng(100 * n + near)
    p = synth.make_pair(1920, 1080, 1080.0, np.eye(3), [1.0, 0.0, 0.0], 8, 0, 0, n,
                        float_desc=False)
    # a strip of 20 rows and a tolerance of 30: every keypoint is a candidate,
    # so entry e of a row is keypoint e
    kp1, kp2 = [np.stack([rng.random(k) * 1900, 500 + 20 * rng.random(k)], 1).astype(np.float32)
                for k in (m, n)]
    d1 = synth.pairs._unit_rows(rng.standard_normal((m, 128)))
    d2 = synth.pairs._unit_rows(rng.standard_normal((n, 128)))
    for grp in range(4):
        lane = np.where((np.arange(n) % 16) // 4 == grp)[0]
        at = np.unique(np.concatenate([lane[-near:], lane[:near]]))[-near:]
        dd = d2.copy()
        for t, j in enumerate(at):  # near all queries' mean, at growing distances; two are equal
            dd[j] = synth.pairs._unit_rows(
                (d1.mean(0) + (0.02 * min(t, 3)) * d2[at[0]])[None].astype(np.float32))[0]
        ro, rc, _ = oracle.candidates(p.F, kp1, kp2, 30.0)
        assert np.all(np.diff(ro) == n)
        rb, rbd, rsd = oracle.match(d1, dd, ro, rc)
        idx = E.Index([E.PairSpec(p.F, 1920, 1080, m, n)], g(kp2), eps=30.0)
        f1, f2 = g(d1), g(dd)
        c1, c2 = E.quantize(f1, "bf16"), E.quantize(f2, "bf16")
        offs, cols, *got = idx.query_match(g(kp1), f1, f2)
        assert np.array_equal(offs.cpu().numpy(), ro) and np.array_equal(cols.cpu().numpy(), rc)
        results = [got, idx.query_match_bf16(g(kp1), c1, c2, f1, f2)[2:]]
        offs, cols = idx.query(g(kp1))
        results.append(idx.match(offs, cols, f1, f2))
        results.append(idx.match(offs, cols, c1, c2, dtype="bf16", desc1_f32=f1, desc2_f32=f2))
        for b, bd, sd in results:
            assert np.array_equal(b.cpu().numpy(), rb)
            assert np.array_equal(bd.cpu().numpy().view(np.uint32), rbd.view(np.uint32))
            assert np.array_equal(sd.cpu().numpy().view(np.uint32), rsd.view(np.uint32))
