"""epm_match with BF16 rows over a caller's CSR: the candidates as the query
wrote them, and rows that did not come from it -- filtered, shuffled, with
repeated or foreign candidates, empty, and longer than 128 -- against the
oracle's FP32 selection, in every schedule."""

import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import torch_gpu

pytestmark = pytest.mark.gpu


def _rows(kind, ro, rc, n, rng):
    rows = [rc[ro[i]:ro[i + 1]] for i in range(len(ro) - 1)]
    if kind == "query":
        return rows
    if kind == "filtered":
        return [r[rng.random(len(r)) < 0.5] for r in rows]
    if kind == "shuffled":
        return [rng.permutation(r) for r in rows]
    if kind == "repeated":
        return [np.concatenate([r, r[:2]]) if i % 3 == 0 else r for i, r in enumerate(rows)]
    if kind == "foreign":
        return [np.concatenate([r, rng.integers(0, n, 3)]) if i % 2 else r
                for i, r in enumerate(rows)]
    if kind == "long":
        return [rng.integers(0, n, 129 + i % 40) if i % 7 == 0 else r for i, r in enumerate(rows)]
    raise ValueError(kind)


@pytest.mark.parametrize("grid", [0, 3])
@pytest.mark.parametrize("kind", ["query", "filtered", "shuffled", "repeated", "foreign", "long"])
def test_bf16_match_of_any_csr(kind, grid):
    import paper_2603_18401_amd as E
    torch = torch_gpu()
    dev = torch.device("cuda:0")
    g = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    p = synth.cfg0_pair(4)
    rng = np.random.default_rng(8)
    m, n = 700, 1000
    kp1, d1 = p.kp1[:m], p.desc1[:m]
    # many equal distances among the rows of a few prototypes
    d2 = p.desc2.copy()
    d2[::9] = d2[0]
    F = p.F
    for eps in (0.4, 2.0, 9.0, 45.0):  # windows and rows beyond the tile's limits at the last
        ro, rc, _ = oracle.candidates(F, kp1, p.kp2, eps)
        rows = _rows(kind, ro, rc, n, rng)
        offs = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
        cols = np.concatenate(rows).astype(np.int32)
        for ratio in (0.0, 0.8):
            # the oracle's rows are sets; a repeated candidate is its own second
            rb = np.full(m, -1, np.int32)
            rbd = np.full(m, np.inf, np.float32)
            rsd = np.full(m, np.inf, np.float32)
            one = np.arange(len(cols) + 1, dtype=np.int64)
            qi = np.repeat(np.arange(m), np.diff(offs))
            _, dist, _ = oracle.match(d1[qi], d2, one, cols)
            for i in range(m):
                d, j = dist[offs[i]:offs[i + 1]], cols[offs[i]:offs[i + 1]]
                o = np.lexsort((j, d))
                if len(o):
                    rb[i], rbd[i] = j[o[0]], d[o[0]]
                if len(o) > 1:
                    rsd[i] = d[o[1]]
                if ratio and rb[i] >= 0 and not rbd[i] < np.float32(ratio) * np.float32(ratio) * rsd[i]:
                    rb[i] = -1
            idx = E.Index([E.PairSpec(F, p.W, p.H, m, n)], g(p.kp2), eps=eps)
            idx.set_sched(E.Sched(0, grid))
            idx.query(g(kp1))
            f1, f2 = g(d1), g(d2)
            b, bd, sd = idx.match(g(offs), g(cols), E.quantize(f1, "bf16"), E.quantize(f2, "bf16"),
                                  dtype="bf16", desc1_f32=f1, desc2_f32=f2, ratio=ratio)
            assert np.array_equal(bd.cpu().numpy().view(np.uint32), rbd.view(np.uint32))
            assert np.array_equal(sd.cpu().numpy().view(np.uint32), rsd.view(np.uint32))
            assert np.array_equal(b.cpu().numpy(), rb)
            st = idx.match_stats()
            assert st["fallback_rows"] <= st["reranked_rows"] <= m
