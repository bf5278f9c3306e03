"""Pairs with many records per query, whose queries per tile are decided on the
device: from few candidates per query to rows far beyond 128, sizes around the
tiles' edges, alone and beside even pairs, in every schedule -- candidates,
fused and separate matches against the oracle."""

import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import fp8_rows, torch_gpu

pytestmark = pytest.mark.gpu

SIZES = {"one": [(1, 60)], "edges": [(63, 1100), (64, 1100), (65, 1100), (129, 2500), (8, 900)],
         "mixed": [(300, 300), (150, 5000), (0, 700), (90, 0), (40, 900), (257, 4200), (500, 200)],
         "crowd": [(100, 1700)] * 40}


@pytest.mark.parametrize("sched", [(0, 0, 0), (3, 2, 1)])
@pytest.mark.parametrize("eps", [0.3, 2.0, 30.0])
@pytest.mark.parametrize("sizes", list(SIZES))
def test_queries_per_tile(sizes, eps, sched):
    import paper_2603_18401_amd as E
    torch = torch_gpu()
    dev = torch.device("cuda:0")
    g = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    rng = np.random.default_rng(len(sizes))
    p = synth.cfg0_pair(5)
    wh = np.array([p.W, p.H])
    m, n = [s[0] for s in SIZES[sizes]], [s[1] for s in SIZES[sizes]]
    qb, kb = (np.concatenate([[0], np.cumsum(v)]).astype(np.int64) for v in (m, n))
    kp1 = (rng.random((qb[-1], 2)) * wh).astype(np.float32)
    kp2 = (rng.random((kb[-1], 2)) * wh).astype(np.float32)
    d1, d2 = (rng.standard_normal((len(k), 128)).astype(np.float32) for k in (kp1, kp2))
    # every third pair crowds around a point
    for k in range(0, len(m), 3):
        kp1[qb[k]:qb[k + 1]] = wh / 3 + 9.0 * rng.standard_normal((m[k], 2))
        kp2[kb[k]:kb[k + 1]] = wh / 3 + 9.0 * rng.standard_normal((n[k], 2))
    ro, rc, _ = oracle.candidates_batch([p.F] * len(m), kp1, kp2, eps, qb[:-1], m, kb[:-1], n)
    want = [np.concatenate(v) for v in zip(*[
        oracle.match(d1[a:b], d2[c:d], ro[a:b + 1] - ro[a], rc[ro[a]:ro[b]])
        for a, b, c, d in zip(qb, qb[1:], kb, kb[1:]) if b > a])]
    idx = E.Index([E.PairSpec(p.F, p.W, p.H, a, b) for a, b in zip(m, n)], g(kp2), eps=eps)
    idx.set_sched(E.Sched(*sched))
    f1, f2, k1 = g(d1), g(d2), g(kp1)
    c1, c2 = E.quantize(f1, "bf16"), E.quantize(f2, "bf16")
    codes, scale, err = (g(a) for a in fp8_rows(d2))
    q1, s1 = E.quantize(f1, "fp8")

    def same(got, what):
        for a, b in zip(got, want):
            assert np.array_equal(a.cpu().numpy().view(np.uint32), b.view(np.uint32)), what

    def csr(offs, cols, what):
        assert np.array_equal(offs.cpu().numpy(), ro), what
        assert np.array_equal(cols.cpu().numpy(), rc), what

    fused = {"f32": lambda: idx.query_match(k1, f1, f2),
             "bf16": lambda: idx.query_match_bf16(k1, c1, c2, f1, f2),
             "fp8": lambda: idx.query_match_fp8(k1, codes, scale, err, f1, f2)}
    for what, call in fused.items():
        offs, cols, *got = call()
        csr(offs, cols, what)
        same(got, what)
    st = idx.stats()
    assert st["candidates"] == len(rc) and st["queries"] == qb[-1]
    offs, cols = idx.query(k1)
    csr(offs, cols, "query")
    masters = dict(desc1_f32=f1, desc2_f32=f2)
    same(idx.match(offs, cols, f1, f2), "match f32")
    same(idx.match(offs, cols, c1, c2, dtype="bf16", **masters), "match bf16")
    same(idx.match(offs, cols, c1, c2, dtype="bf16", qerr1=E.rounding_error(f1, c1, "bf16"),
                   qerr2=E.rounding_error(f2, c2, "bf16"), **masters), "match bf16 errors")
    same(idx.match(offs, cols, q1, codes, dtype="fp8", scale1=s1, scale2=scale, **masters),
         "match fp8")
