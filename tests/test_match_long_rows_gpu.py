"""epm_match over rows around the length of the window kernels' dense lists
(8192 entries with BF16 rows and measured errors or FP8 rows, 4096 with FP32
rows): alone in their tile, where the first row may fill the whole list, and
behind other rows -- against the oracle."""

import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import fp8_rows, torch_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [0, 2])
@pytest.mark.parametrize("dtype,entries", [("f32", 4096), ("bf16", 8192), ("fp8", 8192)])
def test_rows_around_the_list(dtype, entries, grid):
    import paper_2603_18401_amd as E
    torch = torch_gpu()
    dev = torch.device("cuda:0")
    g = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    p = synth.cfg0_pair(2)
    n = entries + 700
    rng = np.random.default_rng(5)
    # a pair per row length (one query, a tile of its own), then one with many rows
    alone = (entries - 1, entries, entries + 1, n)
    many = [30] * 40 + [entries - 1200, 30, entries + 1, 0, 30] + [200] * 10
    lengths = list(alone) + many
    counts = [1] * len(alone) + [len(many)]
    m, P = len(lengths), len(counts)
    wh = np.array([p.W, p.H])
    kp1 = (rng.random((m, 2)) * wh).astype(np.float32)
    kp2 = (rng.random((P * n, 2)) * wh).astype(np.float32)
    d1, d2 = (rng.standard_normal((k, 128)).astype(np.float32) for k in (m, P * n))
    d2[::11] = d2[0]  # ties
    rows = [np.sort(rng.choice(n, L, replace=False)).astype(np.int32) for L in lengths]
    offs = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    cols = np.concatenate(rows)
    pair = np.repeat(np.arange(P), counts)
    want = [np.empty(m, t) for t in (np.int32, np.float32, np.float32)]
    for i in range(m):
        got = oracle.match(d1[i:i + 1], d2[pair[i] * n:(pair[i] + 1) * n],
                           np.array([0, lengths[i]], np.int64), rows[i])
        for w, v in zip(want, got):
            w[i] = v[0]
    # narrow tolerances: none of the tiles is left to the wide-row pass
    idx = E.Index([E.PairSpec(p.F, p.W, p.H, c, n) for c in counts], g(kp2), eps=0.01)
    idx.set_sched(E.Sched(0, grid))
    idx.query(g(kp1))
    f1, f2 = g(d1), g(d2)
    more = {} if dtype == "f32" else dict(desc1_f32=f1, desc2_f32=f2)
    if dtype == "f32":
        r1, r2 = f1, f2
    elif dtype == "bf16":
        r1, r2 = E.quantize(f1, "bf16"), E.quantize(f2, "bf16")
        more.update(qerr1=E.rounding_error(f1, r1, "bf16"), qerr2=E.rounding_error(f2, r2, "bf16"))
    else:
        (c1, s1, _), (c2, s2, _) = fp8_rows(d1), fp8_rows(d2)
        r1, r2 = g(c1), g(c2)
        more.update(scale1=g(s1), scale2=g(s2))
    got = idx.match(g(offs), g(cols), r1, r2, dtype=dtype, **more)
    for name, a, b in zip(("best", "distance", "second"), got, want):
        assert np.array_equal(a.cpu().numpy().view(np.uint32), b.view(np.uint32)), name
    if dtype != "f32":
        longs = [L for L in alone if L > entries]
        assert idx.match_stats()["long_rows"] >= len(longs)
