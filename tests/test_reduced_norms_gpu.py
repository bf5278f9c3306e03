"""Reduced-precision selection of descriptors beside others of very different
norms: norms past FP16's range, in which the row terms of the bounds are kept,
and squared norms that overflow FP32, where the approximate distances are
infinite.  The matches have to be those of the oracle's FP32 selection, in
which a candidate at infinite distance is still a candidate."""

import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import fp8_rows, torch_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("big", [2e19, 1.4e19, 1e9, 1e5])
@pytest.mark.parametrize("call", ["match_bf16", "query_match_bf16", "query_match_fp8"])
def test_norms_of_every_size(call, big):
    import paper_2603_18401_amd as E
    torch = torch_gpu()
    dev = torch.device("cuda:0")
    g = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    p = synth.cfg0_pair(6)
    d1, d2 = p.desc1.copy(), p.desc2.copy()
    d1[::7] *= np.float32(big)  # unit rows: |q|^2 = 4e38 overflows, twice 2e38 does
    d2[::5] *= np.float32(big)
    eps = 6.0
    with np.errstate(over="ignore", invalid="ignore"):
        ro, rc, _ = oracle.candidates(p.F, p.kp1, p.kp2, eps)
        want = oracle.match(d1, d2, ro, rc)
    if big > 1.9e19:
        assert (want[0][np.isinf(want[1])] >= 0).any()  # matches at infinite distance
    idx = E.Index([E.PairSpec(p.F, p.W, p.H, p.m, p.n)], g(p.kp2), eps=eps)
    f1, f2 = g(d1), g(d2)
    c1, c2 = E.quantize(f1, "bf16"), E.quantize(f2, "bf16")
    if call == "match_bf16":
        offs, cols = idx.query(g(p.kp1))
        got = idx.match(offs, cols, c1, c2, dtype="bf16", desc1_f32=f1, desc2_f32=f2)
    elif call == "query_match_bf16":
        got = idx.query_match_bf16(g(p.kp1), c1, c2, f1, f2)[2:]
    else:
        codes, scale, err = fp8_rows(d2)
        got = idx.query_match_fp8(g(p.kp1), g(codes), g(scale), g(err), f1, f2)[2:]
    for name, a, b in zip(("best", "distance", "second"), got, want):
        assert np.array_equal(a.cpu().numpy().view(np.uint32), b.view(np.uint32)), name
