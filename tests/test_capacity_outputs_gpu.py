"""A query call that waits for its total and finds the column buffer too small
returns EPM_ERR_CAPACITY with the row offsets complete, and leaves the columns
and the match outputs as they were; a retry with room enough succeeds.  For
few queries and for more than the pass over the rows takes in one launch."""

import ctypes

import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import fp8_rows, torch_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("repeat", [1, 300])
@pytest.mark.parametrize("call", ["candidates", "f32", "bf16", "fp8"])
def test_outputs_are_left_alone(call, repeat):
    import paper_2603_18401_amd as E
    torch = torch_gpu()
    dev = torch.device("cuda:0")
    g = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    p = synth.cfg0_pair(1)
    kp1, d1 = np.tile(p.kp1, (repeat, 1)), np.tile(p.desc1, (repeat, 1))
    m, n = len(kp1), 200
    kp2, d2 = p.kp2[:n], p.desc2[:n]
    ro, rc, _ = oracle.candidates(p.F, p.kp1, kp2, 3.0)
    rb, rbd, rsd = oracle.match(p.desc1, d2, ro, rc)
    nnz = repeat * len(rc)
    offs = np.concatenate([[0], np.cumsum(np.tile(np.diff(ro), repeat))]).astype(np.int64)
    idx = E.Index([E.PairSpec(p.F, p.W, p.H, m, n)], g(kp2), eps=3.0)
    f1, f2, k1 = g(d1), g(d2), g(kp1)
    desc = {"candidates": [], "f32": [f1, f2],
            "bf16": [E.quantize(f1, "bf16"), E.quantize(f2, "bf16"), f1, f2],
            "fp8": [g(a) for a in fp8_rows(d2)] + [f1, f2]}[call]
    name = {"candidates": "epm_query_candidates", "f32": "epm_query_match"}.get(
        call, "epm_query_match_" + call)
    off = torch.zeros(m + 1, dtype=torch.int64, device=dev)
    out = [torch.full((m,), -7, dtype=t, device=dev)
           for t in (torch.int32, torch.float32, torch.float32)]
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    cols = None
    for room in (1, nnz // 2, nnz - 1, nnz):
        cols = torch.full((nnz,), -7, dtype=torch.int32, device=dev)
        got = ctypes.c_int64(0)
        args = [idx.handle, ptr(k1), ptr(off), ptr(cols), room, ctypes.byref(got)]
        args += [ptr(t) for t in desc]
        if call != "candidates":
            args += [0.0] + [ptr(t) for t in out]
        st = getattr(idx.lib, name)(*args, None)
        torch.cuda.synchronize()
        assert st == (0 if room == nnz else 3) and got.value == nnz, room
        assert np.array_equal(off.cpu().numpy(), offs), room
        if room < nnz:
            assert bool((cols == -7).all()), room
            assert all(bool((t == -7).all()) for t in out), room
    assert np.array_equal(cols.cpu().numpy(), np.tile(rc, repeat))
    if call != "candidates":
        for t, want in zip(out, (rb, rbd, rsd)):
            assert np.array_equal(t.cpu().numpy().view(np.uint32),
                                  np.tile(want, repeat).view(np.uint32))
