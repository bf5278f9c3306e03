"""The pass that turns row lengths into the CSR and the fused matches, at the
edges of its workgroups (256 queries) and of its one-launch form (262144):
rows of 0, under 16, over 16 and over 128 candidates against the oracle."""

import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import torch_gpu

pytestmark = pytest.mark.gpu


def _case(m, n, seed):
    rng = np.random.default_rng(seed)
    p = synth.cfg0_pair(0)
    kp1 = (rng.random((m, 2)) * [640, 480]).astype(np.float32)
    kp2 = (rng.random((n, 2)) * [640, 480]).astype(np.float32)
    # half of the keypoints crowd a narrow band: rows from empty to long
    kp2[: n // 2, 1] = (100 + 60 * rng.random(n // 2)).astype(np.float32)
    d1 = rng.standard_normal((m, 128)).astype(np.float32)
    d2 = rng.standard_normal((n, 128)).astype(np.float32)
    return p.F, kp1, kp2, d1, d2


@pytest.mark.parametrize("m,n,eps", [(1, 40, 3.0), (255, 300, 1.0), (256, 300, 3.0),
                                     (257, 900, 20.0), (513, 700, 6.0), (70000, 60, 2.0),
                                     (262144, 24, 2.0), (262145, 24, 2.0)])
def test_rows_and_matches_at_the_edges(m, n, eps):
    import paper_2603_18401_amd as E
    torch = torch_gpu()
    F, kp1, kp2, d1, d2 = _case(m, n, m + n)
    ro, rc, _ = oracle.candidates(F, kp1, kp2, eps)
    rb, rbd, rsd = oracle.match(d1, d2, ro, rc)
    dev = torch.device("cuda:0")
    g = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    idx = E.Index([E.PairSpec(F, 640, 480, m, n)], g(kp2), eps=eps)
    k1, f1, f2 = g(kp1), g(d1), g(d2)
    for _ in range(2):  # the counters start from zero in every call
        offs, cols = idx.query(k1)
        assert np.array_equal(offs.cpu().numpy(), ro) and np.array_equal(cols.cpu().numpy(), rc)
        offs, cols, b, bd, sd = idx.query_match(k1, f1, f2)
        assert np.array_equal(offs.cpu().numpy(), ro) and np.array_equal(cols.cpu().numpy(), rc)
        assert np.array_equal(b.cpu().numpy(), rb)
        assert np.array_equal(bd.cpu().numpy().view(np.uint32), rbd.view(np.uint32))
        assert np.array_equal(sd.cpu().numpy().view(np.uint32), rsd.view(np.uint32))
    # a buffer two thirds of the size, not waited for: nothing behind it
    cap = max(1, 2 * len(rc) // 3)
    buf = torch.full((cap + 64,), -9, dtype=torch.int32, device=dev)
    offs, _ = idx.query(k1, col_indices=buf[:cap], sync=False)
    got = buf.cpu().numpy()
    assert np.array_equal(offs.cpu().numpy(), ro)
    assert np.array_equal(got[:cap], rc[:cap]) and (got[cap:] == -9).all()
    # and waited for: the size is reported
    with pytest.raises(E.EpmError) as e:
        lib = E.load_library()
        import ctypes
        nnz = ctypes.c_int64(-1)
        st = lib.epm_query_candidates(idx.handle, ctypes.c_void_p(k1.data_ptr()),
                                      ctypes.c_void_p(offs.data_ptr()),
                                      ctypes.c_void_p(buf.data_ptr()), 0, ctypes.byref(nnz),
                                      ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert nnz.value == len(rc)
        E._check(st, "epm_query_candidates")
    assert e.value.status == 3
