"""Keypoints outside their image are legal: pairs whose keypoints reach two and
four times as far as the image size that is given, with the epipole far away,
at infinity and beside the image.  Candidates and matches against the oracle;
the counter of scanned records tells whether the position codes still resolve
the angles beyond the image."""

import numpy as np
import pytest

import oracle
from tests.gpu_util import torch_gpu

pytestmark = pytest.mark.gpu

W, H = 6048, 4032


@pytest.mark.parametrize("scale", [1.0, 0.5, 0.25])
@pytest.mark.parametrize("e", [(-20000.0, 3000.0, 1.0), (1.0, 0.0, 0.0), (-1500.0, 2000.0, 1.0)],
                         ids=["far", "infinite", "beside"])
def test_keypoints_beyond_the_image(e, scale):
    import paper_2603_18401_amd as E
    torch = torch_gpu()
    dev = torch.device("cuda:0")
    g = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    rng = np.random.default_rng(int(100 * scale))
    n = 4000
    e = np.array(e) / np.linalg.norm(e)
    F = np.array([[0, -e[2], e[1]], [e[2], 0, -e[0]], [-e[1], e[0], 0]])
    kp1, kp2 = ((rng.random((n, 2)) * [W, H]).astype(np.float32) for _ in range(2))
    d1, d2 = (rng.standard_normal((n, 128)).astype(np.float32) for _ in range(2))
    eps = 2.0
    ro, rc, _ = oracle.candidates(F, kp1, kp2, eps)
    want = oracle.match(d1, d2, ro, rc)
    idx = E.Index([E.PairSpec(F, int(W * scale), int(H * scale), n, n)], g(kp2), eps=eps)
    offs, cols, *got = idx.query_match(g(kp1), g(d1), g(d2))
    assert np.array_equal(offs.cpu().numpy(), ro) and np.array_equal(cols.cpu().numpy(), rc)
    for a, b in zip(got, want):
        assert np.array_equal(a.cpu().numpy().view(np.uint32), b.view(np.uint32))
    # the queries in the order of their lines, 16 at a time: the records whose
    # tolerance meets the span between the first and the last of them
    if e[2] == 0:
        p1, p2, half = kp1[:, 1].astype(float), kp2[:, 1].astype(float), eps
    else:
        c = e[:2] / e[2]
        p1, p2 = (np.arctan2(*(k.astype(float) - c).T[::-1]) for k in (kp1, kp2))
        half = np.arcsin(eps / np.hypot(*(kp2.astype(float) - c).T))
    p1 = np.sort(p1)
    lo, hi = np.sort(p2 - half), np.sort(p2 + half)
    at = np.concatenate([np.arange(0, n, 16), [n]])
    meets = (np.searchsorted(lo, p1[at[1:] - 1], "right") - np.searchsorted(hi, p1[at[:-1]], "left"))
    # parts of groups that cross from one workgroup to the next may stay unsorted
    assert idx.stats()["records_scanned"] <= 1.5 * int((np.diff(at) * meets).sum())
