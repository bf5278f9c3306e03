"""Inference of the tolerance network row by row: a keypoint's tolerance is
the same whatever the other keypoints of the call are."""

import numpy as np
import pytest

import synth
from tests.gpu_util import torch_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("row", [0, 37, 63, 64, 150])
def test_one_bad_row_leaves_the_others_alone(row):
    """The bad row takes the plain evaluation, the others the matrix one."""
    from paper_2603_18401_amd import learned_eps as L
    torch = torch_gpu()
    dev = torch.device("cuda:0")
    theta = synth.mlp_init(7).astype(np.float32)
    theta[-65:-1] *= 8.0
    rng = np.random.default_rng(2)
    X = rng.uniform([1, 0, -3.1, -1, -0.7, 0], [12, 1, 3.1, 1, 0.7, 6.9], (4 * 64 + 5, 6))
    X = X.astype(np.float32)
    Y = X.copy()
    Y[row, 2] = np.nan
    params = torch.from_numpy(theta).to(dev)
    a, b = (L.infer(torch.from_numpy(v).to(dev), params).cpu().numpy() for v in (X, Y))
    others = np.arange(len(X)) != row
    assert np.array_equal(a[others].view(np.uint32), b[others].view(np.uint32))
