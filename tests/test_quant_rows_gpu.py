"""epm_quantize and epm_rounding_error on rows of 128: the kernels for aligned
arrays against the ones for any width and alignment, bit for bit in the codes
and scales, at row counts around a workgroup's 32 rows."""

import ctypes

import numpy as np
import pytest

import synth
from tests.gpu_util import torch_gpu

pytestmark = pytest.mark.gpu


def _rows(n):
    rng = np.random.default_rng(n)
    x = rng.normal(size=(n, 128)) * 10.0 ** rng.uniform(-6, 4, (n, 1))
    x[rng.random((n, 128)) < 0.02] = -0.0
    x[0, :6] = [448.0, np.inf, -np.inf, np.nan, 1e-42, -448.0]
    return x.astype(np.float32)


def _call(torch, x, fmt, shift):
    """Codes, scales and errors with every array `shift` elements into its buffer."""
    import paper_2603_18401_amd as E
    lib = E.load_library()
    n = len(x)
    p = lambda t, k: ctypes.c_void_p(t.data_ptr() + k * t.element_size())  # noqa: E731
    s = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    src = torch.zeros(n * 128 + 8, device="cuda:0")
    src[shift:shift + n * 128] = torch.from_numpy(x.reshape(-1)).to("cuda:0")
    dst = torch.zeros(n * 128 + 8, device="cuda:0",
                      dtype=torch.int16 if fmt == 1 else torch.uint8)
    scale = torch.ones(n + 1, device="cuda:0")
    err = torch.full((n + 1,), -7.0, device="cuda:0")
    assert lib.epm_quantize(p(src, shift), n, 128, fmt, p(dst, shift), p(scale, 0), s) == 0
    codes = dst.cpu().numpy()
    assert not codes[:shift].any() and not codes[shift + n * 128:].any()
    if fmt == 2:
        dst[shift + 128 * (n - 1)] = 0x7F  # no code of epm_quantize, read as 480
        dst[shift + 128 * (n - 1) + 1] = 0xFF
    assert lib.epm_rounding_error(p(src, shift), n, 128, fmt, p(dst, shift), p(scale, 0),
                                  p(err, 0), s) == 0
    e = err.cpu().numpy()
    assert e[n] == -7.0
    return codes[shift:shift + n * 128], scale.cpu().numpy(), e[:n]


@pytest.mark.parametrize("fmt", [1, 2], ids=["bf16", "fp8"])
@pytest.mark.parametrize("n", [1, 7, 31, 32, 33, 65])
def test_aligned_rows_equal_the_general_kernels(fmt, n):
    torch = torch_gpu()
    x = _rows(n)
    codes, scale, err = _call(torch, x, fmt, 0)
    c1, s1, e1 = _call(torch, x, fmt, 1)
    assert np.array_equal(codes, c1) and np.array_equal(scale, s1)
    # the same FP64 terms added in another order, rounded to float once
    fine = np.isfinite(e1)
    assert np.array_equal(fine, np.isfinite(err))
    assert np.all(np.abs(err[fine] - e1[fine]) <= 2.0 ** -22 * e1[fine])
    if fmt == 1:
        ok = ~np.isnan(x)
        assert np.array_equal(codes.view(np.uint16).reshape(n, 128)[ok], synth.f32_to_bf16(x)[ok])
