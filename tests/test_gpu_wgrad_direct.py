"""The filter gradient as a direct convolution on split operands, through the C ABI: every tile of its kernel, images and bands
of images as the operands' elements, patches that overhang, pieces with and without units, against FP64 and the transforms."""
import numpy as np
import pytest
import torch

import oracle
import paper_2002_00552_amd as dwm
from test_gpu_backward import WSHAPES

pytestmark = pytest.mark.gpu

# (N, C, H, W, K, R, S, stride, pad): tiles of 32 and 64 filters x 32, 64, 96 and 160 columns, each with bands and without
SHAPES = [
    (10, 2, 30, 8, 49, 1, 1, 3, 0), (14, 5, 9, 8, 44, 1, 1, 3, 0), (49, 9, 35, 24, 103, 2, 2, 3, 1), (36, 5, 13, 11, 131, 7, 7, 3, 3),
    (19, 23, 8, 36, 47, 7, 7, 3, 3), (14, 22, 25, 13, 45, 7, 7, 3, 3), (37, 7, 13, 16, 66, 4, 4, 1, 2), (43, 15, 9, 10, 70, 7, 7, 2, 3),
    (30, 1, 30, 32, 86, 1, 1, 1, 0), (48, 1, 36, 30, 136, 1, 1, 2, 0), (60, 4, 31, 20, 42, 3, 3, 1, 1), (65, 10, 12, 32, 40, 2, 2, 1, 1),
    (20, 5, 20, 33, 110, 4, 4, 1, 2), (72, 19, 18, 14, 65, 2, 2, 1, 1), (51, 8, 29, 19, 68, 5, 5, 1, 2), (70, 15, 36, 18, 101, 3, 3, 1, 1),
    (1, 70, 8, 8, 34, 3, 3, 1, 1),     # one unit: dw is written without a second launch
    (3, 9, 6, 7, 7, 2, 5, 3, 4),       # R != S, padding of nearly the kernel, fewer units than XCDs
    (1, 2, 12, 12, 3, 12, 12, 1, 0),   # one output pixel
    (5, 67, 35, 29, 93, 5, 5, 2, 2),   # nothing a multiple of anything
]


def _run(shape, x, dy, path=-1):
    N, C, H, W, K, R, S, s, P = shape
    p = dwm.dwm_bwd_filter_plan_create(*shape)
    try:
        dwm.dwm_bwd_filter_set_variant(p, "path", path)
        assert (dwm.dwm_bwd_filter_kernel(p) == 2) == (path < 0), shape
        ws = torch.full((dwm.dwm_bwd_filter_workspace_bytes(p) // 4,), float("nan"), device="cuda")
        dwm.dwm_bwd_filter_set_workspace(p, ws.data_ptr(), ws.numel() * 4)
        with pytest.raises(dwm.DwmError):
            dwm.dwm_bwd_filter_set_variant(p, "path", path)
        dw = torch.full((K, C, R, S), float("nan"), device="cuda")
        xd, dyd = torch.from_numpy(x).cuda(), torch.from_numpy(dy).cuda()
        dwm.dwm_conv_backward_filter(p, xd.data_ptr(), dyd.data_ptr(), dw.data_ptr(), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        return dw.cpu().numpy()
    finally:
        dwm.dwm_bwd_filter_plan_destroy(p)


def _data(shape, seed):
    N, C, H, W, K, R, S, s, P = shape
    rng = np.random.default_rng(seed)
    return (rng.uniform(-1, 1, (N, C, H, W)).astype(np.float32),
            rng.standard_normal((N, K, (H + 2 * P - R) // s + 1, (W + 2 * P - S) // s + 1)).astype(np.float32))


@pytest.mark.parametrize("shape", SHAPES)
def test_filter_gradient(shape):
    """Every tap within 2e-6 of the largest, in the 2-norm no further from FP64 than the transforms, the same bits again."""
    N, C, H, W, K, R, S, s, P = shape
    x, dy = _data(shape, 1)
    dw = _run(shape, x, dy)
    ref = oracle.backward_filter_f64(x, dy, (K, C, R, S), s, P)
    assert np.all(np.isfinite(dw))
    assert np.max(np.abs(dw - ref)) <= 2e-6 * np.max(np.abs(ref))
    # (each tap's own rounding to binary32, 2^-24 of it at most, is common to both)
    assert np.linalg.norm(dw - ref) <= np.linalg.norm(_run(shape, x, dy, 0) - ref) + 2.0 ** -24 * np.linalg.norm(ref)
    assert np.array_equal(_run(shape, x, dy), dw)


@pytest.mark.parametrize("shape", WSHAPES)
def test_the_transforms_when_asked_for(shape):
    N, C, H, W, K, R, S, s, P = shape
    x, dy = _data(shape, 2)
    dw = _run(shape, x, dy, 0)
    ref = oracle.backward_filter_f64(x, dy, (K, C, R, S), s, P)
    assert np.max(np.abs(dw - ref)) <= 4e-6 * np.max(np.abs(ref))


@pytest.mark.parametrize("how", [(1e-34, 1), (1e-38, 1), (1e-38, 1e30), (1e-30, 3e34)])
@pytest.mark.parametrize("where", ["x", "dy"])
def test_small_and_large_operands(where, how):
    """As at any other scale, and what the sums' last rounding near the end of the range adds."""
    shape = SHAPES[-1]
    N, C, H, W, K, R, S, s, P = shape
    x, dy = _data(shape, 3)
    a, b = (x, dy) if where == "x" else (dy, x)
    a *= np.float32(how[0])
    b *= np.float32(how[1])
    dw = _run(shape, x, dy)
    ref = oracle.backward_filter_f64(x, dy, (K, C, R, S), s, P)
    scale = np.max(np.abs(ref))
    assert np.linalg.norm((dw - ref) / scale) <= 1e-6 * np.linalg.norm(ref / scale) + np.sqrt(dw.size) * 2.0 ** -149 / scale


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38, -1e34])
@pytest.mark.parametrize("where", ["x", "dy"])
@pytest.mark.parametrize("shape", [SHAPES[2], SHAPES[11], SHAPES[16]])
def test_values_that_the_split_cannot_carry(shape, where, value):
    """One such value: the taps that it reaches are what binary32 makes of it, all others as without it."""
    N, C, H, W, K, R, S, s, P = shape
    x, dy = _data(shape, 4)
    a, other = (x, dy) if where == "x" else (dy, x)
    other *= np.float32(1e-3)
    at = (N // 2, 1, a.shape[2] // 2, a.shape[3] // 2)
    a[at] = 0.0
    rest = oracle.backward_filter_f64(x, dy, (K, C, R, S), s, P)
    one = np.zeros_like(a)
    one[at] = 1.0
    part = oracle.backward_filter_f64(one if where == "x" else x, dy if where == "x" else one, (K, C, R, S), s, P)
    a[at] = value
    dw = _run(shape, x, dy).astype(np.float64)
    hit = part != 0
    far = ~hit
    (far[:, 1] if where == "x" else far[1])[...] = False  # (there an infinity meets the zeros around x)
    assert hit.any() and far.any()
    assert np.max(np.abs(dw[far] - rest[far])) <= 2e-6 * np.max(np.abs(rest))
    if np.isnan(value):
        assert np.all(np.isnan(dw[hit]))
    elif np.isinf(value):
        assert np.array_equal(dw[hit], np.where(part[hit] > 0, value, -value))
    else:
        assert np.max(np.abs(dw[hit] - part[hit] * value)) <= 2e-6 * np.max(np.abs(part * value))
