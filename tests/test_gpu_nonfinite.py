"""What the split operands of the plain convolutions (csrc/direct.hip, csrc/wgrad_direct.hip) cannot carry is computed again in
binary32: at the corners of images, where patches hang over, and at a cost that stays a small multiple of the call's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2002_00552_amd as dwm
from test_gpu_backward import WgradRunner
from test_gpu_wgrad_direct import SHAPES as WGRAD_SHAPES

pytestmark = pytest.mark.gpu


def _operands(shape, seed):
    N, C, H, W, K, R, S, s, P = shape
    rng = np.random.default_rng(seed)
    OH, OW = (H + 2 * P - R) // s + 1, (W + 2 * P - S) // s + 1
    return (rng.uniform(-1, 1, (N, C, H, W)).astype(np.float32), rng.standard_normal((N, K, OH, OW)).astype(np.float32),
            (rng.standard_normal((K, C, R, S)) * np.sqrt(2.0 / (C * R * S))).astype(np.float32))


def _us(call):
    """The least time of a call among eight."""
    best = 1e30
    for _ in range(8):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best


@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("where, corner", [("x", 0), ("x", -1), ("dy", 0), ("dy", -1)])
@pytest.mark.parametrize("shape", WGRAD_SHAPES)
def test_filter_gradient_of_a_value_in_a_corner(shape, where, corner, value):
    """The first or last pixel of the first or last image: the taps that it meets are infinite, of the definition's sign, or NaN
    (several units' sums of an infinity among them), all others are as without it."""
    N, C, H, W, K, R, S, s, P = shape
    x, dy, _ = _operands(shape, 41)
    a = x if where == "x" else dy
    at = (corner, corner, corner, corner)
    a[at] = 0.0
    rest = oracle.backward_filter_f64(x, dy, (K, C, R, S), s, P)
    one = np.zeros_like(a)
    one[at] = 1.0
    part = oracle.backward_filter_f64(one if where == "x" else x, dy if where == "x" else one, (K, C, R, S), s, P)
    a[at] = value
    r = WgradRunner(*shape)
    try:
        assert dwm.dwm_bwd_filter_kernel(r.plan) == 2
        dw = r.run(x, dy).astype(np.float64)
    finally:
        r.close()
    hit = part != 0
    far = ~hit
    if where == "dy":
        far[corner] = False  # (there the value meets the zeros around x)
    assert np.max(np.abs(dw[far] - rest[far]), initial=0.0) <= 2e-6 * np.max(np.abs(rest))
    assert np.all(np.isnan(dw[hit])) if np.isnan(value) else np.array_equal(dw[hit], np.where(part[hit] > 0, value, -value))


@pytest.mark.parametrize("shape", [(64, 3, 224, 224, 64, 7, 7, 2, 3), (5, 67, 35, 29, 93, 5, 5, 2, 2), (10, 3, 151, 147, 31, 5, 5, 2, 2)])
def test_time_of_a_filter_gradient_that_is_not_finite(shape):
    x, dy, _ = _operands(shape, 42)
    r = WgradRunner(*shape)
    try:
        assert dwm.dwm_bwd_filter_kernel(r.plan) == 2
        r.run(x, dy)
        xd, dyd = torch.from_numpy(x).cuda(), torch.from_numpy(dy).cuda()
        call = lambda: dwm.dwm_conv_backward_filter(r.plan, xd.data_ptr(), dyd.data_ptr(), r.dw.data_ptr(), torch.cuda.current_stream().cuda_stream)
        plain = _us(call)
        xd[tuple(n // 2 for n in xd.shape)] = float("inf")
        one = _us(call)
        dyd.fill_(float("nan"))
        every = _us(call)
        assert bool(torch.isnan(r.dw).all())
    finally:
        r.close()
    print("%s: %.1f us, one infinity %.1f, NaN throughout %.1f" % (shape, plain, one, every))
    assert max(one, every) <= 4 * plain
