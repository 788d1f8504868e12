"""What the split operands of the plain convolutions (csrc/direct.hip, csrc/wgrad_direct.hip) cannot carry is computed again in
binary32: at the corners of images, where patches hang over, and at a cost that stays a small multiple of the call's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2002_00552_amd as dwm
from dwm_gpu import Runner
from test_gpu_backward import BwdRunner, WgradRunner
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


# (shape, whether the forward pass and the data gradient take the direct convolution): every shape of its workgroup
DIRECT = [
    ((32, 128, 56, 56, 256, 3, 3, 2, 1), (True, True)),    # 256 filters x 128 pixels, 128 x 128
    ((24, 117, 14, 22, 130, 3, 3, 1, 1), (True, True)),    # four waves of 64 filters share a tile
    ((1, 16, 32, 32, 16, 5, 5, 1, 2), (True, False)),      # four of 32
    ((5, 67, 35, 29, 93, 5, 5, 2, 2), (False, True)),
    ((46, 76, 8, 8, 18, 3, 3, 3, 0), (True, True)),        # eight, in pieces
    ((2, 33, 12, 230, 70, 3, 7, 1, 2), (True, True)),      # strips
    ((1, 256, 14, 14, 256, 3, 3, 1, 1), (False, True)),    # pieces
    ((2, 206, 12, 14, 284, 9, 9, 2, 4), (False, True)),    # sums in two levels
]


def _forward(shape, x, w):
    r = Runner(*shape)
    try:
        r.set_filter(w)
        return r.forward(x).astype(np.float64), dwm.dwm_plan_forward_kernel(r.plan)
    finally:
        r.close()


def _gradient(shape, dy, w):
    r = BwdRunner(*shape)
    try:
        return r.run(dy, w).astype(np.float64), dwm.dwm_bwd_data_kernel(r.plan)
    finally:
        r.close()


@pytest.mark.parametrize("corner", [0, -1])
@pytest.mark.parametrize("shape, direct", DIRECT)
def test_direct_convolution_of_a_value_in_a_corner(shape, direct, corner):
    """An infinity in the first or last pixel and channel: infinite, of the tap's sign, where a tap meets it, all else as without it
    (what a wave computes again rounds a tile's products in binary32: 1.2e-6 of the largest, as in the other tests)."""
    N, C, H, W, K, R, S, s, P = shape
    x, dy, w = _operands(shape, 43)
    at = (corner,) * 4
    for run, a, takes in ((_forward, x, direct[0]), (_gradient, dy, direct[1])):
        a[at] = 0.0
        rest, kernel = run(shape, a, w)
        assert (kernel == 2) == takes
        if not takes:
            continue
        a[at] = np.inf
        out, _ = run(shape, a, w)
        tap = np.zeros_like(out)  # the tap of w that meets it
        n, c, h, v = (corner % m for m in a.shape)
        for r in range(R):
            for q in range(S):
                if run is _forward:
                    oh, ow = h + P - r, v + P - q
                    if oh % s == 0 and ow % s == 0 and 0 <= oh // s < out.shape[2] and 0 <= ow // s < out.shape[3]:
                        tap[n, :, oh // s, ow // s] = w[:, c, r, q]
                elif 0 <= s * h + r - P < H and 0 <= s * v + q - P < W:
                    tap[n, :, s * h + r - P, s * v + q - P] = w[c, :, r, q]
        hit = tap != 0
        assert np.max(np.abs(out[~hit] - rest[~hit])) <= 1.2e-6 * np.max(np.abs(rest))
        assert np.array_equal(out[hit], np.where(tap[hit] > 0, np.inf, -np.inf))


@pytest.mark.parametrize("shape", [(64, 128, 28, 28, 128, 3, 3, 1, 1), (32, 128, 56, 56, 256, 3, 3, 2, 1), (36, 300, 28, 28, 150, 3, 3, 2, 1),
                                   (5, 67, 35, 29, 93, 5, 5, 2, 2)])
def test_time_of_a_direct_convolution_that_is_not_finite(shape):
    x, dy, w = _operands(shape, 44)
    st = torch.cuda.current_stream().cuda_stream
    f, b = Runner(*shape), BwdRunner(*shape)
    try:
        kernels = dwm.dwm_plan_forward_kernel(f.plan), dwm.dwm_bwd_data_kernel(b.plan)
        f.set_filter(w)
        f.forward(x)
        b.run(dy, w)
        calls = ((f.x, f.y, lambda: dwm.dwm_conv_forward(f.plan, f.x.data_ptr(), f.Ugw.data_ptr(), f.y.data_ptr(), st)),
                 (b.dy, b.dx, lambda: dwm.dwm_conv_backward_data(b.plan, b.dy.data_ptr(), b.Ugw.data_ptr(), b.dx.data_ptr(), st)))
        for kernel, (a, out, call) in zip(kernels, calls):
            if kernel != 2:
                continue
            plain = _us(call)
            a[tuple(n // 2 for n in a.shape)] = float("inf")
            one = _us(call)
            a.fill_(float("nan"))
            every = _us(call)
            assert bool(torch.isnan(out).any())
            print("%s: %.1f us, one infinity %.1f, NaN throughout %.1f" % (shape, plain, one, every), flush=True)
            assert max(one, every) <= 4.5 * plain
    finally:
        f.close()
        b.close()
