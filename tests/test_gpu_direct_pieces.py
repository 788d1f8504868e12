"""Direct convolutions (csrc/direct.hip) whose tiles are shared by several workgroups, each with a range of the channels: layers
of few tiles and many channels, above all as data gradients at stride 1.  Against the FP64 oracle, with the bar of the direct
convolution's other tests (1e-6 of the largest output), which a sum of 2 to 16 pieces in binary32 does not change."""
import numpy as np
import pytest
import torch

import oracle
import paper_2002_00552_amd as dwm
from dwm_gpu import Runner
from test_gpu_backward import BwdRunner

pytestmark = pytest.mark.gpu

FORWARD = [  # N, C, H, W, K, R, S, stride, pad
    (16, 256, 14, 14, 256, 3, 3, 1, 1),
    (118, 122, 14, 14, 89, 4, 4, 2, 2),
]
GRADIENT = [
    (1, 256, 14, 14, 256, 3, 3, 1, 1),   # sixteen pieces of one chunk
    (4, 255, 14, 14, 250, 3, 3, 1, 1),   # eight pieces of two blocks of filters, channels past the last
    (1, 140, 33, 31, 150, 7, 7, 1, 3),   # three
    (3, 79, 13, 13, 233, 11, 11, 1, 5),  # eight, the last one's chunk shorter
    (8, 38, 27, 27, 224, 3, 3, 1, 1),
    (2, 190, 20, 18, 100, 5, 3, 1, 0),   # no padding: dy's patches reach past it
]


def _rand(shape, seed):
    N, C, H, W, K, R, S, s, P = shape
    rng = np.random.default_rng(seed)
    x = rng.uniform(-1, 1, (N, C, H, W)).astype(np.float32)
    w = (rng.standard_normal((K, C, R, S)) * np.sqrt(2.0 / (C * R * S))).astype(np.float32)
    dy = rng.standard_normal((N, K, (H + 2 * P - R) // s + 1, (W + 2 * P - S) // s + 1)).astype(np.float32)
    return x, w, dy


def _gradient(shape, dy, w, path=-1):
    r = BwdRunner(*shape, path=path)
    try:
        dx = r.run(dy, w)
        kernel = dwm.dwm_bwd_data_kernel(r.plan)
        used = ~np.isnan(r.ws.cpu().numpy())
        assert np.array_equal(r.run(dy, w), dx, equal_nan=True)
        return dx, kernel, used
    finally:
        r.close()


@pytest.mark.parametrize("shape", FORWARD)
def test_forward_in_pieces(shape):
    """The outputs, in place of the contraction's partial ones, leave V alone; and the same bits from the static scratch."""
    x, w, _ = _rand(shape, 21)
    r = Runner(*shape)
    try:
        r.set_filter(w)
        y = r.forward(x)
        assert dwm.dwm_plan_forward_kernel(r.plan) == 2
        used = ~np.isnan(r.ws.cpu().numpy())
        v = r.info.Vblock * (r.info.Tpad // 64)
        assert used[v:].any() and not used[:v].any()
        assert np.array_equal(r.forward(x), y)
        if dwm.dwm_plan_workspace_bytes(r.plan) <= dwm.dwm_static_scratch_bytes():
            r.y.fill_(float("nan"))
            dwm.dwm_conv_forward_static(r.plan, r.x.data_ptr(), r.Ugw.data_ptr(), r.y.data_ptr(), r.stream())
            torch.cuda.synchronize()
            assert np.array_equal(r.y.cpu().numpy(), y)
    finally:
        r.close()
    idx = np.random.default_rng(22).choice(y.size, min(y.size, 4000), replace=False)
    ref = oracle.direct_f64_at(x, w, shape[7], shape[8], idx)
    assert np.all(np.isfinite(y))
    assert np.max(np.abs(y.ravel()[idx] - ref)) <= 1e-6 * np.max(np.abs(ref))


@pytest.mark.parametrize("shape", GRADIENT)
def test_data_gradient_in_pieces(shape):
    N, C, H, W, K, R, S, s, P = shape
    _, w, dy = _rand(shape, 23)
    dx, kernel, used = _gradient(shape, dy, w)
    assert kernel == 2 and used.any()
    ref = oracle.backward_data_f64(dy, w, (N, C, H, W), s, P)
    assert np.max(np.abs(dx - ref)) <= 1e-6 * np.max(np.abs(ref))
    z, kernel, _ = _gradient(shape, dy, w, 0)  # the path that it replaces: every copy of the filter is there
    assert kernel == 0
    assert np.linalg.norm(dx - ref) <= 1.05 * np.linalg.norm(z - ref)


@pytest.mark.parametrize("value", [np.inf, np.nan, 3.4e38])
def test_a_value_that_the_split_cannot_carry(value):
    """It lies in one piece's channels: that piece's sums are computed again, the others' are not."""
    shape = GRADIENT[1]
    N, C, H, W, K, R, S, s, P = shape
    _, w, dy = _rand(shape, 24)
    w *= np.float32(1e-3)
    rest, _, _ = _gradient(shape, dy, w)
    at = (N // 2, K - 1, H // 2, W // 2)
    dy[at] = value
    dx, _, _ = _gradient(shape, dy, w)
    tap = np.zeros_like(dx)
    for r in range(R):
        for q in range(S):
            tap[at[0], :, at[2] - P + r, at[3] - P + q] = w[at[1], :, r, q]
    hit = tap != 0
    # (what a piece computes again rounds 288 products in binary32: sqrt(288) half roundings of the largest sum, 1.1e-6)
    assert np.max(np.abs(dx[~hit] - rest[~hit])) <= 1.2e-6 * np.max(np.abs(rest))
    if np.isnan(value):
        assert np.all(np.isnan(dx[hit]))
    else:
        expect = tap[hit].astype(np.float64) * value
        assert np.array_equal(dx[hit], expect) if np.isinf(value) else np.all(np.abs(dx[hit] - expect) <= 1e-6 * np.abs(expect))
