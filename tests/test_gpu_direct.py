"""The direct convolution on the bfloat16 matrix cores (three-way split operands, no transforms) through the C ABI: forward and
the data gradient in one launch, at the edges of its tiles, chunks, groups of channels and strips, against FP64 and against
the method's transforms."""
import numpy as np
import pytest
import torch

import oracle
import paper_2002_00552_amd as dwm
from dwm_gpu import Runner
from test_gpu_backward import BwdRunner

pytestmark = pytest.mark.gpu

# (N, C, H, W, K, R, S, stride, pad): what the planner gives to it (asserted), between them every shape of its workgroup
BWD = [
    (5, 67, 35, 29, 93, 5, 5, 2, 2),     # nothing a multiple of anything
    (1, 17, 9, 8, 200, 3, 3, 2, 1),      # a handful of outputs, many chunks of channels
    (46, 76, 8, 8, 18, 3, 3, 3, 0),      # one tap a phase, tiles that span images
    (1, 18, 23, 19, 70, 5, 5, 4, 2),     # sixteen phases
    (1, 65, 31, 30, 130, 6, 3, 2, 0),    # R != S, filters one past a tile, rows and columns that no tap reaches
    (3, 24, 18, 6, 100, 3, 3, 2, 1),     # a narrow image
    (2, 33, 3, 230, 17, 3, 11, 2, 5),    # wide rows: strips
    (4, 35, 9, 11, 7, 2, 2, 3, 1),       # stride above the kernel: phases without a tap; fewer than eight channels of dy
    (24, 130, 36, 36, 71, 2, 2, 2, 1),   # tiles of 128 filters
    (36, 300, 28, 28, 150, 3, 3, 2, 1),  # several rounds of the chip
]

# the same for the forward pass; "1": the single-kernel path is what it would be otherwise
FWD = [
    ((1, 16, 32, 32, 16, 5, 5, 1, 2), 1),       # one small image
    ((3, 29, 49, 44, 23, 3, 3, 3, 0), 0),       # three phases of columns, odd rows past the last window
    ((10, 45, 28, 27, 78, 3, 3, 1, 0), 1),      # three slices of filters
    ((105, 28, 32, 36, 62, 2, 2, 1, 1), 1),     # pixels of one tile in two images
    ((1, 65, 7, 9, 33, 1, 1, 1, 0), 0),         # one tap, a channel past a group, a filter past a tile
    ((2, 33, 12, 230, 70, 3, 7, 1, 2), 1),      # wide rows: strips; R != S
    ((3, 17, 25, 31, 300, 4, 4, 2, 3), 0),      # padding of a whole kernel but one tap
    ((200, 18, 5, 5, 33, 3, 3, 1, 0), 0),       # tiles of several images
    ((16, 128, 56, 55, 256, 3, 3, 2, 1), 0),    # tiles of 256 filters
    ((16, 96, 40, 40, 128, 2, 3, 1, 1), 0),     # many workgroups
]


def _data(shape, seed):
    N, C, H, W, K, R, S, s, P = shape
    rng = np.random.default_rng(seed)
    dy = rng.standard_normal((N, K, (H + 2 * P - R) // s + 1, (W + 2 * P - S) // s + 1)).astype(np.float32)
    return dy, (rng.standard_normal((K, C, R, S)) * np.sqrt(2.0 / (C * R * S))).astype(np.float32)


def _grad(shape, dy, w, path=-1):
    r = BwdRunner(*shape, path=path)
    try:
        assert dwm.dwm_bwd_data_kernel(r.plan) == (2 if path < 0 else path)
        r.dx.fill_(float("nan"))
        return r.run(dy, w)
    finally:
        r.close()


@pytest.mark.parametrize("shape", BWD)
def test_strided_data_gradient(shape):
    """Every pixel within 1e-6 of the largest (5e-8 to 3e-7 measured in the 2-norm), in the 2-norm no further from FP64 than the
    sub-convolutions by the method's transforms; and the same bits again."""
    N, C, H, W, K, R, S, s, P = shape
    dy, w = _data(shape, 3)
    dx = _grad(shape, dy, w)
    ref = oracle.backward_data_f64(dy, w, (N, C, H, W), s, P)
    assert np.all(np.isfinite(dx))
    assert np.max(np.abs(dx - ref)) <= 1e-6 * np.max(np.abs(ref)), shape
    assert np.linalg.norm(dx - ref) <= 1.05 * np.linalg.norm(_grad(shape, dy, w, 0) - ref)
    assert np.array_equal(_grad(shape, dy, w), dx)


@pytest.mark.parametrize("how", [(1e-34, 1, 1), (1e-38, 1, 1), (1e-38, 1e30, 1), (1e-36, 1e34, 2), (1e-30, 3e37, 1)])
@pytest.mark.parametrize("where", ["dy", "w"])
def test_small_and_large_operands(where, how):
    """One operand far below 1, all of it or every other channel of dy, the other ordinary or as much larger (3e37: past what
    the split carries): in the 2-norm as at any other scale, and what the sums' last binary32 rounding near the end of the range adds."""
    shape = BWD[0]
    N, C, H, W, K, R, S, s, P = shape
    dy, w = _data(shape, 4)
    a, b = (dy, w.transpose(1, 0, 2, 3)) if where == "dy" else (w.transpose(1, 0, 2, 3), dy)
    a[:, ::how[2]] *= np.float32(how[0])
    b[:, ::how[2]] *= np.float32(how[1])
    dx = _grad(shape, dy, w)
    ref = oracle.backward_data_f64(dy, w, (N, C, H, W), s, P)
    scale = np.max(np.abs(ref))
    assert np.linalg.norm((dx - ref) / scale) <= 1e-6 * np.linalg.norm(ref / scale) + np.sqrt(dx.size) * 2.0 ** -149 / scale


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38, -1e34])
@pytest.mark.parametrize("where", ["dy", "w"])
@pytest.mark.parametrize("shape", [BWD[0], BWD[2], BWD[6]])
def test_values_that_the_split_cannot_carry(shape, where, value):
    """One such value: infinite, of the definition's sign, or NaN wherever it reaches, and all other pixels as without it (of an
    infinite or NaN tap's own channel of dx the others may be NaN, where the tap meets the zeros around dy)."""
    N, C, H, W, K, R, S, s, P = shape
    dy, w = _data(shape, 5)
    (w if where == "dy" else dy)[...] *= np.float32(1e-3)
    a = dy if where == "dy" else w
    a[tuple(n // 2 for n in a.shape)] = value
    dx = _grad(shape, dy, w).astype(np.float64)
    if np.isfinite(value):
        ref = oracle.backward_data_f64(dy, w, (N, C, H, W), s, P)
        assert np.all(np.isfinite(dx))
        assert np.max(np.abs(dx - ref)) <= 1e-6 * np.max(np.abs(ref))
        small = np.abs(ref) < 1e3
        assert np.max(np.abs(dx - ref)[small]) <= 1e-5 * np.max(np.abs(ref[small]))
        return
    d64, w64 = torch.from_numpy(dy).double(), torch.from_numpy(w).double()
    a64 = d64 if where == "dy" else w64
    a64[tuple(n // 2 for n in a.shape)] = 0.0
    rest = oracle.backward_data_f64(d64.numpy().astype(np.float32), w64.numpy().astype(np.float32), (N, C, H, W), s, P)
    one = np.zeros_like(a)
    one[tuple(n // 2 for n in a.shape)] = 1.0
    sign = oracle.backward_data_f64(one if where == "dy" else dy, w if where == "dy" else one, (N, C, H, W), s, P)
    hit = sign != 0.0
    assert hit.any() and not hit.all()
    far = ~hit
    if where == "w":
        far[:, C // 2] = False
    assert np.max(np.abs(dx[far] - rest[far])) <= 1e-6 * np.max(np.abs(rest))
    if np.isnan(value):
        assert np.all(np.isnan(dx[hit]))
    else:
        assert np.array_equal(dx[hit], np.where(sign[hit] > 0, value, -value))


def _forward(shape, x, w, variants=None):
    r = Runner(*shape, variants=variants)
    try:
        r.Ugw.fill_(float("nan"))
        r.set_filter(w)
        y = r.forward(x)
        assert bool(torch.isfinite(r.Ugw).all()) or not np.all(np.isfinite(w))  # every copy, and what lies between them
        return y, dwm.dwm_plan_forward_kernel(r.plan)
    finally:
        r.close()


def _layer(shape, seed):
    N, C, H, W, K, R, S, s, P = shape
    rng = np.random.default_rng(seed)
    return (rng.uniform(-1, 1, (N, C, H, W)).astype(np.float32),
            (rng.standard_normal((K, C, R, S)) * np.sqrt(2.0 / (C * R * S))).astype(np.float32))


@pytest.mark.parametrize("shape, other", FWD)
def test_forward(shape, other):
    """Sampled outputs within 1e-6 of the largest, in the 2-norm no further from FP64 than the transforms' path; the same bits
    again, and without a workspace; and the paths that a variant asks for run."""
    x, w = _layer(shape, 6)
    y, kernel = _forward(shape, x, w)
    assert kernel == 2
    idx = np.random.default_rng(7).choice(y.size, min(y.size, 6000), replace=False)
    ref = oracle.direct_f64_at(x, w, shape[7], shape[8], idx)
    err = y.ravel()[idx] - ref
    assert np.all(np.isfinite(y))
    assert np.max(np.abs(err)) <= 1e-6 * np.max(np.abs(ref))
    for variants in [{"forward": 0}, {"input": 0}] + ([{"forward": 1}] if other else []):
        z, kernel = _forward(shape, x, w, variants)
        assert kernel == (other if variants != {"forward": 0} else 0)
        assert np.max(np.abs(z.ravel()[idx] - ref)) <= 2e-6 * np.max(np.abs(ref))
        assert np.linalg.norm(err) <= 1.05 * np.linalg.norm(z.ravel()[idx] - ref)
    r = Runner(*shape)
    try:
        r.set_filter(w)
        assert np.array_equal(r.forward(x), y)
        if other or dwm.dwm_plan_workspace_bytes(r.plan) <= dwm.dwm_static_scratch_bytes():
            r.y.fill_(float("nan"))
            dwm.dwm_conv_forward_static(r.plan, r.x.data_ptr(), r.Ugw.data_ptr(), r.y.data_ptr(), r.stream())
            torch.cuda.synchronize()
            assert np.array_equal(r.y.cpu().numpy(), y)
        else:
            with pytest.raises(dwm.DwmError):
                dwm.dwm_conv_forward_static(r.plan, r.x.data_ptr(), r.Ugw.data_ptr(), r.y.data_ptr(), r.stream())
    finally:
        r.close()


@pytest.mark.parametrize("shape", [(2, 24, 14, 14, 40, 7, 7, 1, 3), (5, 19, 17, 23, 66, 3, 5, 1, 0), (3, 40, 9, 9, 21, 3, 3, 1, 4)])
def test_data_gradient_at_stride_1(shape):
    N, C, H, W, K, R, S, s, P = shape
    dy, w = _data(shape, 8)
    dx = _grad(shape, dy, w)
    ref = oracle.backward_data_f64(dy, w, (N, C, H, W), s, P)
    assert np.max(np.abs(dx - ref)) <= 1e-6 * np.max(np.abs(ref)), shape
    assert np.linalg.norm(dx - ref) <= 1.05 * np.linalg.norm(_grad(shape, dy, w, 0) - ref)


@pytest.mark.parametrize("value", [np.inf, np.nan, -3.4e38])
def test_forward_of_values_that_the_split_cannot_carry(value):
    """One such value in x: the outputs that its window reaches are infinite, NaN or large as the definition says, all others as
    without it: where a wave's other outputs are computed again, to the rounding of 405 products of 1e-3 added in binary32, whose
    sums lie below the largest output (sqrt(405) half roundings of it, 1.2e-6)."""
    shape = FWD[2][0]
    N, C, H, W, K, R, S, s, P = shape
    x, w = _layer(shape, 9)
    w *= np.float32(1e-3)
    rest, _ = _forward(shape, x, w)
    at = (N // 2, C // 2, H // 2, W // 2)
    x[at] = value
    y, _ = _forward(shape, x, w)
    tap = np.zeros_like(y)  # the tap of w that meets it
    for r in range(R):
        for q in range(S):
            tap[at[0], :, at[2] - r, at[3] - q] = w[:, at[1], r, q]
    hit = tap != 0
    assert np.max(np.abs(y[~hit] - rest[~hit])) <= 1.2e-6 * np.max(np.abs(rest))
    assert np.mean(y[~hit] != rest[~hit]) < 0.01
    if np.isnan(value):
        assert np.all(np.isnan(y[hit]))
    else:
        expect = tap[hit].astype(np.float64) * value
        assert np.array_equal(y[hit], expect) if np.isinf(value) else np.all(np.abs(y[hit] - expect) <= 1e-6 * np.abs(expect))
