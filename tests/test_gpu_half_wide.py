"""GPU parity tests of the 16-bit kernel for layers with many input channels (dwm_f16_* / dwm_bf16_* conv_forward, "wide"),
through the C ABI against the FP64 oracle with 16-bit storage.  Bars: those of the two formats' own suites.  The layers sit
where the kernel can go wrong: chunks of 16 channels, blocks of 128 filters and 64 tiles not filled, tiles of several
images in a block, every class of parts, odd numbers of stages, channels cut into pieces, shares of pixels that need more than
one round, images narrower than the kernel."""
import numpy as np
import pytest
import torch

import dwm_workloads as wl
import oracle
import paper_2002_00552_amd as dwm
import test_gpu_bf16 as tb
import test_gpu_half as th

pytestmark = pytest.mark.gpu

SHAPES = [  # N, C, H, W, K, R, S, stride, pad
    (1, 16, 8, 8, 16, 3, 3, 1, 1),       # one stage
    (1, 17, 10, 10, 18, 1, 5, 1, 0),     # two chunks, the second one channel; (1,3) and (1,2) parts
    (2, 40, 12, 12, 9, 1, 1, 1, 0),      # 1x1 parts only
    (3, 40, 13, 18, 70, 3, 3, 2, 1),     # classes (2,2) (2,1) (1,2) (1,1), partial chunk
    (1, 64, 14, 14, 129, 7, 7, 1, 3),    # nine parts, one filter over a block
    (2, 48, 12, 12, 33, 7, 3, 3, 1),     # stride 3, R != S
    (5, 35, 7, 10, 130, 4, 4, 1, 1),     # (3,3) (3,1) ..., five images in few blocks
    (9, 24, 4, 6, 40, 5, 5, 1, 2),       # six tiles an image: all nine images in one block
    (1, 19, 40, 40, 20, 11, 11, 1, 5),   # sixteen parts
    (2, 100, 21, 16, 96, 6, 6, 2, 2),    # seven chunks
    (1, 256, 14, 14, 256, 3, 3, 1, 1),   # one stage a chunk, cut into pieces
    (1, 20, 66, 226, 24, 3, 3, 1, 0),    # wide rows: more than 1024 pairs of pixels a stage
    (3, 33, 5, 4, 17, 8, 8, 1, 4),       # kernel larger than the image
    (1, 30, 30, 34, 30, 7, 7, 4, 2),     # stride 4
    (3, 120, 13, 17, 40, 3, 3, 2, 1),    # odd W: pixels one by one, a last pair of one pixel
    (64, 40, 7, 7, 70, 3, 3, 1, 1),      # odd W, several images a block, four items a thread
    (5, 67, 35, 29, 93, 5, 5, 2, 2),     # odd W, nothing a multiple of anything
    (1, 40, 66, 225, 24, 3, 3, 1, 0),    # odd W, wide rows
]


# Layers whose workgroups take three chunks of channels and more, so that pixels are staged beside the products, in both
# buffers, and are read there: every form of the kernel (one, two or four items a thread, pairs or single pixels), one to
# sixteen parts a chunk, whole and cut (tests/sanitize/planner_fuzz.cpp holds the planner to these geometries).
STAGED_LATER = [
    (3, 83, 6, 30, 130, 4, 4, 1, 1),     # four parts a chunk, two pieces of three
    (1, 99, 7, 6, 260, 3, 3, 2, 1),      # stride 2, three filter blocks, the last piece one chunk
    (16, 65, 9, 6, 260, 7, 7, 1, 3),     # nine parts, three filter blocks, the last piece shorter
    (23, 61, 36, 40, 20, 10, 10, 1, 4),  # sixteen parts, 130 blocks of tiles, uncut
    (2, 132, 34, 5, 260, 4, 4, 1, 1),    # odd W
    (8, 41, 9, 9, 260, 7, 7, 1, 3),      # odd W, nine parts, uncut
    (18, 102, 29, 39, 20, 10, 10, 1, 4), # odd W, sixteen parts, many workgroups, the last piece one chunk
    (7, 35, 7, 8, 20, 3, 5, 1, 1),       # two pixels a thread, two parts, uncut
    (16, 131, 10, 10, 20, 3, 3, 2, 1),   # two, stride 2, the last chunk three channels
    (24, 40, 4, 6, 40, 5, 5, 1, 2),      # two; six tiles an image: eleven images and more a block
    (2, 108, 14, 14, 300, 3, 3, 1, 1),   # four, one part a chunk, seven chunks
    (4, 34, 31, 37, 20, 4, 4, 1, 1),     # two, odd W, uncut
    (13, 112, 23, 5, 20, 3, 3, 2, 1),    # two, odd W, stride 2
    (1, 108, 38, 5, 130, 3, 3, 1, 1),    # two, odd W, one part, the last piece one chunk
    (6, 39, 9, 32, 20, 3, 3, 2, 1),      # four, stride 2, uncut
    (17, 66, 8, 18, 20, 3, 3, 2, 1),     # four, stride 2
    (64, 48, 28, 28, 300, 3, 3, 1, 1),   # four, one part, three filter blocks, 588 workgroups
    (9, 44, 23, 33, 130, 6, 6, 2, 2),    # four, odd W, stride 2, uncut
    (12, 69, 5, 5, 130, 3, 5, 1, 1),     # four, odd W, two parts
    (1, 40, 66, 226, 24, 3, 3, 1, 0),    # more than 1024 pairs of pixels a stage in later chunks
]

# Long sums into one FP32 accumulator, uncut but for the third, at sizes of real use: error against the oracle relative to the
# largest output, staged path / this kernel: 4.3e-7 / 9.5e-7, 1.9e-7 / 3.0e-7, 7.3e-7 / 8.4e-7, 2.5e-7 / 8.5e-7; all-positive
# data 7.4e-7 / 1.3e-6 at most.  An output of the first layer adds up 392 MFMAs in each of its two accumulators (49 taps, half
# of sixteen chunks), each rounding to 2^-24 of the sum so far: 2^-24 * sqrt(392) = 1.2e-6 if independent; the bar is four times that.
LONG_SUMS = [
    (32, 256, 28, 28, 256, 7, 7, 1, 3),
    (32, 128, 56, 56, 256, 3, 3, 2, 1),
    (32, 384, 14, 14, 384, 11, 11, 1, 5),
    (128, 384, 14, 14, 256, 5, 5, 1, 2),
]
TOL_LONG = 5e-6


def _draw(fmt, shape):
    N, C, H, W, K, R, S, s, P = shape
    rng = np.random.default_rng(97)
    x = rng.standard_normal((N, C, H, W))
    w = rng.standard_normal((K, C, R, S)) * np.sqrt(2.0 / (C * R * S))
    if fmt == "f16":
        x, w = x.astype(np.float16), w.astype(np.float16)
        return x, w, oracle.dwm_half_f64(x, w, s, P)
    x, w = (torch.from_numpy(a).to(torch.bfloat16).float().numpy() for a in (x, w))
    return x, w, oracle.dwm_bf16_f64(x, w, s, P)


def _runner(fmt, shape):
    r = (th.HalfRunner if fmt == "f16" else tb.Bf16Runner)(*shape, forward=-1)
    getattr(dwm, "dwm_%s_set_variant" % fmt)(r.plan, "wide", 1)
    return r


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES + STAGED_LATER)
def test_wide_kernel_against_the_oracle(shape, fmt):
    x, w, ref = _draw(fmt, shape)
    r = _runner(fmt, shape)
    try:
        y = r.run(x, w, f32out=True)
        assert np.all(np.isfinite(y))
        assert float(np.max(np.abs(y - ref))) <= th.TOL_F32OUT * float(np.max(np.abs(ref)))
        (th._check_half_out if fmt == "f16" else tb._check_half_out)(r.run(x, w), ref)
    finally:
        r.close()


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
def test_infinities_and_nan_stay_where_the_staged_path_has_them(fmt):
    shape = (1, 24, 12, 12, 20, 3, 3, 1, 1)
    x, w, _ = _draw(fmt, shape)
    x[0, 3, 5, 5], x[0, 20, 9, 2] = np.inf, -np.inf
    if fmt == "f16":  # (the bfloat16 runner compares its input with itself)
        x[0, 0, 0, 11] = np.nan
    wide = _runner(fmt, shape)
    staged = (th.HalfRunner if fmt == "f16" else tb.Bf16Runner)(*shape, forward=0)
    try:
        a, b = wide.run(x, w, f32out=True), staged.run(x, w, f32out=True)
    finally:
        wide.close()
        staged.close()
    assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(np.isinf(a), np.isinf(b))
    ok = np.isfinite(b)
    assert ok.any() and not ok.all()
    assert float(np.max(np.abs(a[ok] - b[ok]))) <= th.TOL_F32OUT * float(np.max(np.abs(b[ok])))


def test_x_off_a_four_byte_boundary():
    shape = (2, 32, 10, 12, 40, 3, 3, 1, 1)
    x, w, ref = _draw("f16", shape)
    r = _runner("f16", shape)
    try:
        st = torch.cuda.current_stream().cuda_stream
        flat = torch.zeros(x.size + 1, dtype=torch.float16, device="cuda")
        flat[1:] = torch.from_numpy(x).cuda().flatten()
        wd = torch.from_numpy(w).cuda()
        y = torch.full(r.shape_y, float("nan"), dtype=torch.float32, device="cuda")
        dwm.dwm_f16_filter_transform(r.plan, wd.data_ptr(), r.U.data_ptr(), st)
        dwm.dwm_f16_conv_forward_f32out(r.plan, flat.data_ptr() + 2, r.U.data_ptr(), y.data_ptr(), st)
        torch.cuda.synchronize()
    finally:
        r.close()
    assert float(np.max(np.abs(y.cpu().numpy() - ref))) <= th.TOL_F32OUT * float(np.max(np.abs(ref)))


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("shape", [
    (1, 256, 14, 14, 256, 3, 3, 1, 1),   # cut into eight pieces
    (2, 100, 21, 16, 96, 6, 6, 2, 2),    # seven, the filter in a copy of its own
    (1, 16, 8, 8, 16, 3, 3, 1, 1),       # uncut
])
def test_a_whole_call_between_the_two_stages_leaves_v_alone(shape, fmt):
    x, w, _ = _draw(fmt, shape)
    staged = (th.HalfRunner if fmt == "f16" else tb.Bf16Runner)(*shape, forward=0)
    r = _runner(fmt, shape)
    fn = lambda name: getattr(dwm, "dwm_%s_%s" % (fmt, name))  # noqa: E731
    try:
        want = staged.run(x, w)
        r.run(x, w)  # (transforms the filter)
        st = torch.cuda.current_stream().cuda_stream
        xd = torch.from_numpy(np.ascontiguousarray(x)).to(torch.float16 if fmt == "f16" else torch.bfloat16).cuda()
        y, y2 = (torch.full(r.shape_y, float("nan"), dtype=xd.dtype, device="cuda") for _ in range(2))
        fn("input_transform")(r.plan, xd.data_ptr(), st)
        fn("conv_forward")(r.plan, xd.data_ptr(), r.U.data_ptr(), y.data_ptr(), st)
        fn("contract_output")(r.plan, r.U.data_ptr(), y2.data_ptr(), st)
        torch.cuda.synchronize()
    finally:
        staged.close()
        r.close()
    assert np.array_equal(y2.float().cpu().numpy(), np.asarray(want, np.float32))


@pytest.mark.parametrize("dist", ["uniform", "relu", "positive"])
@pytest.mark.parametrize("shape", LONG_SUMS)
def test_long_sums_with_the_planners_choice(shape, dist):
    """The whole batch through the planner's choice; its first image, left in FP32, element by element, in both formats."""
    N, C, H, W, K, R, S, s, P = shape
    rng = np.random.default_rng(5)
    x = rng.uniform(-1, 1, (N, C, H, W)).astype(np.float32) if dist == "uniform" else rng.standard_normal((N, C, H, W), dtype=np.float32)
    w = (rng.standard_normal((K, C, R, S)) * np.sqrt(2.0 / (C * R * S))).astype(np.float32)
    x = np.maximum(x, 0) if dist == "relu" else np.abs(x) if dist == "positive" else x
    w = np.abs(w) if dist == "positive" else w
    for fmt, cls in (("f16", th.HalfRunner), ("bf16", tb.Bf16Runner)):
        if fmt == "f16":
            a, b = x.astype(np.float16), w.astype(np.float16)
            ref = oracle.dwm_half_f64(a[:1], b, s, P)
        else:
            a, b = (torch.from_numpy(v).to(torch.bfloat16).float().numpy() for v in (x, w))
            ref = oracle.dwm_bf16_f64(a[:1], b, s, P)
        r = cls(*shape, forward=-1)
        try:
            assert getattr(dwm, "dwm_%s_forward_kernel" % fmt)(r.plan) == 2
            y = r.run(a, b, f32out=True)
        finally:
            r.close()
        assert np.all(np.isfinite(y))
        assert float(np.max(np.abs(y[:1] - ref))) <= TOL_LONG * float(np.max(np.abs(ref))), fmt


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("index", [1, 2])
def test_full_size_layers_sampled_with_the_planners_choice(index, fmt):
    """The two benchmark layers at full size, as bench.py times them: sampled 16-bit outputs against the exact convolution of the
    16-bit inputs.  Bars: what 16-bit storage of U, V and y costs, as in the formats' own suites."""
    L = wl.CONFIGS[index]
    unit = 2.0 ** -11 if fmt == "f16" else 2.0 ** -8
    x, w = wl.make_layer_tensors(L, index)
    if fmt == "f16":
        x, w = x.astype(np.float16), w.astype(np.float16)
    else:
        x, w = (torch.from_numpy(a).to(torch.bfloat16).float().numpy() for a in (x, w))
    r = (th.HalfRunner if fmt == "f16" else tb.Bf16Runner)(L.N, L.C, L.H, L.W, L.K, L.R, L.S, L.stride, L.pad, forward=-1)
    try:
        y = r.run(x, w)
    finally:
        r.close()
    assert np.all(np.isfinite(y))
    idx = np.random.default_rng(index).choice(y.size, size=4000, replace=False)
    ref = oracle.direct_f64_at(np.asarray(x, np.float32), np.asarray(w, np.float32), L.stride, L.pad, idx)
    got = y.reshape(-1)[idx].astype(np.float64)
    assert np.max(np.abs(got - ref)) <= 8 * unit * float(np.max(np.abs(ref)))
    assert np.sqrt(np.mean((got - ref) ** 2)) <= 2 * unit * np.sqrt(np.mean(ref ** 2))


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
def test_filter_transform_writes_both_copies_in_one_pass(fmt):
    """C off a multiple of sixteen: the kernel's own copy of the filter comes with the staged one.  As long as for the next
    multiple, which needs no copy (1.0 to 1.3 times, the bytes are twice as many); it was 2.6 times by a pass of its own."""
    fn = lambda name: getattr(dwm, "dwm_%s_%s" % (fmt, name))  # noqa: E731
    us = {}
    for C in (345, 352):
        p = fn("plan_create")(11, C, 25, 25, 311, 11, 11, 1, 0)
        assert fn("forward_kernel")(p) == 2
        w = torch.randn((311, C, 11, 11), device="cuda").to(torch.float16 if fmt == "f16" else torch.bfloat16)
        U = torch.empty(fn("filter_bytes")(p), dtype=torch.uint8, device="cuda")
        st = torch.cuda.current_stream().cuda_stream
        e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        times = []
        for _ in range(9):
            e0.record()
            for _ in range(4):
                fn("filter_transform")(p, w.data_ptr(), U.data_ptr(), st)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1))
        us[C] = sorted(times)[4]
        fn("plan_destroy")(p)
    assert us[345] <= 1.7 * us[352], us
