"""GPU parity tests of the 16-bit kernel for layers with many input channels (dwm_f16_* / dwm_bf16_* conv_forward, "wide"),
through the C ABI against the FP64 oracle with 16-bit storage.  Bars: those of the two formats' own suites.  The layers sit
where the kernel can go wrong: chunks of 16 channels, blocks of 128 filters and 64 tiles not filled, tiles of several
images in a block, every class of parts, odd numbers of stages, channels cut into pieces, shares of pixels that need more than
one round, images narrower than the kernel."""
import numpy as np
import pytest
import torch

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
    (9, 24, 4, 6, 40, 5, 5, 1, 2),       # six tiles an image: eleven images a block
    (1, 19, 40, 40, 20, 11, 11, 1, 5),   # sixteen parts
    (2, 100, 21, 16, 96, 6, 6, 2, 2),    # seven chunks
    (1, 256, 14, 14, 256, 3, 3, 1, 1),   # one stage a chunk, cut into pieces
    (1, 20, 66, 226, 24, 3, 3, 1, 0),    # wide rows: more than 1024 pairs of pixels a stage
    (3, 33, 5, 4, 17, 8, 8, 1, 4),       # kernel larger than the image
    (1, 30, 30, 34, 30, 7, 7, 4, 2),     # stride 4
    (3, 120, 13, 17, 40, 3, 3, 2, 1),    # odd W: pixels one by one, a last pair of one pixel
    (64, 40, 7, 7, 70, 3, 3, 1, 1),      # odd W, several images a block, two items a thread
    (5, 67, 35, 29, 93, 5, 5, 2, 2),     # odd W, nothing a multiple of anything
    (1, 40, 66, 225, 24, 3, 3, 1, 0),    # odd W, wide rows
]


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
@pytest.mark.parametrize("shape", SHAPES)
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
