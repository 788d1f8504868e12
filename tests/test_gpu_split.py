"""The single-precision contraction on the bfloat16 matrix cores (three-way split operands) through the C ABI: at the edges
of its tiles, its cuts and its reduction, against FP64 and against the fp32-MFMA contraction of the same layer."""
import numpy as np
import pytest
import torch

import oracle
import paper_2002_00552_amd as dwm
from dwm_gpu import Runner
from test_gpu_backward import BwdRunner, WgradRunner

pytestmark = pytest.mark.gpu

# (N, C, H, W, K, R, S, stride, pad): layers that the planner gives to the split contraction (test_planner_takes_it checks
# that); between them tiles of 128 and of 64 filters, whole tiles and 4 .. 16 pieces, ragged filters, tiles and channels
SHAPES = [
    (1, 256, 14, 14, 256, 3, 3, 1, 1),     # 49 tiles of 64: sixteen pieces
    (2, 64, 9, 9, 33, 4, 4, 1, 1),         # filters just past half a tile, 32 tiles
    (5, 67, 35, 29, 93, 5, 5, 2, 2),       # nothing a multiple of anything
    (4, 200, 21, 23, 129, 3, 3, 1, 0),     # one filter past 128, a piece length that does not divide
    (4, 109, 27, 28, 117, 7, 7, 1, 3),     # tiles of 128 filters cut into pieces
    (256, 128, 28, 28, 128, 3, 3, 1, 1),   # whole tiles
    (1, 300, 2, 2, 40, 3, 3, 1, 1),        # a single 2x2 tile
    (2, 1030, 6, 6, 64, 1, 1, 1, 0),       # one-tap pieces; planes longer than a fold
]


def _data(shape, seed):
    N, C, H, W, K, R, S, s, P = shape
    rng = np.random.default_rng(seed)
    x = rng.uniform(-1, 1, (N, C, H, W)).astype(np.float32)
    w = (rng.standard_normal((K, C, R, S)) * np.sqrt(2.0 / (C * R * S))).astype(np.float32)
    return x, w


def _run(shape, x, w, variants=None):
    r = Runner(*shape, variants=variants)
    try:
        r.set_filter(w)
        return r.forward(x)
    finally:
        r.close()


def test_planner_takes_it():
    """The filter buffer of these layers holds the split copy: two and a half times the classes' own floats."""
    for shape in SHAPES:
        p = dwm.dwm_plan_create(*shape)
        info = dwm.dwm_plan_info(p)
        last = dwm.dwm_plan_class(p, info.n_classes - 1)
        floats = last.u_offset + (last.len_h + 1) * (last.len_w + 1) * info.Kpad * last.Lpad
        assert dwm.dwm_plan_filter_bytes(p) == 10 * floats, shape
        dwm.dwm_plan_destroy(p)


@pytest.mark.parametrize("shape", SHAPES)
def test_no_less_exact_than_fp32_mfma(shape):
    """Sampled outputs against FP64: within 2e-6 of the largest (fp32 sums of up to 1030 x 49 products in runs of at most
    1024, folded: a few 1e-7 measured), and in the 2-norm no further off than the fp32 contraction (variant 10: it applies
    to every layer), which rounds every two products where this one rounds every sixteen."""
    x, w = _data(shape, 1)
    y = _run(shape, x, w)
    y32 = _run(shape, x, w, {"contract": 10, "forward": 0})
    rng = np.random.default_rng(2)
    idx = rng.choice(y.size, min(y.size, 4000), replace=False)
    ref = oracle.direct_f64_at(x, w, shape[7], shape[8], idx)
    scale = np.max(np.abs(ref))
    e, e32 = y.ravel()[idx] - ref, y32.ravel()[idx] - ref
    assert np.all(np.isfinite(y))
    assert np.max(np.abs(e)) / scale <= 2e-6, shape
    assert np.linalg.norm(e) <= np.linalg.norm(e32) * 1.05, (np.linalg.norm(e), np.linalg.norm(e32))


G = {1: np.array([[1.0], [1.0]]), 2: np.array([[1, 0], [1, 1], [0, 1.0]]),
     3: np.array([[1, 0, 0], [.5, .5, .5], [.5, -.5, .5], [0, 0, 1.0]])}


@pytest.mark.parametrize("shape", SHAPES)
def test_filter_copy(shape):
    """The transformed filter, plane by plane, and its split copy: the parts are the bfloat16 nearest to U, to what is left
    and the rest, and they add up to U (24 bits; nothing here is near the subnormals); padding is zero in both."""
    N, C, H, W, K, R, S, s, P = shape
    _, w = _data(shape, 9)
    r = Runner(*shape)
    try:
        r.Ugw.fill_(float("nan"))
        r.set_filter(w)
        U = r.Ugw.cpu().numpy()
        classes, parts, Kpad = r.classes(), r.parts(), r.info.Kpad
    finally:
        r.close()
    end = len(U) * 2 // 5
    copy = U[end:].view(np.uint16).astype(np.uint32) << 16
    copy = copy.view(np.float32).astype(np.float64)
    for i, c in enumerate(classes):
        planes = (c.len_h + 1) * (c.len_w + 1)
        got = U[c.u_offset:c.u_offset + planes * Kpad * c.Lpad].reshape(planes, Kpad, c.Lpad).astype(np.float64)
        sp = copy[3 * c.u_offset:3 * (c.u_offset + planes * Kpad * c.Lpad)]
        sp = sp.reshape(planes, c.Lpad // 16, 3, 2, Kpad, 8).transpose(2, 0, 4, 1, 3, 5).reshape(3, planes, Kpad, c.Lpad)
        want = np.zeros_like(got)
        for q in parts:
            if q.cls != i:
                continue
            g = w[:, :, q.phase_h + s * q.off_h:, q.phase_w + s * q.off_w:][:, :, ::s, ::s][:, :, :q.len_h, :q.len_w]
            u = np.einsum("ia,kcab,jb->ijkc", np.atleast_2d(G[q.len_h]), g.astype(np.float64), np.atleast_2d(G[q.len_w]))
            want[:, :K, q.slot * C:(q.slot + 1) * C] = u.reshape(planes, K, C)
        scale = np.max(np.abs(w))
        assert np.max(np.abs(got - want)) <= 4 * 2.0 ** -24 * 2.25 * scale, (shape, i)  # four roundings, sums of nine
        assert np.array_equal(sp.sum(axis=0), got), (shape, i)
        assert np.all(np.abs(got - sp[0]) <= 2.0 ** -8 * np.abs(sp[0])) and np.all(np.abs(sp[2]) <= 2.0 ** -16 * np.abs(sp[0]))


# filters straight from w, flipped and with their channels: rows past a block of 32, filters past a block of eight
@pytest.mark.parametrize("shape", [(2, 90, 20, 22, 271, 4, 6, 1, 2), (4, 33, 30, 29, 150, 7, 3, 1, 1), (1, 67, 14, 14, 259, 3, 3, 1, 1)])
def test_data_gradient(shape):
    N, C, H, W, K, R, S, s, P = shape
    _, w = _data(shape, 10)
    dy = np.random.default_rng(11).standard_normal((N, K, H + 2 * P - R + 1, W + 2 * P - S + 1)).astype(np.float32)
    r = BwdRunner(*shape, path=0)
    dx = r.run(dy, w)
    r.close()
    ref = oracle.backward_data_f64(dy, w, (N, C, H, W), s, P)
    assert np.max(np.abs(dx - ref)) <= 2e-6 * np.max(np.abs(ref)), shape


@pytest.mark.parametrize("shape", [SHAPES[2], SHAPES[5], SHAPES[7]])
def test_repeats_bit_for_bit(shape):
    x, w = _data(shape, 3)
    r = Runner(*shape)
    try:
        r.set_filter(w)
        first = r.forward(x)
        for _ in range(10):
            r.y.fill_(float("nan"))
            assert np.array_equal(r.forward(x), first)
    finally:
        r.close()


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38])
@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[2], SHAPES[4], SHAPES[7]])
def test_values_the_split_cannot_carry(shape, value):
    """An infinity, a NaN or a value whose bfloat16 rounding overflows, in x or in w: the same outputs are infinite, of the
    same sign, or NaN as in the fp32 contraction, and the others agree to fp32 rounding of their own largest terms.  (The
    other operand is scaled to 1e-3, so that no sum comes near the end of the range, where the order decides.)"""
    for where in ("x", "w"):
        x, w = _data(shape, 4)
        a, other = (x, w) if where == "x" else (w, x)
        other *= np.float32(1e-3)
        a[tuple(n // 2 for n in a.shape)] = value
        y = _run(shape, x, w)
        y32 = _run(shape, x, w, {"contract": 10, "forward": 0})
        assert np.array_equal(np.isnan(y), np.isnan(y32)), (where, np.isnan(y).sum(), np.isnan(y32).sum())
        assert np.array_equal(np.where(np.isinf(y), y, 0), np.where(np.isinf(y32), y32, 0)), where
        assert np.isfinite(value) == bool(np.all(np.isfinite(y32)))
        small = np.isfinite(y32) & (np.abs(y32) < 1e3)  # outputs that the value does not reach
        tall = np.isfinite(y32) & ~small
        if not np.isfinite(value):
            assert np.max(np.abs(y[small] - y32[small])) <= 4e-6 * np.max(np.abs(y32[small])), where
        assert np.all(np.abs(y[tall] - y32[tall]) <= 1e-5 * np.max(np.abs(y32[tall]), initial=0.0)), where


def test_subnormal_operands():
    """x of 1e-38 .. 1e-40, w of ordinary size: within 2e-6 of the largest output, as at any other scale, and what 2304
    roundings of outputs near the end of the range add (2^-150 each; 1e-5 of the largest here)."""
    shape = SHAPES[0]
    x, w = _data(shape, 5)
    x = (x * 1e-38).astype(np.float32)
    y = _run(shape, x, w)
    idx = np.arange(0, y.size, 37)
    ref = oracle.direct_f64_at(x, w, 1, 1, idx)
    bound = 2e-6 * np.max(np.abs(ref)) + 9 * 256 * 16 * 2.0 ** -150
    assert bound < 2e-3 * np.max(np.abs(ref))
    assert np.max(np.abs(y.ravel()[idx] - ref)) <= bound


def _off(a, ref):
    """2-norm of the difference over that of the reference, whatever its scale."""
    scale = np.max(np.abs(ref))
    return np.linalg.norm((a - ref) / scale) / np.linalg.norm(ref / scale)


def _small(a, other, how):
    """(a, other) with a, or its even channels, brought to where its parts leave bfloat16's normal range; other stays or
    makes up for it."""
    scale, up, every = how
    a, other = a.copy(), other.copy()
    a[:, ::every] *= np.float32(scale)
    other[:, ::every] *= np.float32(up)
    return a, other


SMALL = [(1e-31, 1, 1), (1e-34, 1, 1), (1e-36, 1, 1), (1e-38, 1, 1), (1e-34, 1e30, 1), (1e-38, 1e30, 1), (1e-36, 1e34, 2)]


@pytest.mark.parametrize("how", SMALL)
@pytest.mark.parametrize("where", ["x", "w"])
@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[2], SHAPES[7]])
def test_small_operands(shape, where, how):
    """x or w far below 1 (ordinary binary32 numbers whose lower parts bfloat16 has no room for), all of it or every other
    channel, the other operand ordinary or as much larger: in the 2-norm no further from FP64 than the fp32 contraction.
    (Where w is small both run on fp32 matrix cores and differ in the order of their sums: 1.1 is between two draws of the
    same error over 4000 outputs.)"""
    x, w = _data(shape, 4)
    if where == "x":
        x, w = _small(x, w, how)
    else:
        w, x = _small(w, x, how)
    y = _run(shape, x, w)
    y32 = _run(shape, x, w, {"contract": 10, "forward": 0})
    idx = np.random.default_rng(2).choice(y.size, min(y.size, 4000), replace=False)
    ref = oracle.direct_f64_at(x, w, shape[7], shape[8], idx)
    off, off32 = _off(y.ravel()[idx], ref), _off(y32.ravel()[idx], ref)
    assert off <= 1.1 * off32 and off32 < 1e-5, (off, off32)


@pytest.mark.parametrize("value", [1e34, -3.4e38])
@pytest.mark.parametrize("where", ["x", "w"])
def test_large_finite_operands(where, value):
    """A finite value whose h part, or whose scaled h part, is infinite: the outputs it reaches as in the fp32 contraction,
    those that it does not (below 1: the other operand is 1e-3) to fp32 rounding, and no output lost."""
    shape = SHAPES[0]
    x, w = _data(shape, 6)
    a, other = (x, w) if where == "x" else (w, x)
    other *= np.float32(1e-3)
    a[tuple(n // 2 for n in a.shape)] = value
    y = _run(shape, x, w)
    y32 = _run(shape, x, w, {"contract": 10, "forward": 0})
    far = np.abs(y32) < 1.0
    assert np.all(np.isfinite(y)) and 0.3 < np.mean(far) < 1.0
    assert np.max(np.abs(y[far] - y32[far])) <= 4e-6 * np.max(np.abs(y32[far]))
    assert np.max(np.abs(y[~far] - y32[~far])) <= 1e-5 * np.max(np.abs(y32[~far]))


@pytest.mark.parametrize("where, how", [("dy", SMALL[2]), ("w", SMALL[2]), ("dy", SMALL[6])])
def test_data_gradient_of_small_operands(where, how):
    """As test_data_gradient: 2e-6 of the largest, at any scale.  (Channels of dy and filters of w are summed over.)"""
    shape = (4, 33, 30, 29, 150, 7, 3, 1, 1)
    N, C, H, W, K, R, S, s, P = shape
    _, w = _data(shape, 10)
    dy = np.random.default_rng(11).standard_normal((N, K, H + 2 * P - R + 1, W + 2 * P - S + 1)).astype(np.float32)
    wt = w.transpose(1, 0, 2, 3)
    if where == "dy":
        dy, wt = _small(dy, wt, how)
    else:
        wt, dy = _small(wt, dy, how)
    w = np.ascontiguousarray(wt.transpose(1, 0, 2, 3))
    r = BwdRunner(*shape, path=0)
    dx = r.run(dy, w)
    r.close()
    ref = oracle.backward_data_f64(dy, w, (N, C, H, W), s, P)
    assert np.max(np.abs(dx - ref)) <= 2e-6 * np.max(np.abs(ref))


def test_chosen_variants_still_run_the_fp32_contraction():
    """A contraction variant or a way of sharing out the tiles that was asked for by number stays what it was: the layouts
    of the workspace differ, so the sizes tell which one is in use, and -1 / 0 bring the planner's choice back."""
    p = dwm.dwm_plan_create(*SHAPES[0])
    try:
        own = dwm.dwm_plan_workspace_bytes(p)
        dwm.dwm_plan_set_variant(p, "split", 2)  # whole tiles: no partial outputs
        assert dwm.dwm_plan_workspace_bytes(p) < own
        dwm.dwm_plan_set_variant(p, "split", 0)
        assert dwm.dwm_plan_workspace_bytes(p) == own
        dwm.dwm_plan_set_variant(p, "contract", 12)
        assert dwm.dwm_plan_workspace_bytes(p) != own
        dwm.dwm_plan_set_variant(p, "contract", -1)
        assert dwm.dwm_plan_workspace_bytes(p) == own
    finally:
        dwm.dwm_plan_destroy(p)


# ---- the filter gradient's GEMM on the bfloat16 matrix cores ----
# layers that the transforms' plan gives to it: odd and even outputs, filters past 64 and past 128, one to three ranges of tiles,
# strides 1 and 2, pieces of one, two and three taps, a last block of tiles that is nearly empty
WGRAD_SHAPES = [
    (14, 200, 27, 14, 88, 7, 7, 2, 1),
    (8, 128, 20, 18, 209, 4, 4, 1, 1),
    (3, 198, 12, 18, 196, 5, 5, 1, 2),
    (25, 297, 31, 17, 79, 4, 4, 2, 1),
    (7, 300, 14, 23, 261, 3, 3, 2, 2),
]


def _wgrad(shape, x, dy):
    r = WgradRunner(*shape, path=0)  # (the planner gives some of these layers to the plain convolution)
    try:
        assert dwm.dwm_bwd_filter_kernel(r.plan) in (0, 1)
        return r.run(x, dy)
    finally:
        r.close()


def _wgrad_tiles(shape, tile):
    p = dwm.dwm_plan_create(*shape)
    cls = [dwm.dwm_plan_class(p, i) for i in range(dwm.dwm_plan_info(p).n_classes)]
    dwm.dwm_plan_destroy(p)
    return sum((c.len_h + 1) * (c.len_w + 1) * -(-shape[4] // tile) * -(-c.Lpad // tile) for c in cls)


def _wgrad_data(shape, seed):
    x, _ = _data(shape, seed)
    N, C, H, W, K, R, S, s, P = shape
    OH, OW = (H + 2 * P - R) // s + 1, (W + 2 * P - S) // s + 1
    return x, np.random.default_rng(seed + 100).standard_normal((N, K, OH, OW)).astype(np.float32)


@pytest.mark.parametrize("shape", WGRAD_SHAPES)
def test_filter_gradient_on_bf16_matrix_cores(shape):
    """Against FP64, every tap of dw: 1e-6 of the largest (sums of up to 6000 products in at most 64 roundings a run of
    1024; 2e-7 to 4e-7 measured in the 2-norm), repeats bit for bit."""
    g = dwm.dwm_bwd_filter_plan_create(*shape)
    n = dwm.dwm_bwd_filter_plan_info(g).n_tiles
    dwm.dwm_bwd_filter_plan_destroy(g)
    assert n == _wgrad_tiles(shape, 128) != _wgrad_tiles(shape, 64)
    x, dy = _wgrad_data(shape, 7)
    N, C, H, W, K, R, S, s, P = shape
    dw = _wgrad(shape, x, dy)
    ref = oracle.backward_filter_f64(x, dy, (K, C, R, S), s, P)
    assert np.max(np.abs(dw - ref)) / np.max(np.abs(ref)) <= 2e-6
    assert np.linalg.norm(dw - ref) / np.linalg.norm(ref) <= 1e-6
    assert np.array_equal(_wgrad(shape, x, dy), dw)


@pytest.mark.parametrize("how", SMALL)
@pytest.mark.parametrize("where", ["x", "dy"])
@pytest.mark.parametrize("shape", WGRAD_SHAPES[1:3])
def test_filter_gradient_of_small_operands(shape, where, how):
    """x or dy far below 1, the other ordinary or as much larger: within 1e-6 in the 2-norm, as at any other scale.  (The
    channels of both are free here, so those that are small and those that are large are compared each by themselves.)"""
    N, C, H, W, K, R, S, s, P = shape
    x, dy = _wgrad_data(shape, 13)
    if where == "x":
        x, dy = _small(x, dy, how)
    else:
        dy, x = _small(dy, x, how)
    dw = _wgrad(shape, x, dy)
    ref = oracle.backward_filter_f64(x, dy, (K, C, R, S), s, P)
    for k in range(how[2]):
        for c in range(how[2]):
            a, b = dw[k::how[2], c::how[2]], ref[k::how[2], c::how[2]]
            assert np.all(np.isfinite(a)) and _off(a, b) <= 1e-6, (k, c)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38, 1e34])
@pytest.mark.parametrize("where", ["x", "dy"])
def test_filter_gradient_values_the_split_cannot_carry(where, value):
    """One such value in x or in dy: what it reaches is not finite where it is not (every tap of its channel, or of its
    filter, through the transforms), everything else is exact, and a finite one stays finite."""
    shape = WGRAD_SHAPES[1]
    N, C, H, W, K, R, S, s, P = shape
    x, dy = _wgrad_data(shape, 8)
    a, other = (x, dy) if where == "x" else (dy, x)
    other *= np.float32(1e-3)
    a[1, 5, 7, 9] = value
    dw = _wgrad(shape, x, dy)
    reach = np.zeros((K, C), bool)
    reach[:, 5] = where == "x"
    if where == "dy":
        reach[5, :] = True
    ref = oracle.backward_filter_f64(np.where(np.isfinite(x), x, 0).astype(np.float32),
                                     np.where(np.isfinite(dy), dy, 0).astype(np.float32), (K, C, R, S), s, P)
    assert np.all(np.isfinite(dw[~reach]))
    assert np.max(np.abs(dw[~reach] - ref[~reach])) <= 4e-6 * np.max(np.abs(ref[~reach]))
    if np.isfinite(value):
        assert np.all(np.isfinite(dw))
        assert np.max(np.abs(dw[reach] - ref[reach])) <= 4e-6 * np.max(np.abs(ref[reach]))
    else:
        # the tap that multiplies the value directly, where it has one, is never finite
        assert not np.any(np.all(np.isfinite(dw[reach]), axis=(1, 2)))


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38, 1e34])
@pytest.mark.parametrize("where", ["x", "dy"])
@pytest.mark.parametrize("shape", [WGRAD_SHAPES[1], WGRAD_SHAPES[4]])
def test_filter_gradient_is_infinite_where_the_fp32_one_is(shape, where, value):
    """The same taps of dw are infinite, of the same sign, or NaN as from the fp32 matrix cores, and the others agree.
    (A filter's gradient depends on its own channel of dy only, and plans of up to 64 filters run on fp32 matrix cores:
    the comparison is the same gradient, 64 filters at a time.)"""
    N, C, H, W, K, R, S, s, P = shape
    x, dy = _wgrad_data(shape, 14)
    a, other = (x, dy) if where == "x" else (dy, x)
    other *= np.float32(1e-3)
    a[1, 5, min(7, a.shape[2] - 1), min(9, a.shape[3] - 1)] = value
    dw = _wgrad(shape, x, dy)
    parts = [_wgrad((N, C, H, W, min(64, K - k), R, S, s, P), x, dy[:, k:k + 64]) for k in range(0, K, 64)]
    dw32 = np.concatenate(parts)
    assert np.array_equal(np.isnan(dw), np.isnan(dw32))
    assert np.array_equal(np.where(np.isinf(dw), dw, 0), np.where(np.isinf(dw32), dw32, 0))
    if np.isfinite(value):
        assert np.all(np.isfinite(dw32))
    ordinary = np.isfinite(dw32) & (np.abs(dw32) < 1e3)  # (what a finite value reaches is 1e31 and more)
    tall = np.isfinite(dw32) & ~ordinary
    assert np.mean(ordinary) > 0.9
    assert np.max(np.abs(dw[ordinary] - dw32[ordinary])) <= 4e-6 * np.max(np.abs(dw32[ordinary]))
    assert np.all(np.abs(dw[tall] - dw32[tall]) <= 1e-5 * np.max(np.abs(dw32[tall]), initial=0.0))


@pytest.mark.parametrize("shape, splits", [
    ((1, 3, 256, 256, 448, 3, 3, 1, 1), 69),   # four groups of sixteen ranges, then five
    ((1, 3, 256, 256, 40, 3, 3, 1, 1), 256),   # whole groups only
    ((8, 128, 20, 18, 209, 4, 4, 1, 1), None), # few ranges: a thread sums them all
])
def test_partial_filter_gradients_are_summed(shape, splits):
    """The kernel that adds up the ranges' partial sums: every tap of dw against FP64 (2e-6 of the largest, as above)."""
    g = dwm.dwm_bwd_filter_plan_create(*shape)
    n = dwm.dwm_bwd_filter_plan_info(g).splits
    dwm.dwm_bwd_filter_plan_destroy(g)
    assert n == splits if splits else 3 <= n < 16
    x, dy = _wgrad_data(shape, 12)
    N, C, H, W, K, R, S, s, P = shape
    dw = _wgrad(shape, x, dy)
    ref = oracle.backward_filter_f64(x, dy, (K, C, R, S), s, P)
    assert np.max(np.abs(dw - ref)) <= 2e-6 * np.max(np.abs(ref))
    assert np.array_equal(_wgrad(shape, x, dy), dw)
