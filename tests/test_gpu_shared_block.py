"""The single-kernel forward path on layers of a handful of tiles, where a workgroup's four waves share 16 tiles and split the
steps: steps that do not divide by four (waves with fewer, or none), several classes, filters up to and past 16 and 32,
odd outputs, blocks that are not full, and layers on either side of the line where blocks of 64 tiles take over."""
import numpy as np
import pytest

import oracle
import paper_2002_00552_amd as dwm
from dwm_gpu import Runner

pytestmark = pytest.mark.gpu

SHAPES = [
    (1, 16, 32, 32, 16, 5, 5, 1, 2),   # one class, 16 steps, one half of a slice
    (1, 16, 31, 29, 17, 5, 5, 1, 2),   # odd outputs, one filter past a half
    (1, 5, 16, 15, 7, 3, 3, 1, 1),     # two steps: not shared
    (2, 3, 15, 16, 33, 4, 4, 1, 1),    # three steps: not shared
    (1, 9, 18, 18, 40, 5, 5, 1, 0),    # nine steps: waves of 3, 3, 3, 0
    (1, 7, 21, 18, 64, 7, 7, 1, 3),    # three-tap and two-tap pieces in mixed steps
    (1, 6, 32, 30, 20, 3, 3, 2, 1),    # a phase with a single tap: four classes of two steps
    (3, 2, 31, 31, 16, 9, 9, 2, 4),    # eight steps, odd outputs
    (1, 12, 40, 16, 48, 3, 5, 1, 1),   # narrow output, kernel not square, a slice that is half empty
    (16, 3, 64, 64, 64, 7, 7, 2, 3),   # 64 blocks of two slices: the last that is shared
    (17, 3, 64, 64, 64, 7, 7, 2, 3),   # one image more: not shared
]


@pytest.mark.parametrize("shape", SHAPES)
def test_shared_blocks_match_fp64_direct(shape):
    """Within 4e-6 of the largest output (fp32 sums of up to 784 products; 1e-7 to 3e-7 measured in the 2-norm), every
    output written, and the same bits again."""
    N, C, H, W, K, R, S, s, P = shape
    rng = np.random.default_rng(11)
    x = rng.uniform(-1, 1, (N, C, H, W)).astype(np.float32)
    w = (rng.standard_normal((K, C, R, S)) * np.sqrt(2.0 / (C * R * S))).astype(np.float32)
    r = Runner(*shape, variants={"forward": 1})  # (with 16 channels the planner takes the plain convolution)
    try:
        assert dwm.dwm_plan_forward_kernel(r.plan) == 1
        r.set_filter(w)
        y = r.forward(x)
        r.y.fill_(float("nan"))
        assert np.array_equal(r.forward(x), y)
    finally:
        r.close()
    ref = oracle.direct_f64(x, w, s, P)
    assert np.all(np.isfinite(y)) and np.max(np.abs(y - ref)) / np.max(np.abs(ref)) <= 4e-6
