"""Direct convolutions (csrc/direct.hip) whose sums are long, with operands of zero mean and with positive ones, where every
rounding of an accumulator is one of the whole sum: no further from FP64 than the method's transforms (in the 2-norm over sampled
outputs, with the 1.05 of the direct convolution's other tests)."""
import numpy as np
import pytest

import oracle
import paper_2002_00552_amd as dwm
from dwm_gpu import Runner
from test_gpu_backward import BwdRunner

pytestmark = pytest.mark.gpu

GRADIENT = [  # N, C, H, W, K, R, S, stride, pad; steps of a wave's sum, waves that share a tile
    (64, 30, 28, 28, 384, 11, 11, 1, 5),   # 736, 4
    (256, 256, 14, 14, 256, 7, 7, 2, 3),   # 256, 1: tiles of 256 filters
    (16, 247, 32, 30, 139, 5, 5, 2, 2),    # 81, 1: the longest phase only just long
    (32, 123, 28, 25, 211, 3, 3, 1, 1),    # 123, 1
    (2, 206, 12, 14, 284, 9, 9, 2, 4),     # 113, 4
    (16, 289, 19, 9, 299, 9, 9, 2, 4),     # 121, 4: 64 filters a wave
    (16, 34, 19, 18, 193, 11, 11, 1, 5),   # 194, 8
    (16, 47, 9, 18, 340, 11, 11, 1, 5),    # 115, 8, in three pieces
]
FORWARD = [
    (40, 24, 14, 14, 384, 9, 9, 1, 4),     # 122, 1
    (32, 308, 23, 21, 31, 5, 5, 1, 2),     # 122, 4
    (64, 128, 28, 28, 128, 3, 3, 1, 1),    # 72, 1: one level
]


def _operand(rng, shape, kind):
    return (rng.uniform(0, 1, shape) if kind == "positive" else rng.standard_normal(shape)).astype(np.float32)


@pytest.mark.parametrize("kind", ["positive", "normal"])
@pytest.mark.parametrize("shape", GRADIENT)
def test_data_gradient(shape, kind):
    N, C, H, W, K, R, S, s, P = shape
    rng = np.random.default_rng(31)
    w = _operand(rng, (K, C, R, S), kind)
    dy = _operand(rng, (N, K, (H + 2 * P - R) // s + 1, (W + 2 * P - S) // s + 1), kind)
    idx = rng.choice(N * C * H * W, min(N * C * H * W, 4000), replace=False)
    ref = oracle.backward_data_f64_at(dy, w, (N, C, H, W), s, P, idx)
    off = {}
    for path, kernel in ((-1, 2), (0, 0)):
        r = BwdRunner(*shape, path=path)
        try:
            assert dwm.dwm_bwd_data_kernel(r.plan) == kernel
            off[path] = np.linalg.norm(r.run(dy, w).ravel()[idx] - ref)
        finally:
            r.close()
    assert off[-1] <= 1.05 * off[0], (off[-1] / np.linalg.norm(ref), off[0] / np.linalg.norm(ref))


@pytest.mark.parametrize("kind", ["positive", "normal"])
@pytest.mark.parametrize("shape", FORWARD)
def test_forward(shape, kind):
    N, C, H, W, K, R, S, s, P = shape
    rng = np.random.default_rng(32)
    x, w = _operand(rng, (N, C, H, W), kind), _operand(rng, (K, C, R, S), kind)
    idx, off = None, {}
    for variants, direct in (({}, True), ({"forward": 0}, False)):
        r = Runner(*shape, variants=variants)
        try:
            assert (dwm.dwm_plan_forward_kernel(r.plan) == 2) == direct
            r.set_filter(w)
            y = r.forward(x)
        finally:
            r.close()
        if idx is None:
            idx = rng.choice(y.size, 4000, replace=False)
            ref = oracle.direct_f64_at(x, w, s, P, idx)
        off[direct] = np.linalg.norm(y.ravel()[idx] - ref)
    assert off[True] <= 1.05 * off[False], (off[True] / np.linalg.norm(ref), off[False] / np.linalg.norm(ref))
