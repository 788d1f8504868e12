"""Data gradient at stride above one on layers with fewer tiles than CUs: tiles cut into pieces, one tile grid and one input
transform for sub-convolutions of unequal size, one filter transform for all.  Against FP64 at the forward bar (1e-4 of the
largest; a few 1e-7 measured)."""
import numpy as np
import pytest

import oracle
from test_gpu_backward import TOL, BwdRunner, _rand, _relerr

pytestmark = pytest.mark.gpu

SHAPES = [  # N, C, H, W, K, R, S, stride, pad
    (5, 67, 35, 29, 93, 5, 5, 2, 2),     # unequal grids, pieces that do not divide a tile's chunks
    (1, 17, 9, 8, 200, 3, 3, 2, 1),      # one tile a sub-convolution; 1-tap phases: a piece count of one beside longer ones
    (2, 20, 21, 21, 40, 7, 7, 2, 3),     # sub-convolutions of up to four parts, odd image
    (2, 33, 20, 20, 64, 4, 4, 3, 1),     # stride 3: nine sub-convolutions
    (1, 18, 23, 19, 70, 5, 5, 4, 2),     # stride 4: more sub-convolutions than one filter launch takes
    (1, 65, 31, 30, 130, 6, 3, 2, 0),    # R != S, filters one past a tile, rows and columns no tap reaches
    (3, 24, 18, 6, 500, 3, 3, 2, 1),     # a narrow image
    (40, 64, 33, 33, 64, 3, 3, 2, 1),    # more tiles than CUs: whole tiles on an unequal grid
]


@pytest.mark.parametrize("shape", SHAPES)
def test_data_gradient_of_small_strided_layers(shape):
    N, C, H, W, K, R, S, s, P = shape
    w, dy = _rand(*shape, seed=500 + R * 7 + S)
    ref = oracle.backward_data_f64(dy, w, (N, C, H, W), s, P)
    r = BwdRunner(*shape, path=0)
    try:
        dx = r.run(dy, w)
        again = r.run(dy, w)
    finally:
        r.close()
    assert np.all(np.isfinite(dx))
    assert _relerr(dx, ref) <= TOL, shape
    assert np.array_equal(dx, again)  # the pieces are added in a fixed order
