"""Which calls of dwm_plan_set_variant take a layer away from the direct convolution, as the header says: those that ask for a variant
by number, not those that restore the planner's choice; and layers that it has from paths two to four times as slow.  Host only."""
import pytest

import paper_2002_00552_amd as dwm

FEW, MANY = (2, 16, 33, 31, 16, 5, 5, 1, 2), (3, 29, 49, 44, 23, 3, 3, 3, 0)  # (the single kernel would have the first)
PLANNER, NUMBER = [("split", 0), ("input_cg", 0), ("contract", -1), ("input", -1), ("forward", -1)], \
                  [("split", 1), ("split", 2), ("input_cg", 1), ("contract", 10), ("input", 0), ("forward", 0)]


def _kernel(shape, *variants):
    p = dwm.dwm_plan_create(*shape)
    try:
        for v in variants:
            dwm.dwm_plan_set_variant(p, *v)
        return dwm.dwm_plan_forward_kernel(p)
    finally:
        dwm.dwm_plan_destroy(p)


@pytest.mark.parametrize("shape, other", [(FEW, 1), (MANY, 0)])
def test_variants_and_the_direct_convolution(shape, other):
    assert _kernel(shape) == 2
    for v in PLANNER:
        assert _kernel(shape, v) == 2, v
    for v in NUMBER:
        assert _kernel(shape, v) == (0 if v == ("forward", 0) else other), v
        assert _kernel(shape, v, (v[0], 0 if v[0] in ("split", "input_cg") else -1)) == 2, v


def test_data_gradient_of_stride_1_in_pieces_has_a_workspace_for_them():
    shape = (1, 256, 14, 14, 256, 3, 3, 1, 1)
    N, C, H, W = shape[:4]
    p = dwm.dwm_bwd_data_plan_create(*shape)
    try:
        assert dwm.dwm_bwd_data_kernel(p) == 2
        assert dwm.dwm_bwd_data_workspace_bytes(p) >= 2 * N * C * H * W * 4
    finally:
        dwm.dwm_bwd_data_plan_destroy(p)


# (the single kernel's blocks are one to three tiles wide there, 9.6 us against 30, 32 against 64; gradients 14 against 59, 16 against 26, 10 against 16)
@pytest.mark.parametrize("shape", [(2, 49, 15, 15, 112, 5, 3, 1, 2), (116, 17, 24, 24, 73, 3, 3, 1, 1)])
def test_forward_leaves_narrow_blocks(shape):
    assert _kernel(shape) == 2


@pytest.mark.parametrize("shape", [(1, 18, 50, 50, 89, 1, 1, 2, 0), (18, 4, 100, 100, 30, 1, 1, 2, 0), (1, 38, 33, 28, 18, 7, 7, 1, 3)])
def test_data_gradient_leaves_narrow_blocks(shape):
    p = dwm.dwm_bwd_data_plan_create(*shape)
    try:
        assert dwm.dwm_bwd_data_kernel(p) == 2
    finally:
        dwm.dwm_bwd_data_plan_destroy(p)
