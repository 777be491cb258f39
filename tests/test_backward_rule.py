"""One launch or two for a linear's backward (f8_gemm_pair.hip): the rule is a function of the sizes, so it is asked without a
GPU.  The sizes and what they were measured to take are in profiles/linear_backward_one_launch_sample.md."""
import ctypes as C

import pytest

from paper_2410_06511_amd import f8


class PairChoice(C.Structure):
    _fields_ = [("tile", C.c_int), ("x_xcds", C.c_int)]


def choice(M, K, N, rowwise):
    """Of a caller with a full workspace, on 256 compute units."""
    rule = getattr(f8.lib(), f"_ZN2f820gemm_pair_choice_0_{int(rowwise)}Eiiibmi")
    rule.restype, rule.argtypes = PairChoice, [C.c_int, C.c_int, C.c_int, C.c_bool, C.c_size_t, C.c_int]
    d = max(M, K, N)
    c = rule(M, K, N, True, f8.workspace_bytes(d, d), 256)
    return c.tile, c.x_xcds


# one launch takes 1.02 to 1.10 times two, or gives nothing
@pytest.mark.parametrize("M,K,N,rowwise", [(3008, 2928, 4528, False), (2992, 4752, 2256, False), (4896, 2784, 3408, False), (8336, 2592, 3696, False),
                                           (5712, 640, 432, False), (15632, 3792, 432, True), (14496, 3552, 912, True),
                                           (4176, 14736, 352, True), (272, 3232, 15504, True), (10320, 5888, 336, True)])
def test_two_launches_where_one_is_not_clearly_faster(M, K, N, rowwise):
    assert choice(M, K, N, rowwise) == (0, 0)


# another tile in the one launch takes 1.02 to 1.04 times as long
@pytest.mark.parametrize("M,K,N,rowwise,way", [(752, 4528, 15056, False, (256, 4)), (11808, 1232, 1696, False, (192, 4)), (5440, 11440, 272, True, (256, 5))])
def test_the_first_tile_where_another_is_not_clearly_faster(M, K, N, rowwise, way):
    assert choice(M, K, N, rowwise) == way


# 0.84 to 0.91 times two launches; the large tiles on half the XCDs each, predicted to be 0.95, 0.95 to 0.99
@pytest.mark.parametrize("M,K,N,rowwise,way", [(16384, 2048, 1024, False, (128, 4)), (11440, 5568, 512, False, (192, 5)), (480, 3584, 9472, False, (128, 4)),
                                               (8192, 3584, 8192, False, (256, 4)), (8144, 2000, 10432, False, (256, 4)),
                                               (272, 4192, 16336, True, (128, 4)), (464, 3664, 13440, True, (128, 4))])
def test_one_launch_where_it_is(M, K, N, rowwise, way):
    assert choice(M, K, N, rowwise) == way
