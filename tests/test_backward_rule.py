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
                                           (7792, 5536, 1552, False), (3376, 3040, 7760, False)])
def test_two_launches_where_one_is_not_clearly_faster(M, K, N, rowwise):
    assert choice(M, K, N, rowwise) == (0, 0)


# predicted 0.9 to 0.97 times two launches and no more than that: a product in one round of 128x128 and of 256x128 tiles, a contraction of eight steps,
# 64x64 tiles; and rowwise, of more than three rounds
@pytest.mark.parametrize("M,K,N,rowwise,way", [(320, 3072, 10320, False, (128, 4)), (2432, 1552, 9600, False, (128, 4)), (1600, 2048, 15360, False, (192, 4)),
                                               (416, 14336, 3968, False, (128, 4)), (256, 1008, 3616, False, (64, 0)), (13568, 4112, 304, True, (128, 4)),
                                               (10400, 5520, 352, True, (192, 5))])
def test_one_launch_where_operands_are_read_few_times(M, K, N, rowwise, way):
    assert choice(M, K, N, rowwise) == way


# 0.84 to 0.91 times two launches; the large tiles on half the XCDs each, predicted to be 0.95, 0.95 to 0.99
@pytest.mark.parametrize("M,K,N,rowwise,way", [(16384, 2048, 1024, False, (128, 4)), (11440, 5568, 512, False, (192, 5)), (480, 3584, 9472, False, (128, 4)),
                                               (8192, 3584, 8192, False, (256, 4)), (8144, 2000, 10432, False, (256, 4)),
                                               (272, 4192, 16336, True, (128, 4)), (464, 3664, 13440, True, (128, 4))])
def test_one_launch_where_it_is(M, K, N, rowwise, way):
    assert choice(M, K, N, rowwise) == way
