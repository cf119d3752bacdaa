"""Rules of dispatch (host code of the library, no GPU): which calls a path takes, on either side of its lines."""
import ctypes as C

import pytest

from route_util import BOOL, INT, plan, rule


class DwShape(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("N", "C", "H", "W", "Ho", "Wo", "k", "s", "p")]


@pytest.mark.parametrize("N,channels,H,k,s,bf16,se,coef_ahead,folds", [
    (1, 366, 10, 5, 2, False, False, True, False),     # nothing saved
    (1, 366, 10, 5, 2, False, True, True, True),       # the pool is
    (1, 48, 7, 3, 1, True, False, False, True),        # the coefficients' launch is
    (28, 288, 25, 3, 1, False, False, False, False),   # a thread group to a plane: 32256 wavefronts, and fewer
    (24, 288, 25, 3, 1, False, False, False, True),
    (222, 288, 25, 3, 1, False, True, False, True),    # stride 1 with the pool: any size
    (24, 672, 17, 5, 2, False, True, False, False),    # stride 2 with the pool: 64512, 48384, and 93696 with one launch saved
    (18, 672, 17, 5, 2, False, True, False, True),
    (64, 366, 17, 5, 2, False, True, True, False),
    (16, 144, 72, 5, 2, False, True, False, False),    # 1024 threads, 5x5, fp32: 36864, 2304; bf16
    (1, 144, 72, 5, 2, False, True, False, True),
    (16, 144, 72, 5, 2, True, True, False, True),
    (61, 96, 82, 5, 1, False, False, False, True),     # (of dw4 and dw2: dw_fwd folds at any size)
    (16, 144, 72, 5, 1, False, True, False, True),
    (64, 144, 72, 5, 1, False, True, False, False),
    (3, 252, 72, 5, 2, False, True, True, False),
    (192, 144, 56, 5, 2, False, False, False, True),   # more pixels to a wavefront: any size
    (192, 1152, 7, 5, 1, False, False, False, True),
])
def test_evaluation_folds_launches_into_the_depthwise_kernel(N, channels, H, k, s, bf16, se, coef_ahead, folds):
    fold = rule("_ZN3mbk13dw_eval_foldsEbRKNS_7DwShapeEbb", BOOL, BOOL, C.POINTER(DwShape), BOOL, BOOL)
    p = (k - 1) // 2
    out = (H + 2 * p - k) // s + 1
    assert fold(bf16, C.byref(DwShape(N, channels, H, H, out, out, k, s, p)), se, coef_ahead) == folds


@pytest.mark.parametrize("rows,many", [((448, 448), True), ((499, 32), True), ((20, 456), True), ((128, 0), True),
                                       ((64, 64), False), ((8, 13), False), ((42, 0), False)])
def test_sum_of_partial_gradients_goes_by_the_longer_one(rows, many):
    assert rule("_ZN3mbk23reduce_splits_many_rowsEii", BOOL, INT, INT)(*rows) == many


@pytest.mark.parametrize("N,Ma,Mb,HW,splits", [(29, 171, 117, 9, 3), (1, 64, 64, 1, 1), (5, 64, 64, 49, 2), (64, 1152, 192, 49, 11)])
def test_weight_gradient_splits_have_four_chunks(N, Ma, Mb, HW, splits):
    assert plan("_ZN3mbk8wgr_planEbiiiiPi", BOOL, *4 * [INT])(False, Ma, Mb, N, HW) == splits


@pytest.mark.parametrize("bf16,N,Ma,Mb,HW,least", [
    (False, 3500, 96, 7, 3249, 2),           # 4.4 GB in all
    (False, 1, 60000, 8, 16384, 0),          # 4 GB an image: the general kernel's
    (True, 1 << 20, 1100, 8, 1, 2),          # one pixel a plane: the gates are the larger
])
def test_weight_gradients_of_4_gib_and_more(bf16, N, Ma, Mb, HW, least):
    got = plan("_ZN3mbk8wgr_planEbiiiiPi", BOOL, *4 * [INT])(bf16, Ma, Mb, N, HW)
    assert got >= least if least else got is None


@pytest.mark.parametrize("N,M,K,H,chunks", [
    (32, 240, 40, 28, 784), (64, 240, 40, 28, None),     # beside conv_pe: 1200 chunks
    (2, 48, 8, 56, 196), (41, 48, 8, 56, None),
    (12, 144, 24, 56, 1176), (13, 144, 24, 56, None),
    (30, 384, 40, 28, 735), (64, 384, 40, 28, None),
    (17, 240, 40, 27, 388), (18, 240, 40, 27, None),     # odd plane: 12288 wavefronts; so for outputs above conv_pe's
    (11, 400, 40, 28, None), (9, 400, 40, 28, 221),
    (18, 576, 96, 14, 111), (19, 576, 96, 14, None),
    (97, 64, 64, 14, 595), (99, 64, 64, 14, None),       # few rows: conv_xw from 600 chunks on
    (8, 12, 8, 57, 813), (100, 12, 8, 57, 10154),        # (conv_big: no such line)
    (1, 240, 41, 7, None), (1, 1536, 256, 7, None),      # channel counts that it does not take
])
def test_expansion_conv_of_small_launches(N, M, K, H, chunks):
    assert plan("_ZN3mbk12xs_conv_planEiiiiiiPi", *6 * [INT])(N, M, K, H * H, 0, 1) == chunks


def test_benchmark_counts_the_bytes_of_the_kernel_that_runs():
    import bench
    from mbconv_inputs import b0_chain
    blocks = b0_chain()
    s = blocks[1]  # 16 -> 96, no residual: the expansion conv's output is computed again, not read
    px = s.N * s.H * s.W * 4
    assert bench.step_bytes(s)["expand_dgrad"] == px * (s.Cexp + 2 * s.Cin)
    s = blocks[2]  # 24 -> 144 with a residual: read
    px = s.N * s.H * s.W * 4
    assert bench.step_bytes(s)["expand_dgrad"] == px * (2 * s.Cexp + 3 * s.Cin)
