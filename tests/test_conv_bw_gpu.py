"""bf16 storage, short contractions with the weights resident in LDS: one to six steps of the contraction, a last step that
is not full, a last slab of rows and a last chunk of pixels that are not, one chunk and several to a wavefront, against the
oracle at the tolerances of parity_util; and on which side of its lines a shape is."""
import pytest

from mbconv_inputs import BlockShape, make_block_inputs
from oracle import oracle as orc
from parity_util import compare_block, run_gpu_block
from route_util import INT, plan

NONE, BNBWD, STATS, NO_EPILOGUE = 0, 2, 1, 0


def sets(N, M, K, HW, pro):
    return plan("_ZN3mbk12bw_conv_planEiiiiiiPi", *6 * [INT])(N, M, K, HW, pro, STATS if pro == NONE else NO_EPILOGUE)


@pytest.mark.parametrize("N,M,K,HW,pro,taken", [
    (128, 672, 112, 196, NONE, True), (128, 672, 112, 196, BNBWD, True),
    (40, 288, 72, 400, NONE, False), (41, 288, 72, 400, NONE, True), (12, 288, 72, 400, BNBWD, False),  # 320 and 128 groups
    (128, 672, 112, 49, NONE, False), (128, 670, 112, 196, NONE, False), (128, 672, 110, 196, NONE, False),
    (128, 1200, 200, 196, NONE, False), (128, 64, 72, 196, BNBWD, False), (16384, 672, 112, 196, NONE, False),
])
def test_rule(N, M, K, HW, pro, taken):
    assert (sets(N, M, K, HW, pro) is not None) == taken


@pytest.mark.gpu
@pytest.mark.parametrize("N,Cin,Cexp,Cout,H,W,stride", [
    (285, 48, 72, 32, 12, 12, 1),    # two steps and one; two slabs, the second of eight rows
    (85, 72, 200, 88, 16, 17, 1),    # three
    (53, 112, 456, 104, 14, 14, 1),  # four, the last half full; several chunks to a wavefront
    (42, 152, 608, 136, 14, 14, 1),  # five
    (70, 192, 392, 168, 12, 14, 1),  # six
    (33, 40, 640, 64, 18, 18, 2),    # the data gradient's planes four times smaller
])
def test_matches_oracle(N, Cin, Cexp, Cout, H, W, stride):
    s = BlockShape(N=N, Cin=Cin, H=H, W=W, Cexp=Cexp, Cse=8, Cout=Cout, k=3, stride=stride, has_expand=True,
                   residual=False, dtype="bf16")
    wave = Cin <= 40  # (the register-direct kernels)
    assert wave or sets(N, Cexp, Cin, H * W, NONE)
    assert (s.Ho * s.Wo) % 4 or Cout <= 40 or sets(N, Cexp, Cout, s.Ho * s.Wo, BNBWD)
    t = make_block_inputs(s, seed=Cexp)
    print(f"[conv bw] {s}", flush=True)
    res, blk = run_gpu_block(s, t)
    f, b = orc.mbconv_step(s, t)
    compare_block(s, t, res, f, b, blk)
