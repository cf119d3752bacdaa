"""bf16 storage, short contractions with the weights resident in LDS: one to six steps of the contraction, a last step that
is not full, a last slab of rows and a last chunk of pixels that are not, one chunk and several to a wavefront, against the
oracle at the tolerances of parity_util; and on which side of its lines a shape is."""
import numpy as np
import pytest

from mbconv_inputs import BlockShape, make_block_inputs
from oracle import oracle as orc
from paper_2110_10802_amd import binding as B
from parity_util import compare_block, run_gpu_block
from route_util import INT, bw_form, plan

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


# (N, Cin, Cexp, Cout, H, W, stride): of the expansion conv and of the projection conv's data gradient the steps of the
# contraction, the chunks to a wavefront and the pixels of the last chunk (None: another kernel)
# (Inputs for which the storage and the operands leave room below the tolerance: tests/rounding_model.py, 64 bits with those
# roundings, is 1.1e-2 to 1.8e-2 from the oracle in BN1's gamma gradient, the residue of a sum that cancels.  With 672 expanded
# channels in place of 648 it is 2.17e-2, and this kernel 2.21e-2.)
FORMS = {
    (285, 48, 72, 32, 12, 12, 1): ((2, 1, 16), None),           # two slabs, the second of eight rows
    (85, 72, 200, 88, 16, 17, 1): ((3, 1, 16), (3, 1, 16)),
    (53, 112, 456, 104, 14, 14, 1): ((4, 1, 20), (4, 1, 20)),   # the last step half full
    (42, 152, 608, 136, 14, 14, 1): ((5, 1, 40), (5, 1, 40)),
    (70, 192, 392, 168, 12, 14, 1): ((6, 1, 48), (6, 1, 48)),
    (33, 40, 640, 64, 18, 18, 2): ((2, 1, 4), None),            # one pixel run in the last chunk; planes of 81
    (205, 32, 400, 32, 12, 14, 1): ((1, 2, 8), (1, 2, 8)),      # several chunks to a wavefront, in every form
    (101, 48, 640, 64, 14, 14, 1): ((2, 2, 20), (2, 2, 20)),
    (301, 72, 264, 96, 12, 12, 1): ((3, 2, 16), (3, 2, 16)),
    (93, 104, 648, 120, 14, 14, 1): ((4, 2, 52), (4, 2, 52)),
    (150, 136, 136, 136, 18, 18, 1): ((5, 2, 24), (5, 2, 24)),
    (75, 168, 392, 168, 18, 18, 1): ((6, 2, 44), (6, 2, 44)),
}


@pytest.mark.parametrize("shape", list(FORMS), ids=str)
def test_form(shape):
    N, Cin, Cexp, Cout, H, W, stride = shape
    Ho, Wo = -(-H // stride), -(-W // stride)
    # (up to 32 output channels one kernel may compute both gradients of the projection conv)
    both = plan("_ZN3mbk18projbwd_fused_planEiiiiPi", *4 * [INT])(N, Cexp, Cout, Ho * Wo) is not None
    assert (bw_form(N, Cexp, Cin, H * W, False), None if both else bw_form(N, Cexp, Cout, Ho * Wo, True)) == FORMS[shape]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", list(FORMS), ids=str)
def test_matches_oracle(shape):
    N, Cin, Cexp, Cout, H, W, stride = shape
    s = BlockShape(N=N, Cin=Cin, H=H, W=W, Cexp=Cexp, Cse=8, Cout=Cout, k=3, stride=stride, has_expand=True,
                   residual=False, dtype="bf16")
    t = make_block_inputs(s, seed=Cexp)
    print(f"[conv bw] {s}", flush=True)
    res, blk = run_gpu_block(s, t)
    f, b = orc.mbconv_step(s, t)
    compare_block(s, t, res, f, b, blk)


@pytest.mark.gpu
def test_statistics_of_many_chunks_are_exact():
    """The statistics are fp32 sums over 64 pixels, combined in fp64, however many chunks a wavefront has.  Values in [1, 2)
    of bf16 and their squares are multiples of 2^-7 and 2^-14, so such a sum is exact (64 < 2^7 of them below 2^2 take
    7 + 2 + 14 = 23 bits) and what is left is fp64's rounding, 2^-53 a step, over a variance of a thousandth of the squares'
    mean, and the results' own rounding to fp32.  (Eight chunks of a wavefront in one fp32 sum: 1.7e-6.)"""
    import torch
    from paper_2110_10802_amd.harness import DeviceBlock

    s = BlockShape(N=1024, Cin=48, H=32, W=32, Cexp=64, Cse=4, Cout=16, k=3, stride=2, has_expand=True, residual=False,
                   dtype="bf16")
    assert (s.N * s.H * s.W // 64) / (4 * sets(s.N, s.Cexp, s.Cin, s.H * s.W, NONE)) >= 8  # chunks to a wavefront
    t = make_block_inputs(BlockShape(**{**s.__dict__, "N": 1}), seed=5)
    t["w_expand"] = t["w_expand"] * 0 + 0.0078125 * np.sign(t["w_expand"])
    t["w_expand"][:, 0] = 1.5
    blk = DeviceBlock(s, t)
    gen = torch.Generator(device=blk.device).manual_seed(6)
    x = torch.randn((s.N, s.Cin, s.H, s.W), generator=gen, device=blk.device)
    x[:, 0] = 1.0
    blk.forward(x.to(torch.bfloat16))
    torch.cuda.synchronize()
    at = B.mbconv_saved_offsets(blk.desc)
    e = blk.saved[at["e"]:][:2 * s.N * s.Cexp * s.H * s.W].view(torch.bfloat16).view(s.N, s.Cexp, -1)
    assert float(e.min()) >= 1 and float(e.max()) < 2
    got = blk.saved[at["bn1"]:][:16 * s.Cexp].view(torch.float32).view(4, s.Cexp).double()
    mean = torch.stack([e[:, c].double().mean() for c in range(s.Cexp)])
    var = torch.stack([e[:, c].double().var(unbiased=False) for c in range(s.Cexp)])
    rstd = 1 / torch.sqrt(var + blk.desc.bn_eps)
    assert float((got[2] / mean - 1).abs().max()) < 2 ** -23
    assert float((got[3] / rstd - 1).abs().max()) < 2 ** -23
