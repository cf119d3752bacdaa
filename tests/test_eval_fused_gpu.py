"""Evaluation mode, fp32: the expansion and depthwise convs in one launch, and the projection conv of small launches with the
gate and BN3 in another, at the edges of their tiles, slices and rules, against the oracle at the tolerances of parity_util."""
import ctypes as C

import pytest

from mbconv_inputs import BlockShape, make_block_inputs
from route_util import BOOL, INT, plan, rule
from test_eval_routes_gpu import check
from test_routes import DwShape

# (N, Cin, Cexp, Cse, Cout, H, W, k, stride): strips of the fused expansion (None: not taken), projection in one launch
CASES = {
    "one_image_7x7": ((1, 192, 1152, 48, 192, 7, 7, 5, 1), 1, True),
    "one_image_14x14": ((1, 112, 672, 28, 112, 14, 14, 5, 1), 2, True),
    "strips_28x28": ((1, 40, 240, 10, 40, 28, 28, 5, 1), 7, True),
    "strips_odd_width_stride_2": ((2, 16, 36, 4, 20, 61, 59, 3, 2), 8, True),
    "strips_112x112_stride_2": ((1, 16, 96, 4, 24, 112, 112, 3, 2), 28, True),
    "widest_128x128": ((1, 8, 20, 4, 12, 128, 128, 3, 1), 64, True),
    "128x126_5x5": ((1, 8, 20, 4, 12, 128, 126, 5, 1), None, True),
    "masked_channels": ((3, 23, 50, 5, 17, 15, 14, 3, 1), 2, True),
    "last_strip_shorter": ((2, 9, 17, 4, 9, 31, 30, 5, 2), 2, True),
    "images_side_by_side_7x7": ((200, 24, 144, 6, 24, 7, 7, 3, 1), 1, False),
    "images_side_by_side_4x3": ((600, 16, 96, 4, 16, 4, 3, 3, 1), 1, True),
    "several_items_to_a_workgroup": ((2100, 8, 16, 4, 8, 28, 28, 3, 1), 2, False),
    "64_squeezed": ((1, 64, 256, 64, 72, 9, 9, 3, 1), 1, True),
    "65_squeezed": ((1, 64, 256, 65, 72, 9, 9, 3, 1), 1, False),
    "3_squeezed": ((1, 16, 64, 3, 24, 9, 9, 3, 1), 1, False),
    "odd_contraction": ((2, 41, 130, 7, 40, 10, 10, 3, 1), None, True),
    "1x1_plane": ((2, 16, 30, 4, 16, 1, 1, 3, 1), 1, True),
    "2x5_plane_stride_2": ((5, 8, 33, 4, 5, 2, 5, 5, 2), 1, True),
    "longest_slices": ((1, 160, 1280, 33, 16, 5, 5, 3, 1), 1, True),
}


def dw_shape(N, Cexp, H, W, k, s):
    p = (k - 1) // 2
    return DwShape(N, Cexp, H, W, (H + 2 * p - k) // s + 1, (W + 2 * p - k) // s + 1, k, s, p)


def strips(N, Cin, Cexp, H, W, k, s):
    fused = plan("_ZN3mbk19eval_expand_dw_planERKNS_7DwShapeEiPi", C.POINTER(DwShape), INT)
    return fused(C.byref(dw_shape(N, Cexp, H, W, k, s)), Cin)


def projection(N, Cout, Cexp, HW, Cse, act):
    return rule("_ZN3mbk14eval_proj_planEiiiiib", BOOL, *5 * [INT], BOOL)(N, Cout, Cexp, HW, Cse, act)


@pytest.mark.parametrize("name", list(CASES))
def test_route(name):
    (N, Cin, Cexp, Cse, Cout, H, W, k, s), want, proj = CASES[name]
    got = strips(N, Cin, Cexp, H, W, k, s)
    d = dw_shape(N, Cexp, H, W, k, s)
    assert got == want
    assert projection(N, Cout, Cexp, d.Ho * d.Wo, Cse, got is None) == proj


@pytest.mark.parametrize("N,Cin,Cexp,H,W,k,s,taken", [
    (16, 80, 480, 14, 14, 3, 1, True), (18, 80, 480, 14, 14, 3, 1, False),       # 512 workgroups
    (6, 112, 672, 14, 14, 5, 1, True), (7, 112, 672, 14, 14, 5, 1, False),       # 256
    (1, 81, 486, 14, 14, 3, 1, False), (1, 200, 1200, 7, 7, 3, 1, False),        # odd, and longer than any
    (128, 24, 144, 56, 56, 3, 1, True), (64, 24, 144, 56, 56, 5, 2, False),      # up to 24 channels: any size, but
    (64, 16, 64, 127, 127, 5, 1, False), (73, 8, 24, 108, 108, 3, 2, False), (1024, 24, 144, 7, 7, 5, 1, False),
    (8, 16, 96, 72, 72, 3, 1, True), (8, 16, 96, 96, 96, 3, 1, False), (1, 16, 96, 96, 96, 3, 1, True),          # rows computed twice
    (1, 16, 96, 112, 112, 5, 1, False), (8, 16, 96, 72, 72, 5, 2, True), (1, 16, 96, 128, 128, 5, 2, False),
    (16, 80, 320, 12, 12, 3, 1, False), (12, 80, 320, 12, 12, 3, 1, True), (4, 32, 192, 64, 64, 3, 1, False),     # a second
    (17, 80, 320, 14, 14, 3, 1, True), (31, 40, 240, 16, 16, 3, 1, True), (30, 40, 160, 12, 12, 3, 1, False), (9, 32, 192, 36, 36, 3, 2, True), (9, 80, 240, 28, 28, 5, 2, False),       # round
    (3, 160, 960, 12, 12, 3, 1, False), (2, 160, 960, 12, 12, 3, 1, True), (3, 176, 1056, 8, 8, 3, 1, True),      # chunks of
    (4, 144, 432, 16, 16, 3, 1, False), (2, 176, 528, 22, 22, 3, 1, False), (3, 192, 1152, 12, 12, 3, 1, True),   # the longest
    (64, 24, 144, 56, 56, 3, 2, False), (64, 24, 144, 48, 48, 3, 2, True), (17, 22, 132, 112, 112, 3, 2, False),  # strips of
    (26, 24, 144, 68, 68, 3, 2, True), (96, 24, 144, 64, 64, 3, 2, True), (30, 24, 144, 56, 56, 3, 2, True),      # stride 2
    (376, 24, 144, 8, 6, 3, 1, False), (376, 24, 144, 8, 8, 3, 1, True),
    (1, 8, 24, 110, 82, 3, 2, False),                                            # planes that the depthwise kernels refuse
])
def test_rule(N, Cin, Cexp, H, W, k, s, taken):
    assert (strips(N, Cin, Cexp, H, W, k, s) is not None) == taken


@pytest.mark.gpu
@pytest.mark.parametrize("variant", ["se", "no_se", "relu6", "residual", "no_expand"])
@pytest.mark.parametrize("name", list(CASES))
def test_matches_oracle(name, variant):
    (N, Cin, Cexp, Cse, Cout, H, W, k, s), _, _ = CASES[name]
    if variant == "residual":
        if s != 1:
            pytest.skip("a residual needs stride 1")
        Cout = Cin
    expand = variant != "no_expand"
    check(BlockShape(N=N, Cin=Cin if expand else Cexp, H=H, W=W, Cexp=Cexp, Cse=Cse, Cout=Cout, k=k, stride=s,
                     has_expand=expand, residual=variant == "residual", has_se=variant not in ("no_se", "relu6"),
                     activation="relu6" if variant == "relu6" else "swish"), len(name))


@pytest.mark.parametrize("N,Cout,Cexp,HW,Cse,act,taken", [
    (56, 38, 96, 64, 6, True, True), (58, 24, 96, 144, 6, True, False), (25, 38, 114, 256, 9, True, False),  # 256 workgroups
    (11, 10, 24, 4624, 6, True, True),                                      # of a short contraction: more
    (10, 29, 48, 2304, 0, True, False), (29, 21, 32, 324, 0, True, True), (58, 24, 96, 144, 6, False, True),
    (92, 24, 96, 98, 6, True, False), (26, 24, 96, 98, 6, True, True), (26, 40, 480, 98, 6, True, False),  # 2600 wavefronts
])
def test_rule_of_the_projection(N, Cout, Cexp, HW, Cse, act, taken):
    assert projection(N, Cout, Cexp, HW, Cse, act) == taken


# A block without SE stage in one launch: (N, Cin, Cexp, Cout, H, W, k)
WHOLE = {
    "strips_56x56": (21, 24, 144, 24, 56, 56, 3),
    "strips_odd_width": (41, 23, 50, 17, 39, 37, 3),          # a last strip that is shorter, one pixel to a load
    "even_width_masked_channels": (55, 9, 33, 33, 30, 34, 3),
    "36_input_channels_64_rows": (81, 36, 72, 64, 25, 28, 3),
    "two_images_14x14_5x5": (321, 40, 104, 40, 14, 14, 5),
    "eight_images_7x7": (1283, 16, 48, 16, 7, 7, 5),
    "eight_images_5x3": (1281, 11, 17, 5, 5, 3, 3),
}


@pytest.mark.parametrize("N,Cin,Cexp,Cout,H,W,k,s,taken", [
    (17, 24, 144, 24, 56, 56, 3, 1, True), (16, 24, 144, 24, 56, 56, 3, 1, False),   # most of a round's places taken,
    (33, 24, 144, 24, 56, 56, 3, 1, False), (42, 24, 144, 24, 56, 56, 3, 1, True),   # of a second one, too
    (363, 40, 240, 40, 16, 16, 3, 1, True), (128, 40, 240, 40, 16, 16, 3, 1, False), (71, 32, 128, 34, 81, 83, 3, 1, True),
    (132, 32, 192, 23, 24, 24, 3, 1, False), (23, 32, 192, 38, 65, 65, 3, 1, False),  # slower by a third and more
    (126, 24, 96, 39, 40, 40, 5, 1, False), (270, 40, 240, 40, 26, 28, 5, 1, False), (35, 32, 96, 37, 80, 80, 3, 1, False),
    (88, 40, 160, 40, 68, 68, 3, 1, True),                                           # an expanded tensor of 260 MB
    (99, 8, 48, 8, 16, 16, 3, 1, False), (100, 8, 48, 8, 20, 20, 3, 1, True), (67, 24, 72, 36, 22, 22, 3, 1, False),        # a hundred workgroups
    (64, 41, 246, 40, 28, 28, 3, 1, False), (128, 40, 240, 65, 28, 28, 3, 1, False),
    (128, 32, 192, 32, 28, 28, 3, 2, False), (40, 24, 144, 30, 57, 57, 5, 1, False),
])
def test_rule_of_the_whole_block(N, Cin, Cexp, Cout, H, W, k, s, taken):
    whole = rule("_ZN3mbk15eval_block_planERKNS_7DwShapeEii", BOOL, C.POINTER(DwShape), INT, INT)
    assert whole(C.byref(dw_shape(N, Cexp, H, W, k, s)), Cin, Cout) == taken


@pytest.mark.gpu
@pytest.mark.parametrize("activation", ["relu6", "swish"])
@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("name", list(WHOLE))
def test_whole_block_matches_oracle(name, residual, activation):
    N, Cin, Cexp, Cout, H, W, k = WHOLE[name]
    Cout = Cin if residual else Cout
    whole = rule("_ZN3mbk15eval_block_planERKNS_7DwShapeEii", BOOL, C.POINTER(DwShape), INT, INT)
    assert whole(C.byref(dw_shape(N, Cexp, H, W, k, 1)), Cin, Cout)
    check(BlockShape(N=N, Cin=Cin, H=H, W=W, Cexp=Cexp, Cse=1, Cout=Cout, k=k, stride=1, has_expand=True,
                     residual=residual, has_se=False, activation=activation), len(name))


# Every step of an evaluation that another launch may have in it: (N, Cin, Cexp, Cout, H, W, k, SE, bf16), the steps that occur
PROBED = {
    "one_launch": ((21, 24, 144, 24, 56, 56, 3, False, False), "bn1_finalize expand_conv dw_fwd proj_conv bn3_apply"),
    "two_launches": ((1, 24, 144, 40, 56, 56, 3, True, False),
                     "bn1_finalize expand_conv dw_fwd se_pool se_fc proj_conv bn3_apply"),
    "no_expansion": ((1, 32, 32, 16, 112, 112, 3, True, False), "bn2_finalize dw_fwd se_pool se_fc proj_conv bn3_apply"),
    "affine_epilogue": ((128, 112, 672, 112, 14, 14, 5, True, True),
                        "bn1_finalize expand_conv dw_fwd se_pool se_fc proj_conv bn3_apply"),
    "odd_channels": ((64, 33, 99, 20, 15, 13, 5, True, False),
                 "bn1_finalize expand_conv dw_fwd se_pool se_fc proj_conv bn3_apply"),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(PROBED))
def test_every_step_answers_a_probe(name):
    import torch
    from bench import HipEvents
    from paper_2110_10802_amd import binding as B
    from paper_2110_10802_amd.harness import DeviceBlock

    (N, Cin, Cexp, Cout, H, W, k, se, bf16), steps = PROBED[name]
    s = BlockShape(N=N, Cin=Cin, H=H, W=W, Cexp=Cexp, Cse=8, Cout=Cout, k=k, stride=1, has_expand=Cin != Cexp,
                   residual=Cin == Cout, has_se=se, dtype="bf16" if bf16 else "f32")
    t = make_block_inputs(s, seed=3)
    blk = DeviceBlock(s, t)
    x = blk.to_device(t["x"])
    blk.forward_eval(x)
    ev = HipEvents()
    for step in steps.split():
        a, b = ev.create(), ev.create()
        B.mbconv_forward_eval_probed(blk.desc, blk.params, blk.running, x, blk.out, blk.eval_ws, 0,
                                     B.Probe(B.STEPS[step], a, b))
        torch.cuda.synchronize()
        print(f"[probe] {name} {step}", flush=True)
        ms = ev.elapsed_ms(a, b)  # (an error if the events were not recorded)
        assert ms > 0.003 or step != "dw_fwd"
        ev.destroy(a)
        ev.destroy(b)


@pytest.mark.gpu
def test_whole_block_in_place():
    """A call whose output lies over its input is not given to the one-launch kernel, whose workgroups read each other's
    rows."""
    import torch
    from paper_2110_10802_amd import binding as B
    from paper_2110_10802_amd.harness import DeviceBlock

    N, Cin, Cexp, _, H, W, k = WHOLE["strips_56x56"]
    s = BlockShape(N=N, Cin=Cin, H=H, W=W, Cexp=Cexp, Cse=1, Cout=Cin, k=k, stride=1, has_expand=True, residual=True,
                   has_se=False, activation="relu6")
    t = make_block_inputs(s, seed=3)
    blk = DeviceBlock(s, t)
    x = blk.to_device(t["x"])
    want = blk.forward_eval(x).clone()
    for _ in range(2):
        y = x.clone()
        B.mbconv_forward_eval(blk.desc, blk.params, blk.running, y, y, blk.eval_ws, 0)
        torch.cuda.synchronize()
        # two fp32 evaluations of one block, each within 2e-6 of the result's scale
        assert float((y - want).abs().max()) <= 1e-5 * float(want.abs().max())


@pytest.mark.gpu
@pytest.mark.parametrize("Cin", [24, 28, 36, 40])
def test_whole_block_is_as_exact_as_separate_launches(Cin):
    """Error against 64 bits (2-norm) of one launch and of the separate ones, which a call takes whose output lies over
    its input: a chain of MFMAs that is as long as the contraction rounds its whole sum at every step."""
    import numpy as np
    import torch
    from oracle import oracle as orc
    from paper_2110_10802_amd import binding as B
    from paper_2110_10802_amd.harness import DeviceBlock

    s = BlockShape(N=128, Cin=Cin, H=28, W=28, Cexp=3 * Cin, Cse=1, Cout=Cin, k=3, stride=1, has_expand=True, residual=True,
                   has_se=False)
    whole = rule("_ZN3mbk15eval_block_planERKNS_7DwShapeEii", BOOL, C.POINTER(DwShape), INT, INT)
    assert whole(C.byref(dw_shape(s.N, s.Cexp, s.H, s.W, s.k, 1)), Cin, Cin)
    t = make_block_inputs(s, seed=Cin)
    rng = np.random.default_rng(Cin)
    for i, c in ((1, s.Cexp), (2, s.Cexp), (3, s.Cout)):
        t[f"bn{i}_mean"] = (0.3 * rng.standard_normal(c)).astype(np.float32)
        t[f"bn{i}_var"] = rng.uniform(0.5, 2.0, c).astype(np.float32)
    blk = DeviceBlock(s, t)
    x = blk.to_device(t["x"])
    one = blk.forward_eval(x).clone()
    B.mbconv_forward_eval(blk.desc, blk.params, blk.running, x, x, blk.eval_ws, 0)
    torch.cuda.synchronize()
    ref = torch.from_numpy(np.asarray(orc.mbconv_forward_eval(s, t))).to(blk.device)
    error = [float((y.double() - ref).norm() / ref.norm()) for y in (one, x)]
    print(f"[eval] {Cin} channels: one launch {error[0]:.3e}, separate {error[1]:.3e}", flush=True)
    assert error[0] <= error[1]
