"""Small planes: the kernels that finalise a channel's normalisation themselves (pool, BN3's
elementwise pass, BN3's backward sums), at the edges of their splits, against the oracle at the
tolerances of parity_util."""
import pytest

from mbconv_inputs import BlockShape, make_block_inputs
from oracle import oracle as orc
from parity_util import compare_block, run_gpu_block

pytestmark = pytest.mark.gpu


def _s(**kw):
    base = dict(N=17, Cin=40, H=6, W=6, Cexp=80, Cse=10, Cout=40, k=3, stride=1, residual=True)
    base.update(kw)
    return BlockShape(**base)


SHAPES = {
    "last_group_of_one_image": _s(),
    "odd_plane": _s(N=33, H=5, W=7),
    "one_element_planes": _s(N=5, H=1, W=1, Cexp=96),
    # two rounds of images per workgroup, the last one short, planes of four and of three elements
    "rounds": _s(N=55, Cin=48, H=2, W=2, Cexp=1100, Cout=48),
    "rounds_odd": _s(N=35, Cin=48, H=1, W=3, Cexp=1100, Cout=48),
    # the largest plane of 16 lanes, the smallest and the largest of a wavefront, the next one
    "plane_256": _s(N=3, H=16, W=16),
    "plane_258": _s(N=3, H=6, W=43),
    "plane_1024": _s(N=5, H=32, W=32, Cout=24, residual=False),
    "plane_1025": _s(N=2, H=25, W=41),
    # the most images that BN3's backward sums take in one launch, and one more
    "images_128": _s(N=128, H=4, W=4),
    "images_129": _s(N=129, H=4, W=4),
    "images_33": _s(N=33, H=17, W=17),
    # channels times images (in groups of sixteen on small planes) where the BN3 step is inside the last
    # pass for the last time, and where it is a launch
    "bn3_inside": _s(N=2032, Cin=16, H=2, W=2, Cexp=32, Cse=4, Cout=40, residual=False),
    "bn3_launch": _s(N=2064, Cin=16, H=2, W=2, Cexp=32, Cse=4, Cout=40, residual=False),
    # more partial sums than the finalise launch adds in one round, no multiple of it
    "many_partials": _s(N=2064, Cin=16, H=4, W=5, Cexp=32, Cse=4, Cout=40, residual=False),
    # the same for BN2 and the pool (images in pairs of groups); weight images written by either
    "bn2_inside": _s(N=96, Cin=32, H=2, W=2, Cexp=1024, Cse=8, Cout=48, residual=False),
    "bn2_launch": _s(N=97, Cin=32, H=2, W=2, Cexp=1024, Cse=8, Cout=48, residual=False),
    "no_se": _s(has_se=False, Cse=1, activation="relu6"),
    "bf16": _s(N=19, H=10, W=10, dtype="bf16"),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_block_matches_oracle(name):
    s = SHAPES[name]
    t = make_block_inputs(s, seed=29)
    print(f"[channel] {name} {s}", flush=True)
    res, blk = run_gpu_block(s, t)
    f, b = orc.mbconv_step(s, t)
    compare_block(s, t, res, f, b, blk)


def _occurs(s, step):
    """Whether a training forward pass has that step: its events are recorded anew."""
    import torch
    from paper_2110_10802_amd import binding as B
    from paper_2110_10802_amd.harness import DeviceBlock
    t = make_block_inputs(s, seed=30)
    blk = DeviceBlock(s, t)
    x = blk.to_device(t["x"])
    blk.forward(x)
    big = torch.empty(1 << 27, device="cuda:0")
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    big.zero_()  # (half a gigabyte: longer than any step below)
    e1.record()
    torch.cuda.synchronize()
    before = e0.elapsed_time(e1)
    B.mbconv_forward_probed(blk.desc, blk.params, blk.running, x, blk.out, blk.saved, blk.scratch, 0,
                            B.Probe(B.STEPS[step], e0.cuda_event, e1.cuda_event))
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) != before


@pytest.mark.parametrize("shape", [dict(H=2, W=2, N=2064), dict(H=6, W=43, N=520), dict(H=40, W=40, N=130)])
def test_bn3_step_is_a_launch_for_large_batches(shape):
    """Every workgroup of the last pass would read all partial sums of its channel."""
    s = _s(**{**dict(Cin=16, Cexp=32, Cse=4, Cout=40, residual=False), **shape})
    assert _occurs(s, "bn3_finalize")
    assert not _occurs(s.with_batch(s.N // 2), "bn3_finalize")


@pytest.mark.parametrize("shape", [dict(H=2, W=2, N=97), dict(H=6, W=43, N=25)])
def test_bn2_step_is_a_launch_for_large_batches(shape):
    s = _s(**{**dict(Cin=32, Cexp=1024, Cse=4, Cout=16, residual=False), **shape})
    assert _occurs(s, "bn2_finalize")
    assert not _occurs(s.with_batch(s.N - 1), "bn2_finalize")


def test_constant_channel_has_no_variance():
    """The finalise launch of BN1 (the storing policy's) over 49 equal values: their mean and no variance, so that rstd is
    1 / sqrt(eps); 1/49 is not a number of 53 bits, and 49 times its nearest one is not 1."""
    import torch
    from paper_2110_10802_amd import binding as B
    from paper_2110_10802_amd.harness import DeviceBlock

    s = _s(N=1, Cin=16, H=7, W=7, Cexp=96, Cse=4, Cout=16, residual=False, eps=1e-12)
    t = make_block_inputs(s, seed=30)
    t["w_expand"] = t["w_expand"] * 0 + 64
    blk = DeviceBlock(s, t, B.MBCONV_STORE)
    x = torch.ones((s.N, s.Cin, s.H, s.W), device=blk.device)
    blk.forward(x)
    torch.cuda.synchronize()
    mean, rstd = blk.saved_tensor("bn1")[2:]
    assert (mean == 1024).all()
    assert abs(rstd * 1e-6 - 1).max() < 1e-6  # (fp32 holds eps to 6e-8)
