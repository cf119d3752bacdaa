"""The 1x1 convolutions whose contraction is split over a workgroup's wavefronts (conv_xk): block
shapes at the edges of its tiles, against the oracle at the tolerances of parity_util."""
import numpy as np
import pytest

from mbconv_inputs import BlockShape, make_block_inputs
from oracle import oracle as orc
from parity_util import TOL, compare_block, metric_for, run_gpu_block

pytestmark = pytest.mark.gpu


def _s(**kw):
    base = dict(N=2, Cin=48, H=8, W=8, Cexp=288, Cse=12, Cout=48, k=3, stride=1, residual=True)
    base.update(kw)
    return BlockShape(**base)


SHAPES = {
    # contraction and rows that are no multiple of eight; an odd plane; a last chunk of 13 pixels
    "ragged_channels": _s(Cin=43, Cexp=259, Cout=43, H=5, W=9),
    # several images in one 32-pixel chunk (their gates wait in LDS), even and odd planes
    "images_per_chunk": _s(N=9, H=2, W=3),
    "images_per_chunk_odd": _s(N=11, H=1, W=3, residual=False, Cout=40),
    # one image of few pixels: two row tiles per workgroup, eight wavefronts along the contraction
    "one_image": _s(N=1, Cin=192, Cexp=1152, Cout=200, H=7, W=7, residual=False, k=5),
    # one 32-deep step for a single wavefront; rows past the weight image's last tile
    "short_contraction": _s(Cin=24, Cexp=56, Cout=33, H=7, W=9, residual=False),
    # eight, seven and five row tiles per slab, more than one slab
    "slab_8": _s(N=3, Cin=40, Cexp=240, Cout=128, H=14, W=14, residual=False),
    "slab_7": _s(N=70, Cin=56, Cexp=224, Cout=112, H=12, W=16, residual=False),
    "slab_5": _s(N=41, Cin=80, Cexp=320, Cout=320, H=9, W=9, residual=False),
    # no expansion conv; a stride from an even into an odd plane; squeezed channels that are no multiple of four
    "noexpand": _s(Cin=72, Cexp=72, Cse=7, Cout=48, has_expand=False, residual=False),
    "stride2_into_7x7": _s(N=3, Cin=48, Cexp=288, Cout=64, H=14, W=14, stride=2, residual=False),
    "se_ragged": _s(N=3, Cin=42, Cexp=250, Cse=11, Cout=42, H=5, W=5),
    "many_workgroups": _s(N=40, Cin=40, Cexp=160, Cout=40, H=24, W=24),
    # a short contraction on many pixels: one wavefront, all of the steps
    "one_wavefront": _s(N=57, Cin=40, Cexp=80, Cse=10, Cout=40, H=24, W=25),
    "relu6": _s(N=3, H=7, W=7, activation="relu6", has_se=False, Cse=1),
    # bf16: the largest forward launch (2133 chunks of three row tiles), the next one and a contraction too
    # short (both conv_bf)
    "bf16_6399_tiles": _s(N=79, Cin=16, Cexp=128, Cse=8, Cout=40, H=24, W=36, dtype="bf16", residual=False),
    "bf16_6432_tiles": _s(N=67, Cin=16, Cexp=128, Cse=8, Cout=40, H=32, W=32, dtype="bf16", residual=False),
    "bf16_short": _s(N=6, Cin=96, Cexp=96, Cse=8, Cout=40, H=12, W=12, dtype="bf16", residual=False,
                     has_expand=False),
    "bf16": _s(N=16, Cin=64, Cexp=384, Cse=16, Cout=96, H=10, W=10, dtype="bf16", residual=False),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_block_matches_oracle(name):
    s = SHAPES[name]
    t = make_block_inputs(s, seed=17)
    print(f"[conv_xk] {name} {s}", flush=True)
    res, blk = run_gpu_block(s, t)
    f, b = orc.mbconv_step(s, t)
    compare_block(s, t, res, f, b, blk)


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("name", ["one_image", "images_per_chunk", "slab_8", "bf16"])
def test_eval_matches_oracle(name, policy):
    """BN3 and the residual in the epilogue; evaluation mode ignores the policy."""
    import torch
    from paper_2110_10802_amd.harness import DeviceBlock, to_numpy

    s = SHAPES[name]
    t = make_block_inputs(s, seed=18)
    rng = np.random.default_rng(19)
    for i, c in ((1, s.Cexp), (2, s.Cexp), (3, s.Cout)):
        t[f"bn{i}_mean"] = (0.3 * rng.standard_normal(c)).astype(np.float32)
        t[f"bn{i}_var"] = (0.5 + rng.random(c)).astype(np.float32)
    print(f"[conv_xk/eval] {name} policy={policy}", flush=True)
    blk = DeviceBlock(s, t, policy=policy)
    out = to_numpy(blk.forward_eval(blk.to_device(t["x"])))
    torch.cuda.synchronize()
    assert metric_for(s)(out, orc.mbconv_forward_eval(s, t)) <= TOL[s.dtype]["fwd"]


def _small(**kw):
    return _s(**{**dict(Cin=43, Cexp=258, Cout=43, H=9, W=5, activation="relu6", has_se=False, Cse=1), **kw})


INFINITE = {
    # (shape, tensor, {index: value}): in x with ReLU6 (the clamp makes everything behind it finite, the
    # residual carries the infinities), the largest finite values (their bf16 rounding is infinite), in weights
    "x": (_small(), "x", {(0, 3, 2, 2): np.inf, (1, 2, 1, 1): -np.inf}),
    "x_largest": (_small(), "x", {(1, 5, 4, 4): np.finfo(np.float32).max, (0, 7, 0, 0): -3.4e38}),
    "w_expand": (_small(), "w_expand", {(7, 3): np.inf}),
    "w_proj": (_small(), "w_proj", {(7, 3): -np.inf}),
    # the last channel of a contraction that ends inside a 32-deep step (the step's other rows repeat it)
    "last_channel": (_s(Cin=72, Cexp=72, Cout=48, has_expand=False, residual=False, has_se=False, Cse=1, H=5, W=7),
                     "x", {(0, 71, 2, 2): np.inf}),
    "last_channel_bf16": (_s(N=1, Cin=136, Cexp=136, Cout=48, has_expand=False, residual=False, has_se=False,
                             Cse=1, dtype="bf16"), "x", {(0, 135, 2, 2): np.inf}),
}


@pytest.mark.parametrize("name", list(INFINITE))
def test_infinite_operands(name):
    """Evaluation mode: infinities and NaN where 64-bit arithmetic has them, finite values elsewhere."""
    import torch
    from paper_2110_10802_amd.harness import DeviceBlock, to_numpy

    s, what, values = INFINITE[name]
    t = make_block_inputs(s, seed=20)
    t["w_dw"] = np.abs(t["w_dw"])  # (no sums of opposite infinities)
    for i, c in ((1, s.Cexp), (2, s.Cexp), (3, s.Cout)):
        t[f"bn{i}_mean"], t[f"bn{i}_var"] = np.zeros(c, np.float32), np.ones(c, np.float32)
    t[what] = t[what].copy()
    for at, v in values.items():
        t[what][at] = v
    print(f"[conv_xk/inf] {name}", flush=True)
    blk = DeviceBlock(s, t)
    got = to_numpy(blk.forward_eval(blk.to_device(t["x"]))).astype(np.float64)
    torch.cuda.synchronize()
    with np.errstate(all="ignore"):
        ref = orc.mbconv_forward_eval(s, t)
    ref = np.where(np.abs(ref) > np.finfo(np.float32).max, np.sign(ref) * np.inf, ref)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(np.where(np.isinf(got), np.sign(got), 0), np.where(np.isinf(ref), np.sign(ref), 0))
    ok = np.isfinite(ref) & (np.abs(ref) < 1e30)
    assert ok.sum() > ref.size // 2
    assert metric_for(s)(got[ok], ref[ok]) <= TOL[s.dtype]["fwd"]
