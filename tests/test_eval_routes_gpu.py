"""Evaluation mode: the depthwise launch takes the normalisations' coefficients from the running statistics,
sums each plane for the squeeze, and its extra workgroups write what later kernels read.  One shape per
kernel and thread count, at ragged batches, with and without the SE stage and the expansion, against the
oracle at the tolerances of parity_util."""
import numpy as np
import pytest

from mbconv_inputs import BlockShape, make_block_inputs
from oracle import oracle as orc
from parity_util import TOL, metric_for

pytestmark = pytest.mark.gpu

# (N, Cexp, Cout, H, W, k, stride): depthwise kernel
SHAPES = {
    "dwr_7x7_four_planes": (5, 72, 40, 7, 7, 3, 1),
    "dwr_5x3_many_planes": (23, 40, 24, 5, 3, 5, 1),
    "dwr_14x14": (3, 96, 112, 14, 14, 5, 1),
    "dw4_16_wavefront": (3, 50, 24, 16, 16, 3, 1),
    "dw4_28_wavefront": (2, 66, 40, 28, 28, 5, 1),
    "dw4_56_workgroup": (1, 48, 40, 56, 56, 3, 1),
    "dw4_36_two_images": (3, 1024, 8, 36, 36, 3, 1),
    "dw4_68_1024_threads": (1, 66, 70, 68, 68, 5, 1),
    "dw2_14_row_of_16": (5, 90, 112, 14, 14, 5, 2),
    "dw2_30_ragged": (3, 48, 40, 30, 30, 3, 2),
    "dw2_56": (1, 48, 40, 56, 56, 5, 2),
    "dw2_112_1024_threads": (1, 40, 70, 112, 112, 3, 2),
    "dw_15_odd_stride_2": (3, 90, 70, 15, 15, 3, 2),
    "dw_67_odd_stride_2": (1, 40, 40, 67, 67, 5, 2),
}


@pytest.mark.parametrize("variant", ["se", "no_se", "no_expand", "bf16", "relu6_no_se"])
@pytest.mark.parametrize("name", list(SHAPES))
def test_matches_oracle(name, variant):
    import torch
    from paper_2110_10802_amd.harness import DeviceBlock, to_numpy

    N, Cexp, Cout, H, W, k, stride = SHAPES[name]
    expand = variant != "no_expand"
    s = BlockShape(N=N, Cin=16 if expand else Cexp, H=H, W=W, Cexp=Cexp, Cse=6, Cout=Cout, k=k, stride=stride,
                   has_expand=expand, residual=False, has_se="no_se" not in variant,
                   dtype="bf16" if variant == "bf16" else "f32",
                   activation="relu6" if "relu6" in variant else "swish")
    t = make_block_inputs(s, seed=len(name))
    rng = np.random.default_rng(7)
    for i, c in ((1, Cexp), (2, Cexp), (3, Cout)):
        t[f"bn{i}_mean"] = (0.3 * rng.standard_normal(c)).astype(np.float32)
        t[f"bn{i}_var"] = rng.uniform(0.5, 2.0, c).astype(np.float32)
    print(f"[eval] {name} {variant} {s}", flush=True)
    blk = DeviceBlock(s, t)
    got = to_numpy(blk.forward_eval(blk.to_device(t["x"])))
    torch.cuda.synchronize()
    assert metric_for(s)(got, orc.mbconv_forward_eval(s, t)) <= TOL[s.dtype]["fwd"]


def check(s, seed):
    import torch
    from paper_2110_10802_amd.harness import DeviceBlock, to_numpy

    t = make_block_inputs(s, seed=seed)
    rng = np.random.default_rng(7)
    for i, c in ((1, s.Cexp), (2, s.Cexp), (3, s.Cout)):
        t[f"bn{i}_mean"] = (0.3 * rng.standard_normal(c)).astype(np.float32)
        t[f"bn{i}_var"] = rng.uniform(0.5, 2.0, c).astype(np.float32)
    print(f"[eval] {s}", flush=True)
    blk = DeviceBlock(s, t)
    got = to_numpy(blk.forward_eval(blk.to_device(t["x"])))
    torch.cuda.synchronize()
    assert metric_for(s)(got, orc.mbconv_forward_eval(s, t)) <= TOL[s.dtype]["fwd"]


# The other side of the rule: coefficients by a launch of their own, the squeeze by the pool
AHEAD = {
    "image_no_se": (13, 61, 366, 76, 10, 5, 2, False),       # a launch for the expansion conv precedes it anyway
    "image_se": (13, 61, 366, 76, 10, 5, 2, True),           # (folded all the same: the pool is saved)
    "9x9_no_se": (41, 16, 1024, 24, 9, 3, 2, False),         # 41984 wavefronts
    "17x17_se_stride_2": (25, 16, 1000, 24, 17, 3, 2, True), # 100000 wavefronts
    "68x68_5x5": (5, 8, 208, 24, 68, 5, 1, False),           # 1024 threads, 16640 wavefronts: dw4, and dw2
    "68x68_5x5_stride_2": (5, 8, 208, 24, 68, 5, 2, False),
    "67x67_5x5_no_expand": (5, None, 208, 24, 67, 5, 1, False),
}


@pytest.mark.parametrize("name", list(AHEAD))
def test_coefficients_ahead(name):
    N, Cin, Cexp, Cout, H, k, stride, se = AHEAD[name]
    check(BlockShape(N=N, Cin=Cin or Cexp, H=H, W=H, Cexp=Cexp, Cse=6, Cout=Cout, k=k, stride=stride,
                     has_expand=Cin is not None, residual=False, has_se=se), len(name))
