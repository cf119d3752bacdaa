"""Squeeze-and-excitation forward of 128 channels and more: rows whose length is no multiple of four are
read in overlapping pieces, and what two threads read counts once also where it is infinite.  Against
the oracle at the tolerances of parity_util."""
import numpy as np
import pytest

from mbconv_inputs import BlockShape, make_block_inputs
from oracle import oracle as orc
from parity_util import TOL, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("what", ["finite", "se_b1", "se_w1"])
@pytest.mark.parametrize("C,Cse", [(128, 4), (130, 6), (251, 9), (515, 33), (1154, 50), (2047, 63)])
def test_gate_matches_oracle(C, Cse, what):
    import torch
    from paper_2110_10802_amd.harness import DeviceBlock, to_numpy

    s = BlockShape(N=2, Cin=C, H=4, W=4, Cexp=C, Cse=Cse, Cout=16, k=3, stride=1, has_expand=False)
    t = make_block_inputs(s, seed=C + Cse)
    for i, c in ((2, s.Cexp), (3, s.Cout)):
        t[f"bn{i}_mean"], t[f"bn{i}_var"] = np.zeros(c, np.float32), np.ones(c, np.float32)
    if what == "se_b1":  # an infinite squeezed value: gates of zero and one
        t["se_b1"] = t["se_b1"].copy()
        t["se_b1"][Cse - 2] = np.inf
    elif what == "se_w1":  # likewise, by a weight in the columns that two lanes read
        t["se_w1"] = t["se_w1"].reshape(Cse, C).copy()
        t["se_w1"][1, C - 2] = np.inf
        t["bn2_beta"] = t["bn2_beta"].copy()
        t["bn2_beta"][C - 2] = 50.0  # its mean is above zero
    print(f"[se] {C}->{Cse} {what}", flush=True)
    blk = DeviceBlock(s, t)
    got = to_numpy(blk.forward_eval(blk.to_device(t["x"])))
    torch.cuda.synchronize()
    with np.errstate(all="ignore"):
        ref = orc.mbconv_forward_eval(s, t)
    assert np.all(np.isfinite(ref))
    assert rel_err(got, ref) <= TOL["f32"]["fwd"]


@pytest.mark.parametrize("N,C,Cse", [(33, 300, 8), (86, 514, 12), (129, 1030, 7), (300, 640, 20)])
def test_slices_of_any_batch(N, C, Cse):
    """Five, two, one and one slices of an image's channels; more than 256 channels go in rounds."""
    import torch
    from paper_2110_10802_amd.harness import DeviceBlock, to_numpy

    s = BlockShape(N=N, Cin=C, H=1, W=1, Cexp=C, Cse=Cse, Cout=16, k=3, stride=1, has_expand=False)
    t = make_block_inputs(s, seed=N)
    for i, c in ((2, s.Cexp), (3, s.Cout)):
        t[f"bn{i}_mean"], t[f"bn{i}_var"] = np.zeros(c, np.float32), np.ones(c, np.float32)
    print(f"[se] {N} x {C}->{Cse}", flush=True)
    blk = DeviceBlock(s, t)
    got = to_numpy(blk.forward_eval(blk.to_device(t["x"])))
    torch.cuda.synchronize()
    assert rel_err(got, orc.mbconv_forward_eval(s, t)) <= TOL["f32"]["fwd"]
