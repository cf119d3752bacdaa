"""Depthwise chain on small planes: both choices of the number of image ranges, and ranges of unequal
length, against the oracle at the tolerances of parity_util."""
import pytest

from mbconv_inputs import BlockShape, make_block_inputs
from oracle import oracle as orc
from parity_util import compare_block, run_gpu_block

pytestmark = pytest.mark.gpu

SHAPES = {
    # 4096/672 lies between six and seven ranges: seven forward, six backward, the last one short
    "fewer": BlockShape(N=28, Cin=16, H=14, W=14, Cexp=672, Cse=4, Cout=16, k=5, stride=1, residual=True),
    # ... between three and four: four
    "more": BlockShape(N=66, Cin=16, H=7, W=7, Cexp=1152, Cse=4, Cout=16, k=3, stride=1, residual=True),
    # 3x3: six both ways in fp32, seven in bf16
    "3x3": BlockShape(N=56, Cin=16, H=14, W=14, Cexp=672, Cse=4, Cout=16, k=3, stride=1, residual=True),
    "3x3_bf16": BlockShape(N=56, Cin=16, H=14, W=14, Cexp=672, Cse=4, Cout=16, k=3, stride=1, residual=True, dtype="bf16"),
    # no expansion conv: the filter gradient's own reduction
    "noexpand": BlockShape(N=56, Cin=672, H=14, W=14, Cexp=672, Cse=4, Cout=16, k=5, stride=1, has_expand=False),
    # more channels than wavefronts: one range
    "one": BlockShape(N=9, Cin=8, H=5, W=5, Cexp=4200, Cse=2, Cout=8, k=3, stride=1),
    "bf16": BlockShape(N=28, Cin=16, H=14, W=14, Cexp=672, Cse=4, Cout=16, k=5, stride=1, residual=True, dtype="bf16"),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_block_matches_oracle(name):
    s = SHAPES[name]
    t = make_block_inputs(s, seed=31)
    print(f"[dw ranges] {name} {s}", flush=True)
    res, blk = run_gpu_block(s, t)
    f, b = orc.mbconv_step(s, t)
    compare_block(s, t, res, f, b, blk)
