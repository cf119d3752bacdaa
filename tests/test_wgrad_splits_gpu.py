"""Weight gradients of the 1x1 convolutions on the bf16 matrix cores: how tiles and splits of the
contraction are dealt out, and the forms of the sum over the splits, against the oracle at the
tolerances of parity_util."""
import pytest

from mbconv_inputs import BlockShape, make_block_inputs
from oracle import oracle as orc
from parity_util import compare_block, run_gpu_block

pytestmark = pytest.mark.gpu

SHAPES = {
    # seven splits of 27 tiles (no multiple of eight) and five of 45, planes of 81 pixels; sum with 256
    # lanes to a group
    "seven_splits": BlockShape(N=5, Cin=192, H=9, W=9, Cexp=1152, Cse=48, Cout=320, k=3, stride=1),
    # one split, fewer workgroups than the chip has XCDs
    "one_split": BlockShape(N=1, Cin=40, H=6, W=6, Cexp=240, Cse=10, Cout=48, k=3, stride=1),
    # 64-row tiles; many splits, the last one shorter
    "narrow_tile": BlockShape(N=37, Cin=64, H=12, W=12, Cexp=130, Cse=16, Cout=64, k=3, stride=1, residual=True),
    # more tiles than compute units
    "many_tiles": BlockShape(N=2, Cin=768, H=6, W=6, Cexp=5504, Cse=32, Cout=160, k=3, stride=1),
    # both gradients in one launch, the plane of one a multiple of four, the other's not; one and two
    # 64-row tiles, 128-row tiles halved
    "even_and_odd_plane": BlockShape(N=3, Cin=48, H=18, W=18, Cexp=288, Cse=12, Cout=80, k=3, stride=2),
    "even_and_odd_plane_wide": BlockShape(N=2, Cin=96, H=22, W=22, Cexp=384, Cse=24, Cout=144, k=3, stride=2),
    # rows of a tile that are padding, wavefront by wavefront
    "padding": BlockShape(N=9, Cin=72, H=14, W=14, Cexp=216, Cse=18, Cout=88, k=3, stride=1),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_block_matches_oracle(name):
    from paper_2110_10802_amd import binding as B
    s = SHAPES[name]
    for step in ("proj_wgrad", "expand_wgrad"):  # (a shape that another kernel serves tests nothing here)
        assert B.ENGINES[B.mbconv_step_engine(B.make_desc(s), B.STEPS[step])] == "mfma_bf16x3"
    t = make_block_inputs(s, seed=23)
    print(f"[wgrad] {name} {s}", flush=True)
    res, blk = run_gpu_block(s, t)
    f, b = orc.mbconv_step(s, t)
    compare_block(s, t, res, f, b, blk)
