"""The fused backward of an expansion conv of at most 16 channels that computes the conv's output again
(planes of at least 512 chunks of 32 pixels in all): odd counts of 16-channel tiles, ragged channel counts,
a last chunk that is not full, with and without the residual, against the oracle at the tolerances of
parity_util."""
import pytest

from mbconv_inputs import BlockShape, make_block_inputs
from oracle import oracle as orc
from parity_util import compare_block, run_gpu_block

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,Cin,Cexp,H,W,residual", [
    (8, 16, 96, 46, 46, True),    # 529 chunks, the last one of four pixels
    (6, 13, 52, 56, 52, False),   # four tiles, the last of four rows
    (17, 8, 48, 32, 32, True),    # three tiles
    (66, 3, 12, 16, 16, False),   # one tile
    (8, 9, 108, 48, 46, False),   # seven tiles
    (4, 16, 192, 64, 66, True),   # twelve tiles
    (70, 5, 20, 50, 48, False),   # more than 2048 chunks: eight wavefronts a workgroup
])
def test_matches_oracle(N, Cin, Cexp, H, W, residual):
    s = BlockShape(N=N, Cin=Cin, H=H, W=W, Cexp=Cexp, Cse=2, Cout=Cin if residual else 8, k=3, stride=1,
                   has_expand=True, residual=residual)
    from paper_2110_10802_amd import binding as B
    assert B.ENGINES[B.mbconv_step_engine(B.make_desc(s), B.STEPS["expand_dgrad"])] == "mfma_bf16x3"
    t = make_block_inputs(s, seed=Cexp)
    print(f"[bwd1x1_re] {s}", flush=True)
    res, blk = run_gpu_block(s, t)
    f, b = orc.mbconv_step(s, t)
    compare_block(s, t, res, f, b, blk)
