"""Weight gradients of bf16 storage on the bf16 matrix cores: tiles of 128 and 64 rows, a narrow first operand
(the transposed product), ragged channel counts, a last chunk that is not full, one launch for both gradients
and two, against the oracle at the tolerances of parity_util."""
import pytest

from mbconv_inputs import BlockShape, make_block_inputs
from oracle import oracle as orc
from parity_util import compare_block, run_gpu_block
from route_util import block_wgrad_kernels

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,Cin,Cexp,Cout,H,stride", [
    (11, 112, 300, 70, 6, 1),   # 128-row tiles, chunks that span images
    (7, 64, 264, 60, 8, 1),     # 64-row tiles, and the swapped form
    (3, 37, 261, 130, 10, 1),   # ragged channel counts
    (5, 72, 288, 24, 12, 1),    # at most 32 rows on one side
    (4, 80, 320, 96, 14, 2),    # 14x14 -> 7x7: one of the two gradients
])
def test_matches_oracle(N, Cin, Cexp, Cout, H, stride):
    s = BlockShape(N=N, Cin=Cin, H=H, W=H, Cexp=Cexp, Cse=8, Cout=Cout, k=3, stride=stride, has_expand=True,
                   residual=False, dtype="bf16")
    assert block_wgrad_kernels(s) == (("rd" if stride == 2 else "x3"), "x3")
    t = make_block_inputs(s, seed=Cexp)
    print(f"[wgrad bf16] {s}", flush=True)
    res, blk = run_gpu_block(s, t)
    f, b = orc.mbconv_step(s, t)
    compare_block(s, t, res, f, b, blk)
