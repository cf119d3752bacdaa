"""The expansion conv of small launches (a workgroup per 16 rows x 32 pixels, a wavefront per 32 input channels): one
step and six, a last step that is not full, rows and pixels past the end, even and odd planes, chunks that span images,
sizes on either side of the rule, against the oracle at the tolerances of parity_util."""
import pytest

from mbconv_inputs import BlockShape, make_block_inputs
from oracle import oracle as orc
from parity_util import compare_block, run_gpu_block
from route_util import xs_chunks

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,Cin,Cexp,H", [
    (2, 8, 40, 12),      # one step, a quarter of it
    (3, 32, 69, 9),      # a whole step, rows past the end, odd plane
    (5, 40, 240, 7),     # two steps, chunks that span images
    (1, 104, 312, 17),   # a last step that is not full
    (4, 192, 1152, 7),   # six steps
    (18, 96, 576, 14),   # 11988 wavefronts, the most that the rule takes; with another image it does not
    (19, 96, 576, 14),
])
def test_matches_oracle(N, Cin, Cexp, H):
    s = BlockShape(N=N, Cin=Cin, H=H, W=H, Cexp=Cexp, Cse=8, Cout=24, k=3, stride=1, has_expand=True, residual=False,
                   dtype="f32")
    assert (xs_chunks(s) is not None) == (N != 19)
    t = make_block_inputs(s, seed=Cin)
    print(f"[conv_xs] {s}", flush=True)
    res, blk = run_gpu_block(s, t)
    f, b = orc.mbconv_step(s, t)
    compare_block(s, t, res, f, b, blk)
