"""The fp32 MFMA weight gradients (odd planes of at most 64 pixels, skinny blocks on odd planes and, with more than 256
channels on the other side, on even ones, bf16 storage on odd planes): ragged tiles of 64 rows, chunks that span images, a last
chunk that is not full, one launch for both gradients and two, against the oracle at the tolerances of
parity_util."""
import pytest

from mbconv_inputs import BlockShape, make_block_inputs
from oracle import oracle as orc
from parity_util import compare_block, run_gpu_block
from route_util import block_wgrad_kernels

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,Cin,Cexp,Cout,H,W,stride,dtype", [
    (9, 48, 130, 70, 7, 7, 1, "f32"),     # both gradients in one launch, ragged tiles
    (33, 40, 66, 40, 5, 3, 1, "f32"),     # several images to a chunk
    (70, 36, 40, 44, 1, 1, 1, "f32"),     # planes of one pixel
    (5, 20, 72, 24, 13, 11, 1, "f32"),    # skinny sides, odd plane
    (6, 40, 80, 48, 14, 14, 2, "f32"),    # 14x14 -> 7x7: one of the two gradients
    (12, 40, 96, 56, 7, 7, 1, "bf16"),
    (6, 33, 70, 41, 8, 8, 1, "bf16"),     # (the kernel for few channels on even planes)
    (7, 24, 301, 20, 10, 10, 1, "f32"),   # runs of four, both gradients in one launch
    (5, 30, 258, 64, 6, 6, 1, "f32"),     # one of the two
    (4, 40, 64, 64, 15, 15, 1, "bf16"),
])
def test_matches_oracle(N, Cin, Cexp, Cout, H, W, stride, dtype):
    s = BlockShape(N=N, Cin=Cin, H=H, W=W, Cexp=Cexp, Cse=4, Cout=Cout, k=3, stride=stride, has_expand=True,
                   residual=False, dtype=dtype)
    want = ("lt", "lt") if (H, dtype) == (8, "bf16") else ("rd", "x3") if stride == 2 else ("x3", "rd") if H == 6 else ("rd", "rd")
    assert block_wgrad_kernels(s) == want
    t = make_block_inputs(s, seed=N)
    print(f"[wgrad_rd] {s}", flush=True)
    res, blk = run_gpu_block(s, t)
    f, b = orc.mbconv_step(s, t)
    compare_block(s, t, res, f, b, blk)
