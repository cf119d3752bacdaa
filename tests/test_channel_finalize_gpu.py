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
    # several rounds of images per workgroup, the last one short, planes of four and of three elements
    "rounds": _s(N=70, Cin=48, H=2, W=2, Cexp=1100, Cout=48),
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
