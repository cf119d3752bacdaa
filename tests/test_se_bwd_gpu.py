"""Squeeze-and-excitation backward: rows of W2 read in overlapping pieces, tiles of sixteen channels and squeezed
channels that are not full, batches of less than, exactly and more than a round of 64 images, and the plain
kernels of few channels, against the oracle at the tolerances of parity_util."""
import pytest

from mbconv_inputs import BlockShape, make_block_inputs
from oracle import oracle as orc
from parity_util import compare_block, run_gpu_block
from route_util import se_bwd_tiled

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,C,Cse", [(2, 160, 4), (64, 70, 5), (65, 170, 17), (3, 787, 33), (130, 161, 6),
                                     (2, 1154, 63), (9, 200, 64), (7, 60, 4), (6, 300, 3), (4, 40, 70)])
def test_gradients_match_oracle(N, C, Cse):
    s = BlockShape(N=N, Cin=C, H=4, W=4, Cexp=C, Cse=Cse, Cout=16, k=3, stride=1, has_expand=False)
    t = make_block_inputs(s, seed=C + Cse)
    assert se_bwd_tiled(N, C, Cse) == ((C, Cse) not in ((60, 4), (300, 3), (40, 70)))
    print(f"[se bwd] {s}", flush=True)
    res, blk = run_gpu_block(s, t)
    f, b = orc.mbconv_step(s, t)
    compare_block(s, t, res, f, b, blk)


def test_infinite_squeezed_gradient_stays_infinite():
    # One squeezed channel of five has an infinite gradient; it reaches one channel through a weight that is not zero, and
    # that channel's sums are infinite then, not NaN: what fills up the fours of the squeezed channels is left out.
    import numpy as np
    C = 176
    s = BlockShape(N=1, Cin=C, H=4, W=4, Cexp=C, Cse=5, Cout=16, k=3, stride=1, has_expand=False)
    t = make_block_inputs(s, seed=1)
    t["se_w1"][4] = 0.0
    t["se_w1"][4, 7] = 1.0
    t["se_b1"][4] = 0.0
    t["bn2_gamma"][7] = t["bn2_beta"][7] = 0.0  # z[7] = 0, so q[4] = 0: no effect on the gate, swish'(0) = 1/2
    t["se_w2"][:, 4] = 0.0
    t["se_w2"][11, 4] = 3e38  # one infinite term: none of the other sign to cancel it
    t["dout"] *= 100.0
    print(f"[se bwd] {s}", flush=True)
    res, blk = run_gpu_block(s, t)
    assert np.isinf(res["grads"]["bn2_beta"][7])
