"""The fused backward of an expansion conv of at most 16 channels that computes the conv's output again
(planes of at least 512 chunks of 32 pixels in all): odd counts of 16-channel tiles, ragged channel counts,
a last chunk that is not full, with and without the residual, against the oracle at the tolerances of
parity_util."""
import ctypes as C

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


class Operand(C.Structure):
    _fields_ = [("p0", C.c_void_p), ("p1", C.c_void_p), ("c0", C.c_void_p), ("c1", C.c_void_p), ("c2", C.c_void_p),
                ("gate", C.c_void_p), ("pro", C.c_int)]


@pytest.mark.parametrize("N,Cin,Cexp,H,mean", [(16, 16, 96, 64, 5.0), (24, 9, 36, 64, 5.0), (8, 16, 192, 64, 5.0),
                                               (8, 8, 24, 32, 5.0), (16, 16, 96, 64, 0.0), (96, 12, 36, 64, 0.0)])
def test_error_is_that_of_values_rounded_once(N, Cin, Cexp, H, mean):
    """Channels that are far from centred: the gradients' relative error against 64 bits is at most four times that of a
    computation that rounds e and de = c0*dy + c1*e + c2 to fp32 once each and is exact otherwise, and 2^-24 for each
    time that a wavefront adds a chunk's product to its accumulators (they are 2048 at most, a chunk 32 pixels).  An
    error of e that all pixels share would be tens of times as large in the weight gradient.  The mean over the pixels of the
    data gradient's error is an eighth of 2^-25 of it at most: roundings to nearest leave it at their size over the
    square root of the pixels, a truncation of the same sign in every pixel at some 2^-26."""
    import torch
    from paper_2110_10802_amd import binding as B
    launch = getattr(B.load(), "_ZN3mbk19launch_bwd1x1_fusedEbiiiiRKNS_7OperandEPKvS4_PvS4_PfPiP12ihipStream_t")
    launch.argtypes = [C.c_bool] + 4 * [C.c_int] + [C.POINTER(Operand)] + 5 * [C.c_void_p] + [C.POINTER(C.c_int), C.c_void_p]
    gen = torch.Generator(device="cuda").manual_seed(Cexp)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device="cuda")
    x = normal(N, Cin, H * H) + mean * normal(1, Cin, 1)
    w = normal(Cexp, Cin) * (2 / Cin) ** 0.5
    e64 = torch.matmul(w.double(), x.double())
    mu, rstd = e64.mean((0, 2)), (e64.var((0, 2), unbiased=False) + 1e-3).rsqrt()
    gamma = 1 + 0.1 * normal(Cexp).double()
    xhat = (e64 - mu[:, None]) * rstd[:, None]
    y = xhat * gamma[:, None]
    sig = torch.sigmoid(y)
    dy = ((normal(N, Cexp, H * H).double() + 0.3) * (sig * (1 + y * (1 - sig)))).float()
    m = N * H * H
    c1 = -gamma * rstd * rstd * (dy.double() * xhat).sum((0, 2)) / m
    c = torch.stack([gamma * rstd, c1, -gamma * rstd * dy.double().sum((0, 2)) / m - c1 * mu]).float()

    def gradients(e, rounded):
        k = c.double()
        de = k[0][:, None] * dy.double() + (k[1][:, None] * e + k[2][:, None])
        de = de.float().double() if rounded else de
        return (sum(de[n] @ x[n].double().t().contiguous() for n in range(N)),
                torch.matmul(w.double().t().contiguous(), de))
    exact, once = gradients(e64, False), gradients(e64.float().double(), True)
    e32 = e64.float()
    op = Operand(dy.data_ptr(), e32.data_ptr(), c[0].data_ptr(), c[1].data_ptr(), c[2].data_ptr(), None, 2)
    dx, partial, splits = torch.empty_like(x), torch.empty(640 * Cexp * Cin, device="cuda"), C.c_int(0)
    print(f"[bwd1x1_re] {N} x {Cin} -> {Cexp}, {H}x{H}, mean {mean}", flush=True)
    assert launch(False, N, Cexp, Cin, H * H, C.byref(op), x.data_ptr(), w.data_ptr(), dx.data_ptr(), None,
                  partial.data_ptr(), C.byref(splits), None) == 0
    torch.cuda.synchronize()
    dw = partial[:splits.value * Cexp * Cin].view(splits.value, Cexp, Cin).double().sum(0)
    for got, ex, on in zip((dw, dx.double()), exact, once):
        err, ref = float((got - ex).norm() / ex.norm()), float((on - ex).norm() / ex.norm())
        print(f"  {err:.2e}, rounded once {ref:.2e}", flush=True)
        assert err <= 4 * ref + 2.0 ** -24 * -(-m // (32 * 2048))
    offset = (dx.double() - exact[1]).mean((0, 2)).square().mean().sqrt() / exact[1].square().mean().sqrt()
    print(f"  offset {float(offset):.2e}", flush=True)
    assert float(offset) <= 2.0 ** -28
