"""The fp32 MFMA weight gradient of operands of more than 4 GiB, which its 32-bit byte offsets reach from each split's
first image on: against the same sum in 64 bits, held to 2^-24 times the sum of the terms' sizes, times 64 roundings (a
split adds some 22 000 terms, the second stage 500 splits; their errors are of either sign)."""
import ctypes as C

import pytest
import torch

from paper_2110_10802_amd import binding as B

pytestmark = pytest.mark.gpu


class Operand(C.Structure):
    _fields_ = [("p0", C.c_void_p), ("p1", C.c_void_p), ("c0", C.c_void_p), ("c1", C.c_void_p), ("c2", C.c_void_p),
                ("gate", C.c_void_p), ("pro", C.c_int)]


def test_more_than_4_gib():
    launch = getattr(B.load(), "_ZN3mbk10launch_wgrEbiiiiRKNS_7OperandES2_PfPiP12ihipStream_t")
    launch.argtypes = [C.c_bool] + 4 * [C.c_int] + 2 * [C.POINTER(Operand)] + [C.c_void_p, C.POINTER(C.c_int), C.c_void_p]
    N, Ma, Mb, HW = 3500, 96, 7, 57 * 57
    gen = torch.Generator(device="cuda").manual_seed(1)
    dy = torch.randn(N, Ma, HW, generator=gen, device="cuda")
    x = torch.randn(N, Mb, HW, generator=gen, device="cuda")
    assert dy.numel() * 4 > 1 << 32
    c = torch.randn(3, Ma, generator=gen, device="cuda")
    partial = torch.full((640 * Ma * Mb,), float("nan"), device="cuda")
    splits = C.c_int(0)
    u = Operand(dy.data_ptr(), dy.data_ptr(), c[0].data_ptr(), c[1].data_ptr(), c[2].data_ptr(), None, 2)
    v = Operand(x.data_ptr(), None, None, None, None, None, 0)
    print(f"[wgrad_rd] {N} x {Ma} x {HW}", flush=True)
    assert launch(False, N, Ma, Mb, HW, C.byref(u), C.byref(v), partial.data_ptr(), C.byref(splits), None) == 0
    torch.cuda.synchronize()
    got = partial[:splits.value * Ma * Mb].view(splits.value, Ma, Mb).double().sum(0)
    want, size = torch.zeros_like(got), torch.zeros_like(got)
    c = c.double()
    for n in range(0, N, 100):
        d = dy[n:n + 100].double()
        d = ((c[0] + c[1])[:, None] * d + c[2][:, None]).transpose(0, 1).reshape(Ma, -1)
        e = x[n:n + 100].double().permute(0, 2, 1).reshape(-1, Mb).contiguous()
        want += d @ e
        size += d.abs() @ e.abs()
    assert bool(((got - want).abs() <= 64 * 2.0 ** -24 * size).all())
