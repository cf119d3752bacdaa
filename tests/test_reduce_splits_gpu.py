"""The second stage of split reductions, through the gradients of layer normalisation's weights: 4 and 1 outputs to
a lane, few and many partial rows, a workgroup's last lanes past the end.  A gradient is a sum over the rows of
terms that are each rounded a few times, so it is held to 2^-24 times the sum of their sizes, times 16 roundings
(those of a term, and of partial sums whose errors mostly cancel)."""
import pytest
import torch

from mbconv_inputs import BlockShape, make_block_inputs
from oracle import oracle as orc
from paper_2110_10802_amd import dnnops as D
from parity_util import compare_block, run_gpu_block

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols", [(1, 4), (3, 64), (40, 132), (40, 131), (700, 68), (700, 67), (5000, 1028),
                                       (5000, 1025), (20000, 36)])
def test_weight_gradients(rows, cols):
    print(f"[reduce_splits] {rows} x {cols}", flush=True)
    gen = torch.Generator().manual_seed(rows + cols)
    x, dy = torch.randn(rows, cols, generator=gen), torch.randn(rows, cols, generator=gen)
    gamma, beta = torch.ones(cols).cuda(), torch.zeros(cols).cuda()
    xd, dyd = x.cuda(), dy.cuda()
    y, dx = torch.empty_like(xd), torch.empty_like(xd)
    mean, rstd = torch.empty(rows, device="cuda"), torch.empty(rows, device="cuda")
    dg, db = torch.full((cols,), float("nan"), device="cuda"), torch.full((cols,), float("nan"), device="cuda")
    scratch = torch.empty(max(D.layernorm_backward_scratch_bytes(rows, cols), 16), dtype=torch.uint8, device="cuda")
    D.layernorm_forward(xd, gamma, beta, 1e-5, rows, cols, y, mean, rstd)
    D.layernorm_backward(xd, dyd, gamma, mean, rstd, rows, cols, dx, dg, db, scratch)
    xh = (x.double() - mean.cpu().double()[:, None]) * rstd.cpu().double()[:, None]
    for got, terms in ((dg, dy.double() * xh), (db, dy.double())):
        bound = 16 * 2.0 ** -24 * terms.abs().sum(0) + 1e-30
        assert bool(((got.cpu().double() - terms.sum(0)).abs() <= bound).all())


@pytest.mark.parametrize("N,Cin,Cexp,Cout,H,stride", [(5, 8, 48, 8, 54, 2), (6, 24, 72, 22, 36, 2), (3, 13, 70, 9, 31, 1)])
def test_two_gradients_of_unequal_rows(N, Cin, Cexp, Cout, H, stride):
    s = BlockShape(N=N, Cin=Cin, H=H, W=H, Cexp=Cexp, Cse=4, Cout=Cout, k=3, stride=stride)
    t = make_block_inputs(s, seed=N)
    print(f"[reduce_splits] {s}", flush=True)
    res, blk = run_gpu_block(s, t)
    f, b = orc.mbconv_step(s, t)
    compare_block(s, t, res, f, b, blk)
