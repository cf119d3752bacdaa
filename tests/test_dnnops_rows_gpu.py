"""Row operators at the edges of their kernel forms (16 lanes, a wavefront, a workgroup per row; rows
that end in a partial vector) against the oracle, and softmax in place, which must give the same
bits as out of place although partial vectors overlap their neighbours."""
import numpy as np
import pytest

from oracle import dnnops as orc
from parity_util import rel_err

pytestmark = pytest.mark.gpu
FWD, GRAD = 1e-4, 1e-3
SHAPES = [(7, 3), (5, 4), (300, 5), (33, 63), (17, 64), (18, 65), (21, 127), (19, 129), (700, 257), (9, 1023),
          (6, 2047), (5, 2049), (3, 4095), (4, 4098), (2, 8191)]


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to("cuda:0")


def _host(t):
    return t.detach().cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("rows,cols", SHAPES)
def test_rows_match_oracle(rows, cols):
    import torch
    from paper_2110_10802_amd import dnnops as D
    rng = np.random.default_rng(rows * 9176 + cols)
    x = (rng.standard_normal((rows, cols)) * 2 + 0.5).astype(np.float32)
    dy = rng.standard_normal((rows, cols)).astype(np.float32)
    gamma = (1 + 0.1 * rng.standard_normal(cols)).astype(np.float32)
    beta = (0.1 * rng.standard_normal(cols)).astype(np.float32)
    xd, dyd, gd, bd = _dev(x), _dev(dy), _dev(gamma), _dev(beta)
    y, dx = torch.empty_like(xd), torch.empty_like(xd)
    print(f"[rows] {rows}x{cols}", flush=True)
    D.softmax_forward(xd, y, rows, cols)
    D.softmax_backward(y, dyd, dx, rows, cols)
    y2, dx2 = xd.clone(), dyd.clone()
    D.softmax_forward(y2, y2, rows, cols)
    D.softmax_backward(y, dx2, dx2, rows, cols)
    torch.cuda.synchronize()
    assert torch.equal(y, y2) and torch.equal(dx, dx2)
    assert rel_err(_host(y), orc.softmax_fwd(x)) <= FWD
    assert rel_err(_host(dx), orc.softmax_bwd(_host(y), dy)) <= GRAD

    mean, rstd = torch.empty(rows, device="cuda:0"), torch.empty(rows, device="cuda:0")
    dg, db = torch.empty_like(gd), torch.empty_like(bd)
    scratch = torch.empty(D.layernorm_backward_scratch_bytes(rows, cols), dtype=torch.uint8, device="cuda:0")
    D.layernorm_forward(xd, gd, bd, 1e-5, rows, cols, y, mean, rstd)
    D.layernorm_backward(xd, dyd, gd, mean, rstd, rows, cols, dx, dg, db, scratch)
    torch.cuda.synchronize()
    yo, mo, ro = orc.layernorm_fwd(x, gamma, beta, 1e-5)
    dxo, dgo, dbo = orc.layernorm_bwd(x, dy, gamma, mo, ro)
    assert rel_err(_host(y), yo) <= FWD
    # short rows: dx and dgamma are differences of terms that cancel; held to the size of the terms, as
    # in test_dnnops_gpu.py
    scale = float(np.sqrt(np.mean((dy.astype(np.float64) * gamma) ** 2)) * np.max(ro))
    assert rel_err(_host(dx), dxo, abs_floor=scale) <= GRAD
    floor = float(np.sqrt(np.mean(dy.astype(np.float64) ** 2)) * np.sqrt(rows))
    assert rel_err(_host(dg), dgo, abs_floor=floor) <= GRAD and rel_err(_host(db), dbo, abs_floor=floor) <= GRAD


@pytest.mark.parametrize("rows,cols", SHAPES)
def test_infinities_stay_where_the_arithmetic_puts_them(rows, cols):
    """An infinite gradient in the columns that two threads read must count once, as a number: the other
    columns of the row are infinite, not NaN, and the other rows untouched."""
    import torch
    from paper_2110_10802_amd import dnnops as D
    rng = np.random.default_rng(cols)
    y = rng.random((rows, cols)).astype(np.float32) / cols + np.float32(1e-6)
    dy = rng.standard_normal((rows, cols)).astype(np.float32)
    dy[1, cols - 2] = np.inf
    yd, dyd = _dev(y), _dev(dy)
    dx = torch.empty_like(yd)
    print(f"[rows/inf] {rows}x{cols}", flush=True)
    D.softmax_backward(yd, dyd, dx, rows, cols)
    torch.cuda.synchronize()
    got = _host(dx)
    with np.errstate(invalid="ignore"):
        s = (y.astype(np.float64) * dy).sum(1, keepdims=True)
        ref = y * (dy - s)  # row 1: -inf, and inf - inf in the column itself
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.isnan(ref).sum() == 1
    assert np.array_equal(np.isinf(got), np.isinf(ref)) and np.all(got[1][np.isinf(ref[1])] < 0)
    ok = np.isfinite(ref)
    assert rel_err(got[ok], ref[ok]) <= GRAD

    # a row whose reciprocal deviation is infinite (a constant row, eps 0): with gamma and dy above zero
    # both sums of the row are infinite, with x above the mean so are all terms
    x = (1 + rng.random((rows, cols))).astype(np.float32)
    gamma = (1 + rng.random(cols)).astype(np.float32)
    dyp = (1 + rng.random((rows, cols))).astype(np.float32)
    mean, rstd = np.zeros(rows, np.float32), np.ones(rows, np.float32)
    rstd[1] = np.inf
    xd, gd, dyd = _dev(x), _dev(gamma), _dev(dyp)
    dg, db = torch.empty_like(gd), torch.empty_like(gd)
    scratch = torch.empty(D.layernorm_backward_scratch_bytes(rows, cols), dtype=torch.uint8, device="cuda:0")
    D.layernorm_backward(xd, dyd, gd, _dev(mean), _dev(rstd), rows, cols, dx, dg, db, scratch)
    torch.cuda.synchronize()
    got = _host(dx)
    # dx of that row is inf * (dy - m1 - inf * inf): -inf
    assert np.all(np.isinf(got[1])) and np.all(got[1] < 0)
    assert np.all(np.isfinite(np.delete(got, 1, 0)))
    assert np.all(np.isinf(_host(dg))) and np.all(np.isfinite(_host(db)))
