"""The work that programs have this library do, as timed cases.

A case is one pass through the public entry points of ``paper_2110_10802_amd.binding`` (a training
step or an evaluation-mode forward of one MBConv block or of a chain of blocks) or of
``paper_2110_10802_amd.dnnops`` (an operator forward and backward).  Shapes are those of the
repository's own configurations (``mbconv_inputs``) and benchmark, and generic ones of the same
ranges.  The STORE policy is left out: it is the measured alternative to the default, not what a
program is meant to run.
"""
from __future__ import annotations

import math
from typing import Any, Dict, List

import torch

from paper_2110_10802_amd import binding as B
from paper_2110_10802_amd import dnnops as D

EPS, MOMENTUM, LN_EPS = 1e-3, 0.01, 1e-5
DEVICE = "cuda:0"
STORED = ("w_expand", "w_dw", "w_proj")  # kept in the activation dtype

# The EfficientNet-B0 stages (kernel, expand ratio, out channels, stride of first repeat, repeats)
STAGES = [(3, 1, 16, 1, 1), (3, 6, 24, 2, 2), (5, 6, 40, 2, 2), (3, 6, 80, 2, 3), (5, 6, 112, 1, 3),
          (5, 6, 192, 2, 4), (3, 6, 320, 1, 1)]


def _block(N, Cin, H, W, ratio, Cout, k, stride, dtype="f32", act="swish", se=True) -> Dict[str, Any]:
    return {"N": N, "Cin": Cin, "H": H, "W": W, "Cexp": Cin * ratio, "Cse": max(1, Cin // 4),
            "Cout": Cout, "k": k, "stride": stride, "expand": ratio != 1,
            "res": stride == 1 and Cin == Cout, "dtype": dtype, "act": act, "se": se}


def listed() -> List[Dict[str, Any]]:
    return [
        # the smallest training step a program runs (a unit test, a toy network): launches count
        {"name": "train_tiny", "kind": "train", **_block(2, 16, 16, 16, 6, 16, 3, 1)},
        # early repeat block at 56x56: large planes, few channels, bound by memory
        {"name": "train_56_k3", "kind": "train", **_block(32, 24, 56, 56, 6, 24, 3, 1)},
        # downsampling block: 5x5 filter, stride 2
        {"name": "train_56_k5s2", "kind": "train", **_block(64, 24, 56, 56, 6, 40, 5, 2)},
        # mixed-precision training of a middle stage: bf16 storage, 5x5 filter
        {"name": "train_14_bf16", "kind": "train", **_block(128, 112, 14, 14, 6, 112, 5, 1, dtype="bf16")},
        # the last stage: many channels on 7x7 planes (an odd plane size)
        {"name": "train_7_wide", "kind": "train", **_block(64, 192, 7, 7, 6, 320, 3, 1)},
        # a network at another input resolution: 15x15 planes, a batch that is no power of two
        {"name": "train_15_ragged", "kind": "train", **_block(24, 80, 15, 15, 6, 112, 5, 1)},
        # inference with the other activation, without squeeze-and-excitation.  (Not a training step:
        # the derivative jumps at 0 and 6, so a pre-activation within rounding of a kink moves
        # gradients of two correct implementations apart by whole elements.)
        {"name": "eval_56_relu6", "kind": "eval",
         **_block(32, 24, 56, 56, 6, 24, 3, 1, act="relu6", se=False)},
        # the whole network body, one training step: the benchmark's headline
        {"name": "chain_train", "kind": "chain_train", "N": 64, "H": 112, "Cin": 32},
        # the same body answering single requests
        {"name": "chain_eval", "kind": "chain_eval", "N": 1, "H": 112, "Cin": 32},
        # an activation map of a detection network, forward and backward
        {"name": "mish", "kind": "mish", "n": 8 * 64 * 304 * 304},
        # hidden states of a transformer layer, forward and backward
        {"name": "layernorm", "kind": "layernorm", "rows": 4096, "cols": 1024},
        # attention scores of a batch of 8 with 16 heads over a sequence of odd length
        {"name": "softmax_odd", "kind": "softmax", "rows": 8 * 16 * 381, "cols": 381},
    ]


def _log(rng, lo: float, hi: float) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng) -> Dict[str, Any]:
    kind = rng.choice(["train"] * 6 + ["eval", "chain_eval", "mish", "layernorm", "softmax"])
    if kind == "mish":
        return {"kind": kind, "n": _log(rng, 1e3, 6e7)}
    if kind in ("layernorm", "softmax"):
        cols = _log(rng, 32, 8192)
        return {"kind": kind, "rows": max(16, min(65536, _log(rng, 1e4, 4e7) // cols)), "cols": cols}
    if kind == "chain_eval":
        return {"kind": kind, "N": _log(rng, 1, 32), "H": 16 * rng.randint(4, 8), "Cin": 32}
    variant = rng.choice(["f32", "f32", "f32", "bf16", "relu6"])
    k, stride = rng.choice([3, 5]), rng.choice([1, 1, 2])
    H = _log(rng, 6, 112)
    W = H if rng.random() < 0.7 else max(6, min(112, H + rng.randint(-3, 3)))
    if stride == 2 and W % 4 == 2 and H * W > 60 * 60:
        W -= 2  # the library refuses these planes (stride 2, W % 4 == 2, more than 1024 runs of four)
    # few channels on large planes, many on small ones, as networks have them; odd counts among them
    Cin = max(8, min(256, _log(rng, 540, 3360) // max(H, 7)))
    Cin = Cin // 8 * 8 if rng.random() < 0.7 else Cin
    ratio = rng.choice([1, 3, 4, 6, 6, 6])
    Cout = Cin if stride == 1 and rng.random() < 0.6 else max(8, int(Cin * rng.uniform(0.5, 1.8)))
    N = _log(rng, 1, 128)
    N = max(1, min(N, 40_000_000 // (H * W * Cin * ratio)))
    # enough samples per channel behind each normalisation: over a handful, batch statistics
    # amplify rounding noise without bound (in bf16 far more)
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    N = max(N, -(-(4096 if variant == "bf16" else 256) // (Ho * Wo)))
    kind = "eval" if variant == "relu6" else kind
    return {"kind": kind, **_block(N, Cin, H, W, ratio, Cout, k, stride,
                                   dtype="bf16" if variant == "bf16" else "f32",
                                   act="relu6" if variant == "relu6" else "swish",
                                   se=variant != "relu6")}


# ---- shapes and inputs ---------------------------------------------------------------------

def _blocks(case) -> List[Dict[str, Any]]:
    """The block(s) of a case, in order."""
    if not case["kind"].startswith("chain"):
        return [case]
    out, c, h = [], case["Cin"], case["H"]
    for k, ratio, cout, stride, repeats in STAGES:
        for i in range(repeats):
            s = stride if i == 0 else 1
            out.append(_block(case["N"], c, h, h, ratio, cout, k, s))
            c, h = cout, (h - 1) // s + 1
    return out


def _out_hw(b):
    p = (b["k"] - 1) // 2
    return ((b["H"] + 2 * p - b["k"]) // b["stride"] + 1, (b["W"] + 2 * p - b["k"]) // b["stride"] + 1)


def _type(b):
    return torch.bfloat16 if b["dtype"] == "bf16" else torch.float32


def _desc(b) -> B.Desc:
    return B.Desc(b["N"], b["Cin"], b["H"], b["W"], b["Cexp"], b["Cse"], b["Cout"], b["k"], b["stride"],
                  (b["k"] - 1) // 2, int(b["expand"]), int(b["res"]),
                  B.MBCONV_BF16 if b["dtype"] == "bf16" else B.MBCONV_F32, B.MBCONV_RECOMPUTE, EPS, MOMENTUM,
                  B.MBCONV_ACT_RELU6 if b["act"] == "relu6" else B.MBCONV_ACT_SWISH, int(not b["se"]))


def _gen(seed):
    return torch.Generator(device=DEVICE).manual_seed(int(seed))


def _normal(gen, shape, std=1.0, mean=0.0):
    return torch.randn(shape, generator=gen, device=DEVICE).mul_(std).add_(mean)


def _weights(b, gen) -> Dict[str, torch.Tensor]:
    """Kaiming-normal convolutions and FCs, BN gamma near 1 and beta near 0."""
    Ci, Ce, Cs, Co, k = b["Cin"], b["Cexp"], b["Cse"], b["Cout"], b["k"]
    t = {}
    if b["expand"]:
        t["w_expand"] = _normal(gen, (Ce, Ci), math.sqrt(2 / Ci))
        t["bn1_gamma"], t["bn1_beta"] = _normal(gen, (Ce,), 0.1, 1.0), _normal(gen, (Ce,), 0.1)
    t["w_dw"] = _normal(gen, (Ce, k, k), math.sqrt(2 / (k * k)))
    t["bn2_gamma"], t["bn2_beta"] = _normal(gen, (Ce,), 0.1, 1.0), _normal(gen, (Ce,), 0.1)
    if b["se"]:
        t["se_w1"], t["se_b1"] = _normal(gen, (Cs, Ce), math.sqrt(2 / Ce)), _normal(gen, (Cs,), 0.1)
        t["se_w2"], t["se_b2"] = _normal(gen, (Ce, Cs), math.sqrt(2 / Cs)), _normal(gen, (Ce,), 0.1)
    t["w_proj"] = _normal(gen, (Co, Ce), math.sqrt(2 / Ce))
    t["bn3_gamma"], t["bn3_beta"] = _normal(gen, (Co,), 0.1, 1.0), _normal(gen, (Co,), 0.1)
    for n in STORED:
        if n in t:
            t[n] = t[n].to(_type(b))
    return t


def _running(b) -> Dict[str, torch.Tensor]:
    """Fresh running statistics, per normalisation one [2, C] tensor (mean, variance)."""
    def one(c):
        return torch.stack([torch.zeros(c, device=DEVICE), torch.ones(c, device=DEVICE)])
    r = {"bn1": one(b["Cexp"])} if b["expand"] else {}
    return {**r, "bn2": one(b["Cexp"]), "bn3": one(b["Cout"])}


def _block_inputs(case, seed):
    """(weights per block, running statistics per block, x, dout) of a block or chain case."""
    gen, bs = _gen(seed), _blocks(case)
    first, last = bs[0], bs[-1]
    weights = [_weights(b, gen) for b in bs]
    running = [_running(b) for b in bs]
    if case["kind"] in ("eval", "chain_eval"):
        # statistics that fit the weights, as a trained network has them: those of another batch
        n = max(2, min(8, -(-4096 // (last["H"] * last["W"]))))
        y = _normal(gen, (n, first["Cin"], first["H"], first["W"])).to(_type(first)).double()
        for b, w, r in zip(bs, weights, running):
            y, got = _reference(b, {k: v.double() for k, v in w.items()}, y, None)
            for k in r:
                r[k] = got[k].float().contiguous()
    x = _normal(gen, (first["N"], first["Cin"], first["H"], first["W"])).to(_type(first))
    dout = _normal(gen, (last["N"], last["Cout"], *_out_hw(last))).to(_type(last))
    return weights, running, x, dout


# ---- what a program keeps, and one pass -----------------------------------------------------

def _flat_like(tensors: Dict[str, torch.Tensor]):
    """One zeroed fp32 buffer with a 16-byte aligned view per tensor (a gradient bucket)."""
    size = {n: (t.numel() + 3) // 4 * 4 for n, t in tensors.items()}
    flat = torch.zeros(sum(size.values()), device=DEVICE)
    views, at = {}, 0
    for n, t in tensors.items():
        views[n] = flat[at:at + t.numel()].view(t.shape)
        at += size[n]
    return flat, views


def _bn_state(r):
    return B.BNState(**{f"{n}_{what}": t[i].data_ptr() for n, t in r.items()
                        for i, what in enumerate(("mean", "var"))})


def prepare(case, seed):
    kind = case["kind"]
    if kind == "mish":
        gen, n = _gen(seed), case["n"]
        x, dy = _normal(gen, (n,), 2.0), _normal(gen, (n,))
        return {"kind": kind, "n": n, "x": x, "dy": dy, "y": torch.empty_like(x), "dx": torch.empty_like(x)}
    if kind in ("layernorm", "softmax"):
        gen, rows, cols = _gen(seed), case["rows"], case["cols"]
        x, dy = _normal(gen, (rows, cols), 2.0, 0.5), _normal(gen, (rows, cols))
        s = {"kind": kind, "rows": rows, "cols": cols, "x": x, "dy": dy, "y": torch.empty_like(x),
             "dx": torch.empty_like(x)}
        if kind == "layernorm":
            s["gamma"], s["beta"] = _normal(gen, (cols,), 0.1, 1.0), _normal(gen, (cols,), 0.1)
            s["mean"], s["rstd"] = torch.empty(rows, device=DEVICE), torch.empty(rows, device=DEVICE)
            s["dgamma"], s["dbeta"] = torch.empty(cols, device=DEVICE), torch.empty(cols, device=DEVICE)
            s["scratch"] = torch.empty(max(16, D.layernorm_backward_scratch_bytes(rows, cols)),
                                       dtype=torch.uint8, device=DEVICE)
        return s
    weights, running, x, dout = _block_inputs(case, seed)
    train = kind in ("train", "chain_train")
    # all running statistics of a network in one buffer, as its gradients are
    sizes = [t.numel() for r in running for t in r.values()]
    stats = torch.cat([t.reshape(-1) for r in running for t in r.values()])
    parts = iter(stats.split(sizes))
    running = [{n: next(parts).view(t.shape) for n, t in r.items()} for r in running]
    blocks = []
    for b, w, r in zip(_blocks(case), weights, running):
        d = _desc(b)
        k = {"desc": d, "weights": w, "params": B.Params(**{n: t.data_ptr() for n, t in w.items()}),
             "stats": r, "running": _bn_state(r),
             "out": torch.empty((b["N"], b["Cout"], *_out_hw(b)), dtype=_type(b), device=DEVICE)}
        if train:
            saved, scratch = B.mbconv_workspace_size(d)
            k["saved"], k["scratch"] = torch.empty(saved, dtype=torch.uint8, device=DEVICE), scratch
            k["dx"] = torch.empty((b["N"], b["Cin"], b["H"], b["W"]), dtype=_type(b), device=DEVICE)
            k["flat"], k["views"] = _flat_like(w)
            k["grads"] = B.Grads(**{n: t.data_ptr() for n, t in k["views"].items()})
        else:
            k["scratch"] = B.mbconv_eval_workspace_size(d)
        blocks.append(k)
    # one workspace for all blocks of a network
    work = torch.empty(max(k["scratch"] for k in blocks), dtype=torch.uint8, device=DEVICE)
    return {"kind": kind, "blocks": blocks, "work": work, "x": x, "dout": dout, "stats": stats}


def run(s):
    kind = s["kind"]
    if kind == "mish":
        D.mish_forward(s["x"], s["y"], s["n"])
        D.mish_backward(s["x"], s["dy"], s["dx"], s["n"])
        return {"y": s["y"], "dx": s["dx"]}
    if kind == "softmax":
        D.softmax_forward(s["x"], s["y"], s["rows"], s["cols"])
        D.softmax_backward(s["y"], s["dy"], s["dx"], s["rows"], s["cols"])
        return {"y": s["y"], "dx": s["dx"]}
    if kind == "layernorm":
        D.layernorm_forward(s["x"], s["gamma"], s["beta"], LN_EPS, s["rows"], s["cols"], s["y"], s["mean"],
                            s["rstd"])
        D.layernorm_backward(s["x"], s["dy"], s["gamma"], s["mean"], s["rstd"], s["rows"], s["cols"], s["dx"],
                             s["dgamma"], s["dbeta"], s["scratch"])
        return {n: s[n] for n in ("y", "dx", "dgamma", "dbeta")}
    blocks, x = s["blocks"], s["x"]
    if kind in ("eval", "chain_eval"):
        for k in blocks:
            B.mbconv_forward_eval(k["desc"], k["params"], k["running"], x, k["out"], s["work"])
            x = k["out"]
        return {"out": x}
    inputs = []
    for k in blocks:
        inputs.append(x)
        B.mbconv_forward(k["desc"], k["params"], k["running"], x, k["out"], k["saved"], s["work"])
        x = k["out"]
    dy = s["dout"]
    for k, xi in zip(reversed(blocks), reversed(inputs)):
        B.mbconv_backward(k["desc"], k["params"], xi, dy, k["saved"], s["work"], k["dx"], k["grads"])
        dy = k["dx"]
    if kind == "train":
        k = blocks[0]
        return {"out": x, "dx": dy, "grads": k["views"], "running": k["stats"]}
    # a chain: one gradient bucket per block
    return {"out": x, "dx": dy, "grads": [k["flat"] for k in blocks],
            "running": s["stats"]}


# ---- what a pass cannot do without ------------------------------------------------------------

def work(case):
    kind = case["kind"]
    if kind == "mish":  # x read by both calls; dy read; y, dx written
        return {"bytes": 20 * case["n"], "flops": 0}
    if kind in ("layernorm", "softmax"):  # likewise (softmax: y is read in place of x)
        return {"bytes": 20 * case["rows"] * case["cols"], "flops": 0}
    nbytes = flops = 0
    train = kind in ("train", "chain_train")
    for b in _blocks(case):
        size = 2 if b["dtype"] == "bf16" else 4
        Ho, Wo = _out_hw(b)
        Q, Qo = b["N"] * b["H"] * b["W"], b["N"] * Ho * Wo
        X, E, Do, P = Q * b["Cin"], Q * b["Cexp"] * b["expand"], Qo * b["Cexp"], Qo * b["Cout"]
        w = b["Cexp"] * (b["Cin"] * b["expand"] + b["k"] ** 2 + b["Cout"] + 2 * b["Cse"] * b["se"])
        f = 2 * (b["Cexp"] * (b["Cin"] * b["expand"] * Q + (b["k"] ** 2 + b["Cout"]) * Qo))
        if train:
            # forward: x read; out and the tensors that batch statistics keep from being fused
            # away (e, d, p) written.  backward: x, dout, e, d, p read, dx written
            nbytes += size * (3 * X + 2 * P + 2 * (E + Do + P)) + 8 * w
            flops += 3 * f
        else:
            nbytes += size * (X + P) + 4 * w
            flops += f
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the largest relative error (2-norm) against 64 bits that was measured over
    the listed cases and some dozens of drawn ones (fp32 blocks and chains 5e-6, operators 1.4e-7,
    bf16 storage 1.5e-2 in BN1's gamma gradient, the residue of a sum that cancels)."""
    kind = case["kind"]
    if kind in ("mish", "softmax", "layernorm"):
        return {"rel": 1e-6}
    if case.get("dtype") == "bf16":
        return {"rel": 1.6e-2 if kind == "eval" else 3e-2}
    return {"rel": 2e-5}


# ---- the same in 64 bits, in plain torch --------------------------------------------------------

def _norm(v, gamma, beta, stats):
    """Batch normalisation over (N, H, W): with the given statistics, or with the batch's (then the
    batch's mean and unbiased variance come back too)."""
    m = v.shape[0] * v.shape[2] * v.shape[3]
    mean, var = (v.mean((0, 2, 3)), v.var((0, 2, 3), unbiased=False)) if stats is None else (stats[0], stats[1])
    y = (v - mean.view(1, -1, 1, 1)) / torch.sqrt(var.view(1, -1, 1, 1) + EPS)
    y = y * gamma.view(1, -1, 1, 1) + beta.view(1, -1, 1, 1)
    return y, torch.stack([mean, var * (m / max(1, m - 1))])


def _conv1x1(w, v):
    return torch.matmul(w, v.flatten(2)).view(v.shape[0], w.shape[0], v.shape[2], v.shape[3])


def _depthwise(w, v, stride):
    k = w.shape[-1]
    p = (k - 1) // 2
    v = torch.nn.functional.pad(v, (p, p, p, p))
    Ho, Wo = (v.shape[2] - k) // stride + 1, (v.shape[3] - k) // stride + 1
    y = 0
    for i in range(k):
        for j in range(k):
            tap = v[:, :, i:i + (Ho - 1) * stride + 1:stride, j:j + (Wo - 1) * stride + 1:stride]
            y = y + tap * w[:, i, j].view(1, -1, 1, 1)
    return y


def _reference(b, w, x, stats):
    """One block in 64 bits: (out, statistics used).  ``stats`` None: the batch's own."""
    def swish(t):
        return t * torch.sigmoid(t)
    act = (lambda t: t.clamp(0.0, 6.0)) if b["act"] == "relu6" else swish
    of = (lambda n: None) if stats is None else stats.get
    used, v = {}, x
    if b["expand"]:
        v, used["bn1"] = _norm(_conv1x1(w["w_expand"], v), w["bn1_gamma"], w["bn1_beta"], of("bn1"))
        v = act(v)
    v, used["bn2"] = _norm(_depthwise(w["w_dw"], v, b["stride"]), w["bn2_gamma"], w["bn2_beta"], of("bn2"))
    v = act(v)
    if b["se"]:
        q = v.mean((2, 3)) @ w["se_w1"].t() + w["se_b1"]
        v = v * torch.sigmoid(swish(q) @ w["se_w2"].t() + w["se_b2"])[:, :, None, None]
    v, used["bn3"] = _norm(_conv1x1(w["w_proj"], v), w["bn3_gamma"], w["bn3_beta"], of("bn3"))
    return (v + x if b["res"] else v), {n: t.detach() for n, t in used.items()}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("mish", "layernorm", "softmax"):
        s = prepare(case, seed)
        x = s["x"].double().requires_grad_()
        if kind == "mish":
            y = x * torch.tanh(torch.nn.functional.softplus(x, threshold=100))
        elif kind == "softmax":
            y = torch.softmax(x, -1)
        else:
            gamma, beta = s["gamma"].double().requires_grad_(), s["beta"].double().requires_grad_()
            xc = x - x.mean(-1, keepdim=True)
            y = xc / torch.sqrt(xc.square().mean(-1, keepdim=True) + LN_EPS) * gamma + beta
        y.backward(s["dy"].double())
        got = {"y": y.detach(), "dx": x.grad}
        return {**got, "dgamma": gamma.grad, "dbeta": beta.grad} if kind == "layernorm" else got
    weights, running, x, dout = _block_inputs(case, seed)
    bs = _blocks(case)
    if kind in ("eval", "chain_eval"):
        y = x.double()
        for b, w, r in zip(bs, weights, running):
            y, _ = _reference(b, {n: t.double() for n, t in w.items()}, y,
                              {n: t.double() for n, t in r.items()})
        return {"out": y}
    x = x.double().requires_grad_()
    y, new = x, []
    params = [{n: t.double().requires_grad_() for n, t in w.items()} for w in weights]
    for b, w, r in zip(bs, params, running):
        y, used = _reference(b, w, y, None)
        new.append({n: (1 - MOMENTUM) * r[n].double() + MOMENTUM * used[n] for n in r})
    y.backward(dout.double())
    out = {"out": y.detach(), "dx": x.grad}
    if kind == "train":
        return {**out, "grads": {n: t.grad for n, t in params[0].items()}, "running": new[0]}
    pad = torch.nn.functional.pad
    return {**out,
            "grads": [torch.cat([pad(t.grad.reshape(-1), (0, -t.numel() % 4)) for t in w.values()])
                      for w in params],
            "running": torch.cat([t.reshape(-1) for r in new for t in r.values()])}
