"""Timed cases of the 1D dilated convolution layer: what its users have it do, through its public entry points.

Three uses, over every geometry and both data types the layer takes:

* ``step``   forward + both backward passes through the C-ABI binding with buffers the caller keeps (``conv1d_fwd``,
             ``conv1d_bwd``): how a program with its own training loop drives the layer, and what ``bench.py`` times;
* ``train``  a convolution + bias + ReLU layer as a torch module under autograd (``autograd.Conv1d`` in float,
             ``autograd.conv1d`` with bfloat16 activations in bfloat16): forward, then the gradients of the input, the
             weights and the bias for a given upstream gradient;
* ``infer``  the forward pass with the fused bias + ReLU epilogue (``conv1d_fwd_ex``, bfloat16 output for bfloat16
             inputs), a fresh output per call: how a trained layer is served.

Distributions are those of ``paper_2104_08002_amd.inputs``: sparse non-negative tracks for the genomics-shaped layers,
normal or uniform values elsewhere, weights of variance 1 / (C S).
"""
import math

import torch

from paper_2104_08002_amd import autograd, binding


def _same(S, d):
    return (S - 1) * d // 2


def _case(name, use, dtype, N, C, K, W, S, d, P, x):
    return {"name": name, "use": use, "dtype": dtype, "N": N, "C": C, "K": K, "W": W, "S": S, "d": d, "P": P, "x": x}


def listed():
    return [
        # the smallest layer of the test suite: launches and host time are all of it
        _case("tiny_fp32_step", "step", "fp32", 2, 4, 4, 256, 5, 2, 0, "uniform"),
        # the layer of the AtacWorks network (15 channels and filters, 51 taps, dilation 8, 60000 columns, batch 16), the
        # benchmark's workload, in both types
        _case("genomics_bf16_step", "step", "bf16", 16, 15, 15, 60000, 51, 8, _same(51, 8), "sparse"),
        _case("genomics_fp32_step", "step", "fp32", 16, 15, 15, 60000, 51, 8, _same(51, 8), "sparse"),
        # the filter width x dilation sweep (batch 8, 64 channels and filters, 20000 columns): few and many taps, small
        # and large dilations, both types
        _case("sweep_fp32_S5_d1_step", "step", "fp32", 8, 64, 64, 20000, 5, 1, _same(5, 1), "uniform"),
        _case("sweep_fp32_S33_d4_step", "step", "fp32", 8, 64, 64, 20000, 33, 4, _same(33, 4), "uniform"),
        _case("sweep_bf16_S9_d2_step", "step", "bf16", 8, 64, 64, 20000, 9, 2, _same(9, 2), "uniform"),
        _case("sweep_bf16_S51_d8_step", "step", "bf16", 8, 64, 64, 20000, 51, 8, _same(51, 8), "uniform"),
        # many channels, few taps
        _case("wide_bf16_step", "step", "bf16", 32, 256, 256, 8192, 9, 4, _same(9, 4), "normal"),
        # training a layer with bias and ReLU: the bfloat16 shape of the paper's training runs (16 channels, 51 taps,
        # dilation 4, batch 56), and an ordinary float layer with odd sizes (odd width, dilation outside the powers of two)
        _case("train_bf16_c16", "train", "bf16", 56, 16, 16, 20000, 51, 4, _same(51, 4), "normal"),
        _case("train_fp32_odd", "train", "fp32", 12, 24, 40, 4999, 7, 3, 9, "normal"),
        # serving one segment at a time: a single sample through the genomics-shaped layer
        _case("infer_bf16_one", "infer", "bf16", 1, 15, 15, 60000, 51, 8, _same(51, 8), "sparse"),
        # the largest point of the paper's single-layer grid: batch 56, 64 channels and filters, 60000 columns, 51 taps
        _case("grid_fp32_largest_step", "step", "fp32", 56, 64, 64, 60000, 51, 1, _same(51, 1), "uniform"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _flops(case):
    passes = 1 if case["use"] == "infer" else 3
    Q = case["W"] + 2 * case["P"] - (case["S"] - 1) * case["d"]
    return passes * 2 * case["N"] * case["C"] * case["K"] * case["S"] * Q


def draw(rng):
    """A layer of the ranges above: channels 1 ... 256, widths 200 ... 60000, batches 1 ... 56, taps 1 ... 51."""
    most = 0.25 * _flops(listed()[-1])
    while True:
        use = rng.choice(("step", "step", "train", "infer"))
        dtype = rng.choice(("fp32", "bf16"))
        C = _log_int(rng, 4, 256) if rng.random() < 0.9 else rng.choice((1, 2, 3))
        K = C if rng.random() < 0.6 else _log_int(rng, 4, 256)
        if rng.random() < 0.3:  # channel counts are often round
            C, K = (max(16, 16 * round(v / 16)) for v in (C, K))
        S = rng.choice((1, 3, 5, 7, 9, 15, 17, 21, 25, 31, 33, 49, 51)) if rng.random() < 0.8 else rng.randint(1, 51)
        d = rng.choice((1, 2, 4, 8, 16)) if rng.random() < 0.8 else rng.randint(1, 16)
        W = _log_int(rng, 200, 60000)
        if rng.random() < 0.6:
            W = max(8, W // 8 * 8)
        N = _log_int(rng, 1, 56)
        P = _same(S, d) if rng.random() < 0.8 else rng.choice((0, 1, _same(S, d) // 2, S))
        case = {"use": use, "dtype": dtype, "N": N, "C": C, "K": K, "W": W, "S": S, "d": d, "P": P,
                "x": "sparse" if C < 17 and rng.random() < 0.5 else rng.choice(("normal", "uniform"))}
        Q = W + 2 * P - (S - 1) * d
        if Q >= 16 and _flops(case) <= most and max(C * W, K * Q) * N <= 56 * 64 * 60000:
            return case


def _values(gen, dist, shape):
    if dist == "uniform":
        return torch.rand(shape, generator=gen, device="cuda") * 2 - 1
    v = torch.randn(shape, generator=gen, device="cuda")
    if dist == "sparse":  # 80 % exact zeros, the rest exponential: a coverage track
        keep = torch.rand(shape, generator=gen, device="cuda") < 0.2
        v = v.exponential_(1.0, generator=gen) * keep
    return v


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    N, C, K, W, S, d, P = (case[k] for k in ("N", "C", "K", "W", "S", "d", "P"))
    Q = W + 2 * P - (S - 1) * d
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    s = dict(case, x=_values(gen, case["x"], (N, C, W)).to(dtype),
             w=(_values(gen, "normal", (K, C, S)) / math.sqrt(C * S)).to(dtype))
    if case["use"] != "infer":
        s["dy"] = _values(gen, "uniform" if case["x"] == "uniform" else "normal", (N, K, Q)).to(dtype)
    if case["use"] == "step":
        code = binding.CONV1D_BF16 if case["dtype"] == "bf16" else binding.CONV1D_FP32
        s["y"] = torch.empty((N, K, Q), dtype=torch.float32, device="cuda")
        s["dx"] = torch.empty((N, C, W), dtype=torch.float32, device="cuda")
        s["dw"] = torch.empty((K, C, S), dtype=torch.float32, device="cuda")
        need = binding.conv1d_bwd_weight_workspace_bytes(N, C, K, W, S, d, P, code)
        s["ws"] = torch.empty(max(256, need), dtype=torch.uint8, device="cuda")
    else:
        bias = 0.1 * _values(gen, "normal", (K,))
        if case["use"] == "infer":
            s["bias"] = bias
        elif case["dtype"] == "fp32":
            s["net"] = autograd.Conv1d(C, K, S, dilation=d, padding=P, bias=True, relu=True)
            with torch.no_grad():
                s["net"].weight.copy_(s["w"])
                s["net"].bias.copy_(bias)
            s["x"].requires_grad_(True)
        else:
            s["bias"] = bias.requires_grad_(True)
            s["x"].requires_grad_(True)
            s["w"].requires_grad_(True)
    return s


def run(s):
    x, w, d, P = s["x"], s["w"], s["d"], s["P"]
    if s["use"] == "step":
        binding.conv1d_fwd(x, w, d, P, out=s["y"])
        binding.conv1d_bwd(x, s["dy"], w, d, P, out_dx=s["dx"], out_dw=s["dw"], workspace=s["ws"])
        return {"y": s["y"], "dx": s["dx"], "dw": s["dw"]}
    if s["use"] == "infer":
        return binding.conv1d_fwd_ex(x, w, d, P, bias=s["bias"], relu=True, out_bf16=s["dtype"] == "bf16")
    if s["dtype"] == "fp32":
        net = s["net"]
        y = net(x)
        dx, dw, db = torch.autograd.grad(y, (x, net.weight, net.bias), s["dy"])
    else:
        y = autograd.conv1d(x, w, s["bias"], dilation=d, padding=P, relu=True, bf16_out=True)
        dx, dw, db = torch.autograd.grad(y, (x, w, s["bias"]), s["dy"])
    return {"y": y.detach(), "dx": dx, "dw": dw, "db": db}


def exact(case, seed):
    """The passes in 64 bits with plain torch: one product of matrices per tap."""
    s = prepare(case, seed)
    w, d, P = s["w"] if "w" in s else s["net"].weight, s["d"], s["P"]
    x, w = s["x"].detach().double(), w.detach().double()
    W, S = x.shape[2], w.shape[2]
    Q = W + 2 * P - (S - 1) * d
    if s["N"] * max(s["C"] * (W + 2 * P), s["K"] * Q) > 3e8:
        return None
    xp = torch.nn.functional.pad(x, (P, P))
    z = torch.zeros((s["N"], s["K"], Q), dtype=torch.float64, device="cuda")
    for t in range(S):
        z += torch.matmul(w[:, :, t].contiguous(), xp[:, :, t * d:t * d + Q].contiguous())
    if s["use"] != "step":
        bias = s["bias"] if "bias" in s else s["net"].bias
        z = (z + bias.detach().double()[None, :, None]).clamp(min=0)
    if s["use"] == "infer":
        return z
    g = s["dy"].double()
    if s["use"] == "train":
        g = g * (z > 0)
    dxp = torch.zeros_like(xp)
    dw = torch.empty_like(w)
    gt = g.transpose(1, 2).contiguous()
    for t in range(S):
        dxp[:, :, t * d:t * d + Q] += torch.matmul(w[:, :, t].t().contiguous(), g)
        dw[:, :, t] = torch.matmul(xp[:, :, t * d:t * d + Q].contiguous(), gt).sum(0).t()
    r = {"y": z, "dx": dxp[:, :, P:P + W].contiguous(), "dw": dw}
    if s["use"] == "train":
        r["db"] = g.sum((0, 2))
    return r


def work(case):
    """Each input read once, each output written once; 2 N C K S Q operations per pass."""
    N, C, K, W, S, d, P = (case[k] for k in ("N", "C", "K", "W", "S", "d", "P"))
    Q = W + 2 * P - (S - 1) * d
    e = 2 if case["dtype"] == "bf16" else 4
    x, w, y = N * C * W, K * C * S, N * K * Q
    if case["use"] == "step":  # in: x, w, dy; out: y, dx, dw in float
        nbytes = (x + w + y) * e + (y + x + w) * 4
    elif case["use"] == "infer":
        nbytes = (x + w + y) * e + 4 * K
    else:  # in: x, w, bias, dy; out: y, dx, dw, dbias, in the inputs' type
        nbytes = 2 * (x + w + y) * e + 8 * K
    return {"bytes": nbytes, "flops": _flops(case)}


def tolerance(case):
    """Four times what the passes differ by from themselves in 64 bits.  Float sums: 8e-7 in the norm for the passes over
    channels and taps, 4.5e-9 sqrt(n) for weight gradients of n = N Q terms (1.8e-6 at 160000, 8.3e-6 at 3.4 million),
    single values ten times that.  Results stored as bfloat16: 5e-5 in the norm (values on the edge between two bfloat16
    numbers), single values one step of 2^-7.  Where a ReLU is differentiated, an activation within a rounding error of
    zero may fall on either side (about one in two million): its whole gradient then comes or goes."""
    n = case["N"] * (case["W"] + 2 * case["P"] - (case["S"] - 1) * case["d"])
    rel = 4 * (8e-7 + 4.5e-9 * math.sqrt(n))
    tol = {"rel": rel, "max": 10 * rel}
    if case["use"] != "step" and case["dtype"] == "bf16":
        tol = {"rel": 2e-4, "max": 0.03}
    if case["use"] == "train" and n * case["K"] > 20000:
        n *= case["K"]
        tol = {"rel": tol["rel"] + 2 * math.sqrt((1 + 1e-6 * n) / n), "max": 0.5}
    return tol
