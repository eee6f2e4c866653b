"""Workloads of the library, each one pass through its public entry points.

Every case is one kind of call that a program makes, at a size that the
repository's benchmark, tests or configurations use, or an ordinary size of
its kind.  ``listed`` holds one of each kind; ``draw`` gives another size of
one of the same kinds.  Plans are left to the library, as a program that only
names its operator leaves them.

``prepare`` makes the inputs on the GPU from a seed; ``run`` is one pass;
``work`` counts each input read once and each output written once; ``exact``
is the same result in FP64, by plain torch.
"""
from __future__ import annotations

import math

import torch

from paper_2609_01864_amd import autograd as A
from paper_2609_01864_amd import credit as C

DEV = "cuda:0"
EPS = 1e-5
DT = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn}
SIZE = {"f32": 4, "bf16": 2, "fp8": 1}

# kind -> (dtypes, rows, widths, most elements of a drawn case)
KINDS = {
    # RMSNorm of a few rows, statistics not kept: one token per sequence of a
    # small batch, where the call's latency is all there is
    "rms_decode": (("bf16", "f32"), (1, 64), (1024, 16384), 1 << 20),
    # RMSNorm of many rows of a hidden width, statistics not kept: a prompt
    "rms_prefill": (("bf16", "f32"), (1024, 16384), (1024, 16384), 1 << 27),
    # softmax over short rows, many of them: attention scores, class scores
    "softmax_short": (("bf16", "f32"), (4096, 32768), (256, 4096), 1 << 26),
    # LayerNorm as a training step runs it: forward, then dx, dgamma, dbeta
    "ln_train": (("bf16", "f32"), (1024, 16384), (1024, 16384), 1 << 26),
    # the same for RMSNorm, with odd sizes listed
    "rms_train": (("f32", "bf16"), (1024, 16384), (1024, 16384), 1 << 26),
    # LayerNorm backward of wide rows from saved statistics (the benchmark's
    # backward workload, M = 2048, N = 131072)
    "ln_bwd_wide": (("bf16", "f32"), (512, 2048), (16384, 131072), 1 << 28),
    # LayerNorm forward of very wide FP32 rows (the benchmark's bandwidth
    # workload, M = 1024, N up to 524288)
    "ln_wide": (("f32",), (256, 1024), (8192, 524288), 1 << 29),
    # FP8 softmax of wide rows (the benchmark's precision workload)
    "softmax_fp8": (("fp8",), (1024, 4096), (16384, 262144), 1 << 28),
    # FP8 LayerNorm of wide rows (the benchmark's precision workload)
    "ln_fp8": (("fp8",), (1024, 4096), (16384, 262144), 1 << 28),
    # softmax over a vocabulary and its gradient from the logits; vocabulary
    # sizes are rarely round
    "softmax_vocab": (("bf16", "f32"), (256, 4096), (16384, 131072), 1 << 27),
    # int8 codes and row scales of an activation matrix
    "quant": (("bf16", "f32"), (1024, 8192), (2048, 65536), 1 << 28),
    # an FP32 matrix to e4m3 codes under given row scales, and back
    "codec": (("f32",), (256, 8192), (1024, 65536), 1 << 27),
}


def listed():
    return [
        {"name": "rms_decode_4x5120_bf16", "kind": "rms_decode", "dtype": "bf16", "M": 4, "N": 5120},
        {"name": "rms_prefill_8192x5120_bf16", "kind": "rms_prefill", "dtype": "bf16", "M": 8192, "N": 5120},
        {"name": "softmax_short_16384x1000_bf16", "kind": "softmax_short", "dtype": "bf16", "M": 16384, "N": 1000},
        {"name": "ln_train_8192x4096_bf16", "kind": "ln_train", "dtype": "bf16", "M": 8192, "N": 4096},
        {"name": "rms_train_4095x5003_f32", "kind": "rms_train", "dtype": "f32", "M": 4095, "N": 5003},
        {"name": "ln_bwd_2048x131072_bf16", "kind": "ln_bwd_wide", "dtype": "bf16", "M": 2048, "N": 131072},
        {"name": "ln_wide_1024x524288_f32", "kind": "ln_wide", "dtype": "f32", "M": 1024, "N": 524288},
        {"name": "softmax_fp8_4096x65536", "kind": "softmax_fp8", "dtype": "fp8", "M": 4096, "N": 65536},
        {"name": "ln_fp8_4096x65536", "kind": "ln_fp8", "dtype": "fp8", "M": 4096, "N": 65536},
        {"name": "softmax_vocab_2048x50257_bf16", "kind": "softmax_vocab", "dtype": "bf16", "M": 2048, "N": 50257},
        {"name": "quant_int8_4096x11008_bf16", "kind": "quant", "dtype": "bf16", "M": 4096, "N": 11008},
        {"name": "codec_e4m3_4096x16384", "kind": "codec", "dtype": "f32", "M": 4096, "N": 16384},
    ]


def _between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(sorted(KINDS))
    dtypes, rows, widths, most = KINDS[kind]
    M, N = _between(rng, *rows), _between(rng, *widths)
    # a third of the widths as they fall (odd ones among them), a third whole
    # vectors, a third multiples of 256
    step = rng.choice((1, 16, 256))
    N = max(widths[0], N // step * step)
    while M * N > most:
        M = max(1, M // 2)
    return {"kind": kind, "dtype": rng.choice(dtypes), "M": M, "N": N}


def work(case):
    kind, M, N, e = case["kind"], case["M"], case["N"], SIZE[case["dtype"]]
    n = M * N
    if kind in ("rms_decode", "rms_prefill"):
        return {"bytes": 2 * n * e + 4 * N, "flops": 4 * n}
    if kind == "softmax_short":
        return {"bytes": 2 * n * e, "flops": 5 * n}
    if kind == "ln_train":  # x -> y with mean, rstd; then x, dy -> dx and the column sums
        return {"bytes": 5 * n * e + 16 * M + 20 * N, "flops": 20 * n}
    if kind == "rms_train":
        return {"bytes": 5 * n * e + 8 * M + 12 * N, "flops": 14 * n}
    if kind == "ln_bwd_wide":
        return {"bytes": 3 * n * e + 8 * M + 12 * N, "flops": 13 * n}
    if kind == "ln_wide":
        return {"bytes": 2 * n * e + 8 * M + 8 * N, "flops": 7 * n}
    if kind == "softmax_fp8":
        return {"bytes": 2 * n + 8 * M, "flops": 6 * n}
    if kind == "ln_fp8":
        return {"bytes": 2 * n + 16 * M + 8 * N, "flops": 9 * n}
    if kind == "softmax_vocab":  # x -> y; then x, dy -> dx
        return {"bytes": 5 * n * e, "flops": 13 * n}
    if kind == "quant":
        return {"bytes": n * (e + 1) + 4 * M, "flops": 3 * n}
    return {"bytes": 2 * (5 * n + 4 * M), "flops": 2 * n}  # codec: 4 -> 1, then 1 -> 4


# ------------------------------------------------------------------- inputs
def _inputs(case, seed):
    """The case's tensors by name, from the seed alone."""
    kind, dt, M, N = case["kind"], case["dtype"], case["M"], case["N"]
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))

    def normal(mean=0.0, std=1.0):
        return torch.randn((M, N), generator=g, device=DEV).mul_(std).add_(mean)

    def outliers():  # 3 N(0, 1) with 1% of the values at +-40
        x = normal(0.0, 3.0)
        u = torch.rand((M, N), generator=g, device=DEV)
        x.masked_fill_(u < 0.005, -40.0)
        return x.masked_fill_(u > 0.995, 40.0)

    def codes(x):
        s = x.abs().amax(dim=1) / 448.0
        return x.div_(s[:, None]).clamp_(-448.0, 448.0).to(DT["fp8"]), s

    t = {}
    if kind in ("rms_decode", "rms_prefill"):
        t["x"] = normal().to(DT[dt])
    elif kind in ("softmax_short", "softmax_vocab"):
        t["x"] = normal(0.0, 4.0).to(DT[dt])
    elif kind in ("ln_train", "rms_train", "ln_bwd_wide", "ln_wide"):
        t["x"] = normal(10.0 if kind.startswith("ln") else 0.0).to(DT[dt])
    elif kind in ("softmax_fp8", "ln_fp8"):
        t["x"], t["xs"] = codes(outliers())
    elif kind == "quant":
        t["x"] = outliers().to(DT[dt])
    else:
        t["x"] = normal()
        t["xs"] = t["x"].abs().amax(dim=1) / 448.0
    if kind in ("ln_train", "rms_train", "ln_bwd_wide", "softmax_vocab"):
        t["dy"] = normal().to(DT[dt])
    if kind.startswith(("rms", "ln")):
        t["gamma"] = torch.rand(N, generator=g, device=DEV).add_(0.5)
    if kind.startswith("ln") and kind != "ln_bwd_wide":
        t["beta"] = torch.randn(N, generator=g, device=DEV).mul_(0.1)
    return t


def prepare(case, seed):
    s = dict(_inputs(case, seed), kind=case["kind"])
    if case["kind"] in ("ln_train", "rms_train", "softmax_vocab"):
        for k in ("x", "gamma", "beta"):
            if k in s:
                s[k].requires_grad_(True)
    if case["kind"] == "ln_bwd_wide":  # what the forward saved
        x = s["x"].float()
        var, mean = torch.var_mean(x, dim=1, correction=0)
        s["mean"], s["rstd"] = mean, torch.rsqrt(var + EPS)
    C.handle(0)
    return s


def run(s):
    kind, x = s["kind"], s["x"]
    if kind in ("rms_decode", "rms_prefill"):
        y, _, _ = C.rmsnorm_fwd(x, s["gamma"], EPS, save_stats=False)
        return y
    if kind == "softmax_short":
        y, _ = C.softmax_fwd(x)
        return y
    if kind == "ln_train":
        y = A.layer_norm(x, s["gamma"], s["beta"], EPS)
        return [y, *torch.autograd.grad(y, (x, s["gamma"], s["beta"]), s["dy"])]
    if kind == "rms_train":
        y = A.rms_norm(x, s["gamma"], EPS)
        return [y, *torch.autograd.grad(y, (x, s["gamma"]), s["dy"])]
    if kind == "ln_bwd_wide":
        dx, _, dg, db = C.layernorm_bwd(x, s["dy"], s["gamma"], s["mean"], s["rstd"], EPS)
        return [dx, dg, db]
    if kind == "ln_wide":
        y, _, mean, rstd = C.layernorm_fwd(x, s["gamma"], s["beta"], EPS)
        return [y, mean, rstd]
    if kind == "softmax_fp8":
        return list(C.softmax_fwd(x, s["xs"]))
    if kind == "ln_fp8":
        return list(C.layernorm_fwd(x, s["gamma"], s["beta"], EPS, s["xs"]))
    if kind == "softmax_vocab":
        y = A.softmax(x, save="logits")
        return [y, *torch.autograd.grad(y, (x,), s["dy"])]
    if kind == "quant":
        return list(C.quantize_rows(x, "int8"))
    codes = C.encode(x, C.FP8, s["xs"])
    return [codes, C.decode(codes, s["xs"])]


# -------------------------------------------------------------------- exact
def _norm64(x, rms):
    if rms:
        return 0.0, torch.rsqrt(x.square().mean(dim=1, keepdim=True) + EPS)
    mean = x.mean(dim=1, keepdim=True)
    return mean, torch.rsqrt((x - mean).square().mean(dim=1, keepdim=True) + EPS)


def _norm_bwd64(x, dy, gamma, rms):
    mean, rstd = _norm64(x, rms)
    xh = (x - mean) * rstd
    g = dy * gamma
    dx = g - xh * (g * xh).mean(dim=1, keepdim=True)
    if not rms:
        dx -= g.mean(dim=1, keepdim=True)
    return dx * rstd, (dy * xh).sum(dim=0)


def exact(case, seed):
    kind = case["kind"]
    t = _inputs(case, seed)
    x = t["x"].double()
    gamma, beta, dy = (t[k].double() if k in t else None for k in ("gamma", "beta", "dy"))
    if kind in ("rms_decode", "rms_prefill"):
        return x * _norm64(x, True)[1] * gamma
    if kind == "softmax_short":
        return torch.softmax(x, dim=1)
    if kind == "ln_train":
        mean, rstd = _norm64(x, False)
        return [(x - mean) * rstd * gamma + beta, *_norm_bwd64(x, dy, gamma, False), dy.sum(dim=0)]
    if kind == "rms_train":
        return [x * _norm64(x, True)[1] * gamma, *_norm_bwd64(x, dy, gamma, True)]
    if kind == "ln_bwd_wide":
        return [*_norm_bwd64(x, dy, gamma, False), dy.sum(dim=0)]
    if kind == "ln_wide":
        mean, rstd = _norm64(x, False)
        return [(x - mean).mul_(rstd).mul_(gamma).add_(beta), mean[:, 0], rstd[:, 0]]
    if kind in ("softmax_fp8", "ln_fp8"):
        x *= t["xs"].double()[:, None]
        if kind == "softmax_fp8":
            y = torch.softmax(x, dim=1)
            s = y.amax(dim=1) / 448.0
            return [y.div_(s[:, None]), s]
        mean, rstd = _norm64(x, False)
        y = (x - mean).mul_(rstd).mul_(gamma).add_(beta)
        s = y.abs().amax(dim=1) / 448.0
        return [y.div_(s[:, None]), s, mean[:, 0], rstd[:, 0]]
    if kind == "softmax_vocab":
        y = torch.softmax(x, dim=1)
        return [y, y * (dy - (dy * y).sum(dim=1, keepdim=True))]
    if kind == "quant":
        return [None, x.abs().amax(dim=1) / 127.0]
    return [None, x]  # the decoded codes stand for x
