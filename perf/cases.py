"""The calls that the speed of this library is judged by: its public entry points at the sizes its users meet.

A case is one operator (`op`), one storage type and one shape:

    step       fdl_forward then fdl_backward: the training step of the dense-layer block       M, K, N
    infer      fdl_forward_inference: the same block when serving                              M, K, N
    relu       fdl_linear_relu_forward then fdl_linear_relu_backward                           M, K, N
    layernorm  fdl_layernorm_forward                                                           M, N
    rmsnorm    fdl_rmsnorm_forward                                                             M, N
    ffn        fdl_llama_ffn_forward (N: the hidden width)                                     M, K, N

Buffers and workspace are allocated once, before the timed calls, as a caller of this library does.
"""
import math

import torch

from paper_2509_14279_amd import api

EPS = 1e-5


def listed():
    return [
        # a small layer in full precision: seven launches of a few microseconds each, so latency is everything
        {"name": "step_f32_small", "op": "step", "dtype": "f32", "M": 256, "K": 256, "N": 256},
        # full precision with every dimension odd: rows that start at any element, partial tiles on every edge
        {"name": "step_f32_ragged", "op": "step", "dtype": "f32", "M": 3001, "K": 771, "N": 1537},
        # an ordinary layer: one training micro-batch of 8192 rows
        {"name": "step_bf16_mid", "op": "step", "dtype": "bf16", "M": 8192, "K": 1024, "N": 4096},
        # the largest: the workload that bench.py reports
        {"name": "step_bf16_large", "op": "step", "dtype": "bf16", "M": 65536, "K": 2048, "N": 8192},
        # a layer whose widths are no multiple of anything
        {"name": "step_bf16_odd", "op": "step", "dtype": "bf16", "M": 3001, "K": 771, "N": 1537},
        # rows longer than a wavefront's or workgroup's registers hold (an expansion to four times the width)
        {"name": "step_bf16_long_rows", "op": "step", "dtype": "bf16", "M": 4096, "K": 4096, "N": 16384},
        # serving a handful of requests: fewer rows than one tile of the large contractions
        {"name": "infer_bf16_few_rows", "op": "infer", "dtype": "bf16", "M": 32, "K": 4096, "N": 4096},
        # the sibling layer, forward and backward, with widths that are multiples of 8 but of no tile
        {"name": "relu_bf16_ragged", "op": "relu", "dtype": "bf16", "M": 10000, "K": 1000, "N": 3000},
        # stand-alone normalisations: full precision at an ordinary batch, bf16 at a prefill's
        {"name": "layernorm_f32", "op": "layernorm", "dtype": "f32", "M": 8192, "N": 4096},
        {"name": "rmsnorm_bf16", "op": "rmsnorm", "dtype": "bf16", "M": 16384, "N": 4096},
        # the feed-forward block over a long prefill, and for one decoding step of a small batch
        {"name": "ffn_bf16_prefill", "op": "ffn", "dtype": "bf16", "M": 16384, "K": 4096, "N": 11008},
        {"name": "ffn_bf16_decode", "op": "ffn", "dtype": "bf16", "M": 16, "K": 4096, "N": 11008},
    ]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# smallest and largest M, K, N of a drawn case
_RANGES = {
    "step": ((256, 65536), (128, 4096), (256, 16384)),
    "infer": ((1, 32768), (128, 4096), (256, 16384)),
    "relu": ((64, 65536), (128, 4096), (64, 8192)),
    "layernorm": ((1, 65536), None, (64, 16384)),
    "rmsnorm": ((1, 65536), None, (64, 16384)),
    "ffn": ((1, 16384), (512, 4096), (1024, 11008)),
}


def draw(rng):
    op = rng.choice(["step"] * 7 + ["infer"] * 3 + ["relu"] * 2 + ["layernorm", "rmsnorm"] + ["ffn"] * 3)
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    m, k, n = _RANGES[op]
    # widths: whole tiles (the usual case), multiples of 8, anything
    grain = rng.choice([256, 256, 8, 1])
    snap = lambda v: max(grain, (v + grain // 2) // grain * grain)  # noqa: E731
    M, N = _spread(rng, *m), snap(_spread(rng, *n))
    if rng.random() < 0.4 and M >= 256:
        M = (M + 128) // 256 * 256
    if k is None:
        return {"op": op, "dtype": dtype, "M": M, "N": N}
    K = snap(_spread(rng, *k))
    # the product of the three stays where the call takes no longer than the largest listed one
    most = 1 << 33 if dtype == "f32" else (1 << 40 if grain == 256 else 1 << 37)
    while M * K * N > most:
        M = max(1, M // 2)
    return {"op": op, "dtype": dtype, "M": M, "K": K, "N": N}


def _inputs(case, seed):
    """The input tensors on the GPU, in the storage types the entry points take: activations of unit scale, weights
    scaled by their fan-in, small biases, normalisation weights around one."""
    dev = torch.device("cuda")
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))

    def normal(*shape, std=1.0, mean=0.0, to=torch.float32):
        t = torch.randn(*shape, device=dev, generator=g, dtype=torch.float32)
        return (t * std + mean).to(to)

    op, M, N = case["op"], case["M"], case["N"]
    if op == "layernorm":
        return {"A": normal(M, N, std=2.0, mean=0.5, to=dt), "gamma": normal(N, std=0.1 ** 0.5, mean=1.0),
                "beta": normal(N, std=0.1 ** 0.5)}
    if op == "rmsnorm":
        return {"A": normal(M, N, std=2.0, mean=0.5, to=dt), "weight": normal(N, std=0.1 ** 0.5, mean=1.0)}
    K = case["K"]
    if op == "ffn":
        return {"X": normal(M, K, to=dt), "Wg": normal(N, K, std=K ** -0.5, to=dt), "Wu": normal(N, K, std=K ** -0.5, to=dt),
                "Wd": normal(K, N, std=N ** -0.5, to=dt)}
    t = {"X": normal(M, K, to=dt), "W": normal(N, K, std=K ** -0.5, to=dt), "b": normal(N, std=0.02 ** 0.5)}
    if op in ("step", "infer"):
        t["gamma"] = normal(N, std=0.1 ** 0.5, mean=1.0)
        t["beta"] = normal(N, std=0.1 ** 0.5)
    if op in ("step", "relu"):
        t["dY"] = normal(M, N, to=dt)
    return t


def prepare(case, seed):
    s = _inputs(case, seed)
    op, dtype, M, N = case["op"], case["dtype"], case["M"], case["N"]
    dev = torch.device("cuda")
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32

    def matrix(r, c):
        return torch.empty(r, c, device=dev, dtype=dt)

    def vector(n):
        return torch.empty(n, device=dev, dtype=torch.float32)

    s["op"], s["dtype"] = op, dtype
    if op in ("layernorm", "rmsnorm"):
        s["Y"] = matrix(M, N)
        if op == "layernorm":
            s["mean"], s["rstd"] = vector(M), vector(M)
        return s
    K = case["K"]
    need = {"step": api.fdl_workspace_bytes, "infer": api.fdl_forward_inference_workspace_bytes,
            "relu": api.fdl_linear_relu_workspace_bytes, "ffn": api.fdl_llama_ffn_workspace_bytes}[op](dtype, M, K, N)
    s["workspace"] = torch.empty(need, device=dev, dtype=torch.uint8)
    s["Y"] = matrix(M, K if op == "ffn" else N)
    if op == "step":
        s["Zsave"], s["mean"], s["rstd"] = matrix(M, N), vector(M), vector(M)
        s["dgamma"], s["dbeta"] = vector(N), vector(N)
    if op in ("step", "relu"):
        s["dX"], s["dW"], s["db"] = matrix(M, K), matrix(N, K), vector(N)
    return s


def run(s):
    op, dtype = s["op"], s["dtype"]
    if op == "step":
        api.fdl_forward(dtype, s["X"], s["W"], s["b"], s["gamma"], s["beta"], EPS, s["Y"], s["Zsave"], s["mean"], s["rstd"],
                        s["workspace"])
        api.fdl_backward(dtype, s["dY"], s["X"], s["W"], s["gamma"], s["Zsave"], s["mean"], s["rstd"], s["dX"], s["dW"],
                         s["db"], s["dgamma"], s["dbeta"], s["workspace"])
        names = ("Y", "Zsave", "mean", "rstd", "dX", "dW", "db", "dgamma", "dbeta")
    elif op == "infer":
        api.fdl_forward_inference(dtype, s["X"], s["W"], s["b"], s["gamma"], s["beta"], EPS, s["Y"], s["workspace"])
        names = ("Y",)
    elif op == "relu":
        api.fdl_linear_relu_forward(dtype, s["X"], s["W"], s["b"], s["Y"], s["workspace"])
        api.fdl_linear_relu_backward(dtype, s["dY"], s["X"], s["W"], s["b"], s["dX"], s["dW"], s["db"], s["workspace"])
        names = ("Y", "dX", "dW", "db")
    elif op == "layernorm":
        api.fdl_layernorm_forward(dtype, s["A"], s["gamma"], s["beta"], EPS, s["Y"], s["mean"], s["rstd"])
        names = ("Y", "mean", "rstd")
    elif op == "rmsnorm":
        api.fdl_rmsnorm_forward(dtype, s["A"], s["weight"], EPS, s["Y"])
        names = ("Y",)
    else:
        api.fdl_llama_ffn_forward(dtype, s["X"], s["Wg"], s["Wu"], s["Wd"], s["Y"], s["workspace"])
        names = ("Y",)
    return {k: s[k] for k in names}


def work(case):
    op, M, N = case["op"], case["M"], case["N"]
    e = 2 if case["dtype"] == "bf16" else 4
    if op == "layernorm":
        return {"bytes": 2 * M * N * e + 8 * M + 8 * N, "flops": 8 * M * N}
    if op == "rmsnorm":
        return {"bytes": 2 * M * N * e + 4 * N, "flops": 4 * M * N}
    K = case["K"]
    if op == "ffn":
        return {"bytes": e * (2 * M * K + 3 * N * K), "flops": 6 * M * N * K}
    if op == "infer":
        return {"bytes": e * (M * K + N * K + M * N) + 12 * N, "flops": 2 * M * N * K}
    if op == "step":      # reads X, W, dY; writes Y, Zsave, dX, dW
        return {"bytes": e * (2 * M * K + 2 * N * K + 3 * M * N) + 24 * N + 8 * M, "flops": 6 * M * N * K}
    # relu: reads X, W, dY; writes Y, dX, dW; only inputs are kept, so the backward pass forms the product again
    return {"bytes": e * (2 * M * K + 2 * N * K + 2 * M * N) + 8 * N, "flops": 8 * M * N * K}


def tolerance(case):
    # about four times the distances from 64 bits that were measured.  bf16: 1.7e-3 to 2.6e-3, 3.5e-3 for the feed-forward
    # block, largest 1.6e-2; fp32 results are fp64 sums rounded once or twice: 5e-8, largest 2.7e-7
    if case["dtype"] == "f32":
        return {"rel": 2e-7, "max": 1e-6}
    if case["op"] == "relu":
        # where a pre-activation is within rounding of zero its whole gradient passes or not, as the sum's order has it
        return {"rel": 1e-2, "max": 0.5}
    return {"rel": 1.4e-2 if case["op"] == "ffn" else 1e-2, "max": 6e-2}


def _phi(z):
    return torch.exp(z.square().mul_(-0.5)).mul_(1.0 / math.sqrt(2.0 * math.pi))


def _cdf(z):
    return torch.erfc(z * (-1.0 / math.sqrt(2.0))).mul_(0.5)


def exact(case, seed):
    t = {k: v.double() for k, v in _inputs(case, seed).items()}
    op = case["op"]
    if op == "layernorm":
        A = t["A"]
        mean = A.mean(1)
        rstd = (A.var(1, unbiased=False) + EPS).rsqrt()
        return {"Y": (A - mean[:, None]) * rstd[:, None] * t["gamma"] + t["beta"], "mean": mean, "rstd": rstd}
    if op == "rmsnorm":
        A = t["A"]
        return {"Y": A * (A.square().mean(1, keepdim=True) + EPS).rsqrt() * t["weight"]}
    X = t["X"]
    if op == "ffn":
        h = X @ t["Wg"].t()
        h = h / (1.0 + torch.exp(-h))
        h *= X @ t["Wu"].t()
        return {"Y": h @ t["Wd"].t()}
    W = t["W"]
    Z = X @ W.t()
    Z += t["b"]
    if op == "relu":
        G = torch.where(Z > 0, t["dY"], torch.zeros((), dtype=Z.dtype, device=Z.device))
        # db, a sum of unrounded values, has no one value in bf16: a single mask that the order of fp32 sums decides moves
        # it by a thousand times its own rounding (2.6e-8 to 3e-4 from seed to seed)
        return {"Y": Z.clamp_(min=0), "dX": G @ W, "dW": G.t() @ X, "db": G.sum(0) if case["dtype"] == "f32" else None}
    P = _cdf(Z)
    A = Z * P
    mean = A.mean(1)
    rstd = (A.var(1, unbiased=False) + EPS).rsqrt()
    Ahat = (A - mean[:, None]).mul_(rstd[:, None])
    del A
    Y = Ahat * t["gamma"] + t["beta"]
    if op == "infer":
        return {"Y": Y}
    dY = t["dY"]
    dbeta, dgamma = dY.sum(0), (dY * Ahat).sum(0)
    g = dY * t["gamma"]
    c1, c2 = g.mean(1, keepdim=True), (g * Ahat).mean(1, keepdim=True)
    dZ = (g - c1 - Ahat * c2) * rstd[:, None]
    del g, Ahat
    dZ *= P + Z * _phi(Z)
    return {"Y": Y, "Zsave": Z, "mean": mean, "rstd": rstd, "dX": dZ @ W, "dW": dZ.t() @ X, "db": dZ.sum(0),
            "dgamma": dgamma, "dbeta": dbeta}
