"""The bf16 kernel for few rows, and what is picked beside it, at the edges of its tiles (16 rows, 16 or 32 columns, steps of 32): one row to a few row
blocks, reductions shorter than a step and ending inside one, widths that end inside a group of four columns; every
epilogue.  Bars as in the other parity tests, against the fp64 oracles; guard bytes around every output."""
import numpy as np
import pytest
import torch

from oracle import siblings_oracle as S
from paper_2509_14279_amd import api, inputs as I
import harness as H

pytestmark = pytest.mark.gpu


def f64(t):
    return {k: v.numpy().astype(np.float64) for k, v in t.items()}


@pytest.mark.parametrize("M,K,N", [(1, 7, 1), (1, 32, 17), (15, 33, 3), (16, 264, 16), (17, 8, 260), (31, 4100, 33), (32, 520, 31),
                                   (33, 771, 130), (64, 1000, 1000), (65, 96, 34), (127, 2048, 514), (300, 136, 264),
                                   (130, 70, 200), (200, 512, 4096), (2048, 100, 64), (2049, 100, 64),
                                   (4096, 104, 64), (4097, 104, 64),
                                   # the estimates prefer the generic kernel: few rows with many columns, and batches whose
                                   # gradients run on padded copies (the masked gradient then has a pitch, zeros behind it)
                                   (100, 33, 40000), (60, 259, 20001), (140, 136, 8200), (1000, 136, 1000), (5000, 200, 264)])
def test_linear_relu(M, K, N):
    cfg = I.custom("bf16", M, K, N, seed=9000 + M + K + N)
    print(f"[few rows] {cfg.name}", flush=True)
    t = I.generate(cfg)
    X, W, dY = (t[k].to("cuda", torch.bfloat16) for k in ("X", "W", "dY"))
    b = t["b"].to("cuda")
    out = {"Y": H.Guarded((M, N), torch.bfloat16), "dX": H.Guarded((M, K), torch.bfloat16),
           "dW": H.Guarded((N, K), torch.bfloat16), "db": H.Guarded((N,), torch.float32)}
    ws = H.Guarded((max(256, api.fdl_linear_relu_workspace_bytes("bf16", M, K, N)),), torch.uint8)
    api.fdl_linear_relu_forward("bf16", X, W, b, out["Y"].view, ws.view)
    api.fdl_linear_relu_backward("bf16", dY, X, W, b, out["dX"].view, out["dW"].view, out["db"].view, ws.view)
    torch.cuda.synchronize()
    for k, g in list(out.items()) + [("workspace", ws)]:
        assert g.intact(), f"kernel wrote outside the {k} buffer"
    n = f64(t)
    H.check("bf16", "Y", H.to_f64(out["Y"].view), S.linear_relu_forward(n["X"], n["W"], n["b"])["Y"])
    # the masks the kernel chose are those of the exact pre-activation, except within 2^-20 of the sum of its terms
    # (fp32 sums of at most 4100 products); the gradients are then compared with those masks
    ref = S.linear_relu_backward(n["dY"], n["X"], n["W"], n["b"])
    scale = np.abs(n["X"]) @ np.abs(n["W"]).T + np.abs(n["b"])
    unsure = np.abs(ref["Z"]) <= 2.0 ** -20 * scale
    slack = np.abs(n["dY"]) * unsure
    add = {"dX": slack @ np.abs(n["W"]), "dW": slack.T @ np.abs(n["X"]), "db": slack.sum(axis=0)}
    for k in ("dX", "dW", "db"):
        got = H.to_f64(out[k].view)
        err = np.abs(got - ref[k])
        assert np.all(err <= 2e-2 * np.abs(ref[k]).max() + add[k]), k


@pytest.mark.parametrize("M,D,Hd", [(1, 8, 1), (3, 40, 19), (16, 512, 264), (17, 100, 130), (40, 333, 77), (64, 1024, 768),
                                    (100, 264, 1000), (260, 128, 512)])
def test_feed_forward_block(M, D, Hd):
    print(f"[few rows] ffn {M}x{D}x{Hd}", flush=True)
    t = I.generate_ffn("bf16", M, D, Hd, seed=9100 + M + D + Hd)
    d = {k: v.to("cuda", torch.bfloat16) for k, v in t.items()}
    Y = H.Guarded((M, D), torch.bfloat16)
    ws = H.Guarded((max(256, api.fdl_llama_ffn_workspace_bytes("bf16", M, D, Hd)),), torch.uint8)
    api.fdl_llama_ffn_forward("bf16", d["X"], d["Wg"], d["Wu"], d["Wd"], Y.view, ws.view)
    torch.cuda.synchronize()
    assert Y.intact() and ws.intact()
    n = f64(t)
    H.check("bf16", "Y", H.to_f64(Y.view), S.llama_ffn_forward(n["X"], n["Wg"], n["Wu"], n["Wd"])["Y"])


# Reductions from 2048 on, whose loads take whole lines of 8 rows: whole steps of 64 alone, with 8 indices left, with one, with four; every
# tile (1 and 2 blocks of 16 rows; 2 of them with two of columns, and 4, which keep the shorter loads; the gated one with 1, 2 and, from
# 4096 on, 4); widths that end inside a block of 16 columns and inside a group of four.  test_routes_host.py: all run on this kernel.
LINES = [(M, K, 1003) for M in (1, 16, 17, 33, 64) for K in (2048, 2056, 2049, 4100) if M <= 32 or K % 8 == 0] + [(40, 2056, 8203), (1, 8191, 40)]
LINES_FFN = [(M, D, H) for M in (1, 16, 17, 33, 64) for D, H in ((2048, 2056), (2056, 2048), (2049, 2056))]
LINES_FFN += [(16, 2112, 2059), (9, 4100, 2049), (40, 4104, 1096), (64, 4097, 1003)]


@pytest.mark.parametrize("M,K,N", LINES)
def test_linear_relu_of_long_reductions(M, K, N):
    print(f"[few rows] lines {M}x{K}x{N}", flush=True)
    t = I.generate(I.custom("bf16", M, K, N, seed=9200 + M + K + N))
    X, W, dY = (t[k].to("cuda", torch.bfloat16) for k in ("X", "W", "dY"))
    b = t["b"].to("cuda")
    Y = H.Guarded((M, N), torch.bfloat16)
    dX, dW, db = (torch.empty(s, device="cuda", dtype=d) for s, d in (((M, K), X.dtype), ((N, K), X.dtype), ((N,), torch.float32)))
    ws = torch.empty(max(256, api.fdl_linear_relu_workspace_bytes("bf16", M, K, N)), dtype=torch.uint8, device="cuda")
    api.fdl_linear_relu_forward("bf16", X, W, b, Y.view, ws)
    api.fdl_linear_relu_backward("bf16", dY, X, W, b, dX, dW, db, ws)
    torch.cuda.synchronize()
    assert Y.intact()
    z = X.double() @ W.double().t() + b.double()
    # fp32 sums of K + 1 terms, rounded to bf16 once (half a unit: 2^-8 at most)
    near = (K + 1) * 2.0 ** -24 * (X.double().abs() @ W.double().abs().t() + b.double().abs())
    assert torch.all((Y.view.double() - z.clamp(min=0)).abs() <= 2.0 ** -8 * z.clamp(min=0) + near)
    # db: sums of dY over the rows whose mask the recomputation leaves open (M terms in fp32 or more)
    mask, d = (z > 0).double(), dY.double()
    unsure = (z.abs() <= near).double()
    assert torch.all((db.double() - (d * mask).sum(0)).abs() <= (d.abs() * unsure).sum(0) + M * 2.0 ** -24 * d.abs().sum(0))


@pytest.mark.parametrize("M,D,Hd", LINES_FFN)
def test_feed_forward_block_of_long_reductions(M, D, Hd):
    print(f"[few rows] lines ffn {M}x{D}x{Hd}", flush=True)
    t = I.generate_ffn("bf16", M, D, Hd, seed=9300 + M + D + Hd)
    d = {k: v.to("cuda", torch.bfloat16) for k, v in t.items()}
    Y = H.Guarded((M, D), torch.bfloat16)
    ws = H.Guarded((max(256, api.fdl_llama_ffn_workspace_bytes("bf16", M, D, Hd)),), torch.uint8)
    api.fdl_llama_ffn_forward("bf16", d["X"], d["Wg"], d["Wu"], d["Wd"], Y.view, ws.view)
    torch.cuda.synchronize()
    assert Y.intact() and ws.intact()
    x, wg, wu, wd = (d[k].double() for k in ("X", "Wg", "Wu", "Wd"))
    g, u = x @ wg.t(), x @ wu.t()
    act = torch.nn.functional.silu(g) * u
    ref = act @ wd.t()
    # gate and up sums in fp32 (|SiLU'| <= 1.1; its exp2 and reciprocal 2^-20), the activation rounded to bf16, the down sums in fp32,
    # the output rounded to bf16
    s = 2.0 ** -24 * D
    err = 1.1 * s * (x.abs() @ wg.abs().t()) * u.abs() + s * (x.abs() @ wu.abs().t()) * torch.nn.functional.silu(g).abs() + 2.0 ** -20 * act.abs()
    err = err + 2.0 ** -8 * (act.abs() + err)
    bound = err @ wd.abs().t() + 2.0 ** -24 * Hd * (act.abs() @ wd.abs().t())
    assert torch.all((Y.view.double() - ref).abs() <= bound + 2.0 ** -8 * (ref.abs() + bound))
