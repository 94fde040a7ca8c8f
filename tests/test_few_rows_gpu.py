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
