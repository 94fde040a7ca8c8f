"""The bf16 products in 128 x 128 tiles (gemm_mid.hip): reductions and widths around the slice of 64, the tile and the last eight
elements, rows that start at any element, the last row read with and without a pitch behind it, reductions split for either
gradient, both or neither and for the forward product, long rows (two-kernel row pass), the activation's mask, a padded forward
product before unpadded gradients, few rows; the gated pair of products of the feed-forward block, widths around its 64 columns.  Workspaces start as NaNs and have guard bytes, as have the outputs; the same calls in
the smallest workspaces run unsplit.  Bars as in the other parity tests, against the fp64 oracles."""
import numpy as np
import pytest
import torch

from oracle import fdl_oracle as O
from oracle import siblings_oracle as S
from paper_2509_14279_amd import api, inputs as I
import harness as H

pytestmark = pytest.mark.gpu

SHAPES = [(129, 8, 9), (64, 64, 64), (128, 128, 128), (1024, 777, 513), (1025, 776, 513), (1023, 65, 640), (533, 10, 493),
          (35, 10, 3545), (4097, 130, 8), (200, 4099, 130), (700, 136, 8200), (333, 1030, 2177), (2500, 1000, 300), (40, 3000, 1001),
          (2429, 739, 3676), (4043, 277, 3345), (803, 1216, 884), (5000, 333, 96)]


def nans(nbytes):
    ws = H.Guarded((max(256, nbytes),), torch.uint8)
    ws.view.fill_(0xff)
    return ws


def block(M, K, N, t, eps, ws):
    bf = torch.bfloat16
    X, W, dY = (t[k].to("cuda", bf) for k in ("X", "W", "dY"))
    b, gamma, beta = (t[k].to("cuda") for k in ("b", "gamma", "beta"))
    f = torch.float32
    out = {k: H.Guarded(s, d) for k, s, d in (
        ("Y", (M, N), bf), ("Z", (M, N), bf), ("mean", (M,), f), ("rstd", (M,), f), ("dX", (M, K), bf), ("dW", (N, K), bf),
        ("db", (N,), f), ("dgamma", (N,), f), ("dbeta", (N,), f))}
    v = {k: g.view for k, g in out.items()}
    api.fdl_forward("bf16", X, W, b, gamma, beta, eps, v["Y"], v["Z"], v["mean"], v["rstd"], ws.view)
    ws.view.fill_(0xff)
    api.fdl_backward("bf16", dY, X, W, gamma, v["Z"], v["mean"], v["rstd"], v["dX"], v["dW"], v["db"], v["dgamma"], v["dbeta"],
                     ws.view)
    torch.cuda.synchronize()
    for k, g in list(out.items()) + [("workspace", ws)]:
        assert g.intact(), f"kernel wrote outside the {k} buffer"
    return v


@pytest.mark.parametrize("M,K,N", SHAPES)
def test_block(M, K, N):
    cfg = I.custom("bf16", M, K, N, seed=7100 + M + K + N)
    print(f"[mid] {cfg.name}", flush=True)
    t = I.generate(cfg)
    n = {k: v.numpy().astype(np.float64) for k, v in t.items()}
    ref = O.forward_backward(n["X"], n["W"], n["b"], n["gamma"], n["beta"], n["dY"], cfg.eps)
    full = api.fdl_workspace_bytes("bf16", M, K, N)
    P, BAD = 0x10000, 0x10004

    def accepted(nbytes):          # (a misaligned matrix is rejected only after the workspace has been accepted)
        a = api.fdl_forward_raw("bf16", M, K, N, BAD, P, P, P, P, 1e-5, P, P, P, P, P, nbytes, None)
        b = api.fdl_backward_raw("bf16", M, K, N, BAD, P, P, P, P, P, P, P, P, P, P, P, P, nbytes, None)
        return a == b == api.FDL_ERR_ALIGN

    lo, hi = 0, (full + 255) // 256
    assert accepted(hi * 256)
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if accepted(mid * 256) else (mid, hi)
    for nbytes in (full, hi * 256):
        v = block(M, K, N, t, cfg.eps, nans(nbytes))
        for k in H.OUTPUTS + ("Z", "mean"):
            H.check("bf16", k, H.to_f64(v[k]), ref[k])


@pytest.mark.parametrize("M,K,N", SHAPES)
def test_linear_relu(M, K, N):
    cfg = I.custom("bf16", M, K, N, seed=7200 + M + K + N)
    print(f"[mid] relu {cfg.name}", flush=True)
    t = I.generate(cfg)
    bf = torch.bfloat16
    X, W, dY = (t[k].to("cuda", bf) for k in ("X", "W", "dY"))
    b = t["b"].to("cuda")
    out = {"Y": H.Guarded((M, N), bf), "dX": H.Guarded((M, K), bf), "dW": H.Guarded((N, K), bf), "db": H.Guarded((N,), torch.float32)}
    ws = nans(api.fdl_linear_relu_workspace_bytes("bf16", M, K, N))
    api.fdl_linear_relu_forward("bf16", X, W, b, out["Y"].view, ws.view)
    ws.view.fill_(0xff)
    api.fdl_linear_relu_backward("bf16", dY, X, W, b, out["dX"].view, out["dW"].view, out["db"].view, ws.view)
    torch.cuda.synchronize()
    for k, g in list(out.items()) + [("workspace", ws)]:
        assert g.intact(), f"kernel wrote outside the {k} buffer"
    n = {k: v.numpy().astype(np.float64) for k, v in t.items()}
    H.check("bf16", "Y", H.to_f64(out["Y"].view), S.linear_relu_forward(n["X"], n["W"], n["b"])["Y"])
    # a mask within 2^-20 of the sum of its terms (fp32 sums of at most 4099 products) may go either way
    ref = S.linear_relu_backward(n["dY"], n["X"], n["W"], n["b"])
    unsure = np.abs(n["dY"]) * (np.abs(ref["Z"]) <= 2.0 ** -20 * (np.abs(n["X"]) @ np.abs(n["W"]).T + np.abs(n["b"])))
    add = {"dX": unsure @ np.abs(n["W"]), "dW": unsure.T @ np.abs(n["X"]), "db": unsure.sum(axis=0)}
    for k in ("dX", "dW", "db"):
        got = H.to_f64(out[k].view)
        assert np.all(np.abs(got - ref[k]) <= 2e-2 * np.abs(ref[k]).max() + add[k]), k


@pytest.mark.parametrize("M,D,Hd", [(40, 1026, 1500), (129, 136, 1001), (300, 1042, 1027), (512, 515, 1090), (103, 3197, 581), (1000, 640, 1000)])
def test_feed_forward_block(M, D, Hd):
    print(f"[mid] ffn {M}x{D}x{Hd}", flush=True)
    t = I.generate_ffn("bf16", M, D, Hd, seed=7300 + M + D + Hd)
    d = {k: v.to("cuda", torch.bfloat16) for k, v in t.items()}
    Y = H.Guarded((M, D), torch.bfloat16)
    ws = nans(api.fdl_llama_ffn_workspace_bytes("bf16", M, D, Hd))
    api.fdl_llama_ffn_forward("bf16", d["X"], d["Wg"], d["Wu"], d["Wd"], Y.view, ws.view)
    torch.cuda.synchronize()
    assert Y.intact() and ws.intact()
    n = {k: v.numpy().astype(np.float64) for k, v in t.items()}
    H.check("bf16", "Y", H.to_f64(Y.view), S.llama_ffn_forward(n["X"], n["Wg"], n["Wu"], n["Wd"])["Y"])
