"""The fp32-storage contractions at the edges of their tiles and of the split over the reduction: whole rounds of tiles with
and without an incomplete last one, small outputs with long reductions, reductions shorter than a slice or ending inside one,
rows of one to five elements, every epilogue.  The workspace starts as NaNs.  Bar: |got - ref| <= 1e-5 + 1e-4 |ref|, and
2^-23 of the sum of magnitudes as the products' own bound (fp64 sums, rounded once), against fp64."""
import numpy as np
import pytest
import torch

from oracle import siblings_oracle as S
from paper_2509_14279_amd import api, inputs as I
import harness as H

pytestmark = pytest.mark.gpu

# (M, K, N): N x K, M x N and M x K outputs
SHAPES = [(1, 1, 1), (5, 3, 2), (63, 1, 65), (64, 16, 64), (65, 17, 33), (130, 2, 515), (1100, 70, 1000), (2050, 33, 1030),
          (16, 2049, 300), (300, 1025, 1), (1026, 1030, 64), (257, 4, 4099)]


@pytest.mark.parametrize("M,K,N", SHAPES)
def test_linear_relu(M, K, N):
    cfg = I.custom("f32", M, K, N, seed=9600 + M + K + N)
    print(f"[f64] {cfg.name}", flush=True)
    t = I.generate(cfg)
    d = {k: t[k].to("cuda") for k in ("X", "W", "b", "dY")}
    f = torch.float32
    out = {"Y": H.Guarded((M, N), f), "dX": H.Guarded((M, K), f), "dW": H.Guarded((N, K), f), "db": H.Guarded((N,), f)}
    ws = H.Guarded((max(256, api.fdl_linear_relu_workspace_bytes("f32", M, K, N)),), torch.uint8)
    ws.view.fill_(0xff)
    api.fdl_linear_relu_forward("f32", d["X"], d["W"], d["b"], out["Y"].view, ws.view)
    ws.view.fill_(0xff)
    api.fdl_linear_relu_backward("f32", d["dY"], d["X"], d["W"], d["b"], out["dX"].view, out["dW"].view, out["db"].view, ws.view)
    torch.cuda.synchronize()
    for k, g in list(out.items()) + [("workspace", ws)]:
        assert g.intact(), f"kernel wrote outside the {k} buffer"
    n = {k: v.numpy().astype(np.float64) for k, v in t.items()}
    ref = dict(S.linear_relu_backward(n["dY"], n["X"], n["W"], n["b"]))
    G = ref["G"]
    ref["Y"] = S.linear_relu_forward(n["X"], n["W"], n["b"])["Y"]
    mag = {"Y": np.abs(n["X"]) @ np.abs(n["W"]).T + np.abs(n["b"]), "dX": np.abs(G) @ np.abs(n["W"]),
           "dW": np.abs(G).T @ np.abs(n["X"]), "db": np.abs(G).sum(axis=0)}
    for k in ("Y", "dX", "dW", "db"):
        got = H.to_f64(out[k].view)
        H.check("f32", k, got, ref[k])
        assert np.all(np.abs(got - ref[k]) <= 2.0 ** -23 * mag[k]), k


@pytest.mark.parametrize("M,D,Hd", [(3, 5, 7), (20, 300, 1000), (500, 130, 1050)])
def test_feed_forward_block(M, D, Hd):
    t = I.generate_ffn("f32", M, D, Hd, seed=9700 + M + D + Hd)
    d = {k: v.to("cuda") for k, v in t.items()}
    Y = H.Guarded((M, D), torch.float32)
    ws = H.Guarded((max(256, api.fdl_llama_ffn_workspace_bytes("f32", M, D, Hd)),), torch.uint8)
    ws.view.fill_(0xff)
    api.fdl_llama_ffn_forward("f32", d["X"], d["Wg"], d["Wu"], d["Wd"], Y.view, ws.view)
    torch.cuda.synchronize()
    assert Y.intact() and ws.intact()
    n = {k: v.numpy().astype(np.float64) for k, v in t.items()}
    H.check("f32", "Y", H.to_f64(Y.view), S.llama_ffn_forward(n["X"], n["Wg"], n["Wu"], n["Wd"])["Y"])


# all tiles of the forward product split, their parts added by the row kernel: one, two vectors per lane, a wavefront or a
# workgroup per row, rows that end inside a vector or a tile, one row, a partial last row tile
@pytest.mark.parametrize("M,K,N", [(1, 300, 65), (64, 256, 256), (129, 700, 257), (65, 515, 1023), (300, 300, 1027), (33, 2050, 2047),
                                   (500, 300, 130)])
def test_forward_passes(M, K, N):
    from oracle import fdl_oracle as O
    cfg = I.custom("f32", M, K, N, seed=9800 + M + K + N)
    t = I.generate(cfg, with_dY=False)
    d = {k: t[k].to("cuda") for k in ("X", "W", "b", "gamma", "beta")}
    f = torch.float32
    out = {"Y": H.Guarded((M, N), f), "Z": H.Guarded((M, N), f), "I": H.Guarded((M, N), f), "mean": H.Guarded((M,), f), "rstd": H.Guarded((M,), f)}
    v = {k: g.view for k, g in out.items()}
    ws = H.Guarded((max(256, api.fdl_workspace_bytes("f32", M, K, N)),), torch.uint8)
    ws.view.fill_(0xff)
    api.fdl_forward("f32", d["X"], d["W"], d["b"], d["gamma"], d["beta"], cfg.eps, v["Y"], v["Z"], v["mean"], v["rstd"], ws.view)
    ws.view.fill_(0xff)
    api.fdl_forward_inference("f32", d["X"], d["W"], d["b"], d["gamma"], d["beta"], cfg.eps, v["I"], ws.view)
    torch.cuda.synchronize()
    for k, g in list(out.items()) + [("workspace", ws)]:
        assert g.intact(), f"kernel wrote outside the {k} buffer"
    assert torch.equal(v["I"], v["Y"])
    n = {k: x.numpy().astype(np.float64) for k, x in t.items()}
    Z = n["X"] @ n["W"].T + n["b"]
    # fp64 sums, rounded once
    assert np.all(np.abs(H.to_f64(v["Z"]) - Z) <= 2.0 ** -24 * np.abs(Z) + 1e-12 * (np.abs(n["X"]) @ np.abs(n["W"]).T + np.abs(n["b"])))
    ref = O.forward(n["X"], n["W"], n["b"], n["gamma"], n["beta"], cfg.eps)
    for k in ("Y", "mean"):
        H.check("f32", k, H.to_f64(v[k]), ref[k])
