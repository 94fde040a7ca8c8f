"""Calls in a workspace that lacks the optional part (the room for split reductions, and in the block's forward passes for copies
of operands): the smallest size that each entry point accepts, found by asking with a misaligned matrix, which is rejected only
after the workspace has been accepted.  The workspace starts as NaNs and has guard bytes; bars as in the other parity tests,
against the fp64 oracles."""
import numpy as np
import pytest
import torch

from oracle import fdl_oracle as O
from oracle import siblings_oracle as S
from paper_2509_14279_amd import api, inputs as I
import harness as H

pytestmark = pytest.mark.gpu

P, BAD = 0x10000, 0x10004


def smallest(call, most):
    """least workspace size (a multiple of 256) that `call(bytes)` accepts"""
    lo, hi = 0, (most + 255) // 256
    assert call(hi * 256) == api.FDL_ERR_ALIGN
    while hi - lo > 1:
        mid = (lo + hi) // 2
        if call(mid * 256) == api.FDL_ERR_ALIGN:
            hi = mid
        else:
            lo = mid
    return hi * 256


def workspace(nbytes):
    ws = H.Guarded((nbytes,), torch.uint8)
    ws.view.fill_(0xff)
    return ws


# fp32: all tiles split, the last round split; bf16: 128 x 128 tiles, split and whole; 256 x 256 tiles with copies for padding, of X's
# last rows, and split, whole and padded (a test of the routes asks for these), gradients in one launch and with rows left over
SHAPES = [("f32", 256, 256, 256), ("f32", 300, 1025, 771), ("bf16", 512, 4096, 2048), ("bf16", 500, 2560, 4104),
          ("bf16", 700, 4099, 520), ("bf16", 1000, 256, 768), ("bf16", 2048, 1024, 2048), ("bf16", 4300, 256, 768),
          ("bf16", 4529, 157, 6144), ("bf16", 8425, 768, 1536), ("bf16", 1337, 3072, 3328), ("bf16", 2062, 2651, 2073)]


@pytest.mark.parametrize("dtype,M,K,N", SHAPES)
def test_block_and_siblings(dtype, M, K, N):
    print(f"[room] {dtype} {M}x{K}x{N}", flush=True)
    cfg = I.custom(dtype, M, K, N, seed=9990 + M)
    t = I.generate(cfg)
    n = {k: v.numpy().astype(np.float64) for k, v in t.items()}
    dt = I.storage_torch_dtype(dtype)
    d = {k: t[k].to("cuda", dt) for k in ("X", "W", "dY")}
    d.update({k: t[k].to("cuda") for k in ("b", "gamma", "beta")})
    f = torch.float32
    out = {k: H.Guarded(s, ty) for k, s, ty in (("Y", (M, N), dt), ("Z", (M, N), dt), ("I", (M, N), dt), ("R", (M, N), dt), ("mean", (M,), f),
           ("rstd", (M,), f), ("dX", (M, K), dt), ("dW", (N, K), dt), ("db", (N,), f), ("dgamma", (N,), f), ("dbeta", (N,), f),
           ("rX", (M, K), dt), ("rW", (N, K), dt), ("rb", (N,), f))}
    v = {k: g.view for k, g in out.items()}
    full = api.fdl_workspace_bytes(dtype, M, K, N)
    least = max(smallest(lambda b: api.fdl_forward_raw(dtype, M, K, N, BAD, P, P, P, P, 1e-5, P, P, P, P, P, b, None), full),
                smallest(lambda b: api.fdl_backward_raw(dtype, M, K, N, BAD, P, P, P, P, P, P, P, P, P, P, P, P, b, None), full))
    ws = workspace(least)
    api.fdl_forward(dtype, d["X"], d["W"], d["b"], d["gamma"], d["beta"], cfg.eps, v["Y"], v["Z"], v["mean"], v["rstd"], ws.view)
    ws.view.fill_(0xff)
    api.fdl_backward(dtype, d["dY"], d["X"], d["W"], d["gamma"], v["Z"], v["mean"], v["rstd"], v["dX"], v["dW"], v["db"], v["dgamma"],
                     v["dbeta"], ws.view)
    full_i = api.fdl_forward_inference_workspace_bytes(dtype, M, K, N)
    least_i = smallest(lambda b: api.fdl_forward_inference_raw(dtype, M, K, N, BAD, P, P, P, P, 1e-5, P, P, b, None), full_i)
    wi = workspace(least_i)
    api.fdl_forward_inference(dtype, d["X"], d["W"], d["b"], d["gamma"], d["beta"], cfg.eps, v["I"], wi.view)
    full_r = api.fdl_linear_relu_workspace_bytes(dtype, M, K, N)
    least_r = smallest(lambda b: api.fdl_linear_relu_forward_raw(dtype, M, K, N, BAD, P, P, P, P, b, None), full_r)
    wr = workspace(least_r)
    api.fdl_linear_relu_forward(dtype, d["X"], d["W"], d["b"], v["R"], wr.view)
    wr.view.fill_(0xff)
    api.fdl_linear_relu_backward(dtype, d["dY"], d["X"], d["W"], d["b"], v["rX"], v["rW"], v["rb"], wr.view)
    torch.cuda.synchronize()
    assert least < full or least_i < full_i or least_r < full_r
    for k, g in list(out.items()) + [("workspace", w) for w in (ws, wi, wr)]:
        assert g.intact(), f"kernel wrote outside the {k} buffer"
    ref = O.forward_backward(n["X"], n["W"], n["b"], n["gamma"], n["beta"], n["dY"], cfg.eps)
    for k in H.OUTPUTS + ("Z", "mean"):
        H.check(dtype, k, H.to_f64(v[k]), ref[k])
    H.check(dtype, "I", H.to_f64(v["I"]), ref["Y"])
    H.check(dtype, "R", H.to_f64(v["R"]), S.linear_relu_forward(n["X"], n["W"], n["b"])["Y"])
    rb = S.linear_relu_backward(n["dY"], n["X"], n["W"], n["b"])
    # a mask within 2^-20 (fp32 sums of at most 4099 products; fp64 ones: 2^-48) of the sum of its terms may go either way
    near = np.abs(rb["Z"]) <= (2.0 ** -20 if dtype == "bf16" else 2.0 ** -48) * (np.abs(n["X"]) @ np.abs(n["W"]).T + np.abs(n["b"]))
    slack = np.abs(n["dY"]) * near
    add = {"rX": slack @ np.abs(n["W"]), "rW": slack.T @ np.abs(n["X"]), "rb": slack.sum(axis=0)}
    for k, r in (("rX", rb["dX"]), ("rW", rb["dW"]), ("rb", rb["db"])):
        tol = 2e-2 * np.abs(r).max() if dtype == "bf16" else 1e-5 + 1e-4 * np.abs(r)
        assert np.all(np.abs(H.to_f64(v[k]) - r) <= tol + add[k]), k


@pytest.mark.parametrize("dtype,M,D,Hd", [("f32", 130, 300, 515), ("bf16", 1000, 640, 1000), ("bf16", 512, 1024, 2816),
                                          ("bf16", 600, 700, 1280), ("bf16", 1024, 1024, 2816), ("bf16", 4526, 1077, 1120),
                                          ("bf16", 2037, 1039, 3834), ("bf16", 1540, 2560, 3840)])
def test_feed_forward_block(dtype, M, D, Hd):
    t = I.generate_ffn(dtype, M, D, Hd, seed=9991 + M)
    d = {k: x.to("cuda", I.storage_torch_dtype(dtype)) for k, x in t.items()}
    Y = H.Guarded((M, D), I.storage_torch_dtype(dtype))
    ws = workspace(smallest(lambda b: api.fdl_llama_ffn_forward_raw(dtype, M, D, Hd, BAD, P, P, P, P, P, b, None),
                            api.fdl_llama_ffn_workspace_bytes(dtype, M, D, Hd)))
    api.fdl_llama_ffn_forward(dtype, d["X"], d["Wg"], d["Wu"], d["Wd"], Y.view, ws.view)
    torch.cuda.synchronize()
    assert Y.intact() and ws.intact()
    n = {k: x.numpy().astype(np.float64) for k, x in t.items()}
    H.check(dtype, "Y", H.to_f64(Y.view), S.llama_ffn_forward(n["X"], n["Wg"], n["Wu"], n["Wd"])["Y"])
