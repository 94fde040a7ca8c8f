"""The tuned bf16 contractions on widths that are no multiple of their tile: rows that start at any element (X goes through a
padded copy), rows of 16-byte pieces (X as it is), reductions below 128, widths that end inside a vector, batches that end
inside a tile or a pipeline round; dX and dW in one launch and in two; every epilogue.  The workspace starts as NaNs, so that
nothing is read that was not written.  Bars as in the other parity tests, against the fp64 oracles."""
import numpy as np
import pytest
import torch

from oracle import fdl_oracle as O
from oracle import siblings_oracle as S
from paper_2509_14279_amd import api, inputs as I
import harness as H

pytestmark = pytest.mark.gpu

SHAPES = [(129, 1451, 1451), (700, 100, 4096), (3001, 771, 120), (1000, 515, 2049), (640, 1000, 4101), (2500, 1000, 300),
          (385, 1285, 770), (257, 4099, 264), (20000, 130, 126)]
# and widths beside the tile with batches for whole row tiles or with reductions long enough to be split (these and the ones above
# run in 128 x 128 tiles or on the few-row kernel)
TILED = [(4097, 771, 1100), (4500, 384, 1100), (4300, 515, 2049), (4224, 1000, 1096), (500, 4096, 2000), (640, 2560, 4104),
         (1030, 4099, 520), (512, 4096, 2048), (700, 2560, 4096), (4700, 256, 768)]
SHAPES += TILED
# Large enough for the 256 x 256 tiles: the forward product on padded copies (X as it is and copied) and on operands as they are
# (whole and partial row tiles), then both with the reduction split; gradients padded and on whole tiles, in one launch and in two,
# with rows left over.  test_routes_host.py asks the planning code whether they get there.
LARGE = [(6737, 77, 4352), (4529, 157, 6144), (8760, 128, 5167), (4100, 1024, 3644), (11008, 128, 512), (2988, 128, 2816),
         (8425, 768, 1536), (6087, 2363, 1412),
         (1280, 3072, 3584), (1337, 3072, 3328), (4824, 3531, 1207), (2062, 2651, 2073), (2425, 3820, 1979)]
# the feed-forward block's gate and down products: padded (D as it is, D odd), the down product split, both on whole tiles, one of
# them in 128 x 128 tiles
LARGE_FFN = [(5827, 672, 1144), (4526, 1077, 1120), (2037, 1039, 3834), (1540, 2560, 3840), (5832, 1536, 1024), (1177, 3840, 3072),
             (3383, 512, 1280)]


def nan_workspace(nbytes):
    ws = H.Guarded((max(256, nbytes),), torch.uint8)
    ws.view.fill_(0xff)
    return ws


def f64(t):
    return {k: v.numpy().astype(np.float64) for k, v in t.items()}


@pytest.mark.parametrize("M,K,N", SHAPES)
def test_block(M, K, N):
    cfg = I.custom("bf16", M, K, N, seed=9300 + M + K + N)
    print(f"[padded] {cfg.name}", flush=True)
    t = I.generate(cfg)
    bf = torch.bfloat16
    X, W, dY = (t[k].to("cuda", bf) for k in ("X", "W", "dY"))
    b, gamma, beta = (t[k].to("cuda") for k in ("b", "gamma", "beta"))
    out = {k: H.Guarded(sh, dt) for k, sh, dt in (
        ("Y", (M, N), bf), ("Z", (M, N), bf), ("mean", (M,), torch.float32), ("rstd", (M,), torch.float32),
        ("dX", (M, K), bf), ("dW", (N, K), bf), ("db", (N,), torch.float32), ("dgamma", (N,), torch.float32),
        ("dbeta", (N,), torch.float32))}
    ws = nan_workspace(api.fdl_workspace_bytes("bf16", M, K, N))
    v = {k: g.view for k, g in out.items()}
    api.fdl_forward("bf16", X, W, b, gamma, beta, cfg.eps, v["Y"], v["Z"], v["mean"], v["rstd"], ws.view)
    ws.view.fill_(0xff)
    api.fdl_backward("bf16", dY, X, W, gamma, v["Z"], v["mean"], v["rstd"], v["dX"], v["dW"], v["db"], v["dgamma"],
                     v["dbeta"], ws.view)
    torch.cuda.synchronize()
    for k, g in list(out.items()) + [("workspace", ws)]:
        assert g.intact(), f"kernel wrote outside the {k} buffer"
    n = f64(t)
    ref = O.forward_backward(n["X"], n["W"], n["b"], n["gamma"], n["beta"], n["dY"], cfg.eps)
    for k in H.OUTPUTS + ("Z", "mean"):
        H.check("bf16", k, H.to_f64(v[k]), ref[k])


@pytest.mark.parametrize("M,K,N", SHAPES)
def test_linear_relu(M, K, N):
    cfg = I.custom("bf16", M, K, N, seed=9400 + M + K + N)
    print(f"[padded] relu {cfg.name}", flush=True)
    t = I.generate(cfg)
    bf = torch.bfloat16
    X, W, dY = (t[k].to("cuda", bf) for k in ("X", "W", "dY"))
    b = t["b"].to("cuda")
    out = {"Y": H.Guarded((M, N), bf), "dX": H.Guarded((M, K), bf), "dW": H.Guarded((N, K), bf), "db": H.Guarded((N,), torch.float32)}
    ws = nan_workspace(api.fdl_linear_relu_workspace_bytes("bf16", M, K, N))
    api.fdl_linear_relu_forward("bf16", X, W, b, out["Y"].view, ws.view)
    ws.view.fill_(0xff)
    api.fdl_linear_relu_backward("bf16", dY, X, W, b, out["dX"].view, out["dW"].view, out["db"].view, ws.view)
    torch.cuda.synchronize()
    for k, g in list(out.items()) + [("workspace", ws)]:
        assert g.intact(), f"kernel wrote outside the {k} buffer"
    n = f64(t)
    H.check("bf16", "Y", H.to_f64(out["Y"].view), S.linear_relu_forward(n["X"], n["W"], n["b"])["Y"])
    # a mask within 2^-20 of the sum of its terms (fp32 sums of at most 4099 products) may go either way
    ref = S.linear_relu_backward(n["dY"], n["X"], n["W"], n["b"])
    unsure = np.abs(n["dY"]) * (np.abs(ref["Z"]) <= 2.0 ** -20 * (np.abs(n["X"]) @ np.abs(n["W"]).T + np.abs(n["b"])))
    add = {"dX": unsure @ np.abs(n["W"]), "dW": unsure.T @ np.abs(n["X"]), "db": unsure.sum(axis=0)}
    for k in ("dX", "dW", "db"):
        got = H.to_f64(out[k].view)
        assert np.all(np.abs(got - ref[k]) <= 2e-2 * np.abs(ref[k]).max() + add[k]), k


@pytest.mark.parametrize("M,D,Hd", [(130, 1451, 1500), (1000, 640, 1000), (777, 1000, 1003), (4096, 264, 257), (512, 512, 1100),
                                    (600, 700, 1280)] + LARGE_FFN)
def test_feed_forward_block(M, D, Hd):
    print(f"[padded] ffn {M}x{D}x{Hd}", flush=True)
    t = I.generate_ffn("bf16", M, D, Hd, seed=9500 + M + D + Hd)
    d = {k: v.to("cuda", torch.bfloat16) for k, v in t.items()}
    Y = H.Guarded((M, D), torch.bfloat16)
    ws = nan_workspace(api.fdl_llama_ffn_workspace_bytes("bf16", M, D, Hd))
    api.fdl_llama_ffn_forward("bf16", d["X"], d["Wg"], d["Wu"], d["Wd"], Y.view, ws.view)
    torch.cuda.synchronize()
    assert Y.intact() and ws.intact()
    n = f64(t)
    H.check("bf16", "Y", H.to_f64(Y.view), S.llama_ffn_forward(n["X"], n["Wg"], n["Wu"], n["Wd"])["Y"])


@pytest.mark.parametrize("M,K,N", TILED + LARGE)
def test_unrounded_fp32_biases(M, K, N):
    # b is fp32 by contract also with bf16 matrices and is added in fp32: the stored
    # pre-activation is the correctly rounded one, within half a bf16 unit in the last place and the fp32 accumulation's error
    # (at most K terms: measured against 8 x 2^-24 of the sum of magnitudes, sixteen partial sums of matrix instructions)
    cfg = I.custom("bf16", M, K, N, seed=9600 + M + K + N)
    t = I.generate(cfg, with_dY=False)
    g = torch.Generator(device="cpu")
    g.manual_seed(4141)
    t["b"] = torch.randn(N, generator=g) * 0.1414 + 0.001
    got = H.run_fdl(cfg, t, backward=False)
    n = f64(t)
    Z = n["X"] @ n["W"].T + n["b"]
    ulp = 2.0 ** (np.floor(np.log2(np.maximum(np.abs(Z), 1e-30))) - 7)
    mag = np.abs(n["X"]) @ np.abs(n["W"]).T + np.abs(n["b"])
    tol = 0.5 * ulp * (1 + 1e-6) + 8 * 2.0 ** -24 * mag
    assert np.all(np.abs(H.to_f64(got["Z"]) - Z) <= tol)
    # the bound has teeth: a bias cut to its first piece leaves it
    low = (n["X"] @ n["W"].T + t["b"].to(torch.bfloat16).float().numpy().astype(np.float64))
    low = torch.from_numpy(low).float().to(torch.bfloat16).float().numpy().astype(np.float64)
    assert (np.abs(low - Z) > tol).any()


@pytest.mark.parametrize("M,K,N", [(300, 200, 264), (640, 1000, 1000), (400, 771, 1100), (256, 384, 520),
                                   (4097, 771, 1100), (4224, 1000, 1096), (4300, 515, 2049), (640, 2560, 4104),
                                   (4529, 157, 6144), (4100, 1024, 3644), (8425, 768, 1536), (2062, 2651, 2073), (1337, 3072, 3328),
                                   (5827, 672, 1144), (2037, 1039, 3834)])
def test_an_infinity_stays_in_its_row(M, K, N):
    # rows of a product are independent: an infinite and a NaN element of X change their own rows of the outputs only
    cfg = I.custom("bf16", M, K, N, seed=9800 + M + K + N)
    t = I.generate(cfg)
    bf = torch.bfloat16
    W = t["W"].to("cuda", bf)
    b, gamma, beta = (t[k].to("cuda") for k in ("b", "gamma", "beta"))
    bad = (7, M // 2, M - 1)

    def run(X):
        Y = torch.empty(M, N, device="cuda", dtype=bf)
        Z = torch.empty_like(Y); R = torch.empty_like(Y); F = torch.empty(M, K, device="cuda", dtype=bf)
        mean = torch.empty(M, device="cuda"); rstd = torch.empty(M, device="cuda")
        ws = torch.empty(max(api.fdl_workspace_bytes("bf16", M, K, N), api.fdl_linear_relu_workspace_bytes("bf16", M, K, N),
                             api.fdl_llama_ffn_workspace_bytes("bf16", M, K, N)), device="cuda", dtype=torch.uint8)
        api.fdl_forward("bf16", X, W, b, gamma, beta, cfg.eps, Y, Z, mean, rstd, ws)
        api.fdl_linear_relu_forward("bf16", X, W, b, R, ws)
        api.fdl_llama_ffn_forward("bf16", X, W, W, W.t().contiguous(), F, ws)
        torch.cuda.synchronize()
        return Y, Z, R, F

    X = t["X"].to("cuda", bf)
    clean = run(X)
    X = X.clone()
    X[bad[0], 0] = float("inf"); X[bad[1], 1] = float("nan"); X[bad[2], 0] = float("-inf")
    good = [r for r in range(M) if r not in bad]
    for a, c in zip(run(X), clean):
        assert torch.equal(a[good].view(torch.int16), c[good].view(torch.int16))


@pytest.mark.parametrize("M,K,N", LARGE)
def test_shapes_that_keep_the_large_tiles(M, K, N):
    test_block(M, K, N)
    test_linear_relu(M, K, N)
