"""Infinities, NaN and the largest finite numbers in the products' epilogues, on every kernel that forms a forward product: the
256 x 256 tiles on operands as they are, on padded copies and with a split reduction, the 128 x 128 ones whole and split, the
few-row and the generic one.  A bias of
-infinity closes a unit and one of +infinity opens it, whatever the rest; the gradient of a unit whose pre-activation is NaN
is zero; a row of the feed-forward block overflows to infinity where its exact value does."""
import numpy as np
import pytest
import torch

from paper_2509_14279_amd import api, inputs as I

pytestmark = pytest.mark.gpu

BIG = 3.4e38          # above the largest bf16 number: it rounds to infinity there, in fp32 it is finite
# 128 x 128 tiles; 256 x 256, one round of the pipeline; 128 x 128, two of them split; few rows
SHAPES = [(4608, 256, 768), (4700, 256, 768), (16384, 128, 256), (4500, 384, 1100), (4097, 771, 1100), (512, 4096, 2048),
          (500, 4096, 2000), (32, 128, 256), (200, 136, 264), (127, 33, 1030)]
# 256 x 256 tiles: as they are; ragged rows; padded, X as it is / as a copy; split, ragged rows, padded; and the generic kernel
SHAPES += [(11008, 128, 512), (8425, 768, 1536), (8760, 128, 5167), (4529, 157, 6144), (1280, 3072, 3584), (1337, 3072, 3328),
           (2062, 2651, 2073), (4864, 151, 70)]


def data(M, K, N):
    t = I.generate(I.custom("bf16", M, K, N, seed=9900 + M + N))
    d = {k: t[k].to("cuda", torch.bfloat16) for k in ("X", "W", "dY")}
    d["b"] = t["b"].to("cuda")
    d["b"][:4] = torch.tensor([float("-inf"), float("inf"), BIG, -BIG])
    return d


def relu(d, M, K, N):
    ws = torch.empty(max(256, api.fdl_linear_relu_workspace_bytes("bf16", M, K, N)), dtype=torch.uint8, device="cuda")
    Y = torch.empty(M, N, device="cuda", dtype=torch.bfloat16)
    dX = torch.empty(M, K, device="cuda", dtype=torch.bfloat16)
    dW = torch.empty(N, K, device="cuda", dtype=torch.bfloat16)
    db = torch.empty(N, device="cuda")
    api.fdl_linear_relu_forward("bf16", d["X"], d["W"], d["b"], Y, ws)
    api.fdl_linear_relu_backward("bf16", d["dY"], d["X"], d["W"], d["b"], dX, dW, db, ws)
    torch.cuda.synchronize()
    return Y, dX, dW, db


@pytest.mark.parametrize("M,K,N", SHAPES)
def test_biases_that_open_or_close_a_unit(M, K, N):
    print(f"[special] bias {M}x{K}x{N}", flush=True)
    d = data(M, K, N)
    Y, dX, dW, db = relu(d, M, K, N)
    inf = float("inf")
    assert torch.all(Y[:, 0] == 0) and torch.all(Y[:, 3] == 0) and torch.all(Y[:, 1] == inf) and torch.all(Y[:, 2] == inf)
    assert torch.isfinite(Y[:, 4:].float()).all()
    assert torch.all(dW[[0, 3]] == 0) and db[0] == 0 and db[3] == 0
    # the open units' gradients are all of dY: sums of M terms in fp32 parts and fp64
    want = d["dY"][:, 1:3].double().sum(0)
    assert torch.all((db[1:3].double() - want).abs() <= 2.0 ** -16 * d["dY"][:, 1:3].double().abs().sum(0))
    assert torch.isfinite(dX.float()).all() and torch.isfinite(dW.float()).all()
    # the stored pre-activation of the block
    Yb = torch.empty_like(Y); Z = torch.empty_like(Y); mean = torch.empty(M, device="cuda"); rstd = torch.empty(M, device="cuda")
    ws = torch.empty(api.fdl_workspace_bytes("bf16", M, K, N), dtype=torch.uint8, device="cuda")
    one = torch.ones(N, device="cuda")
    api.fdl_forward("bf16", d["X"], d["W"], d["b"], one, one, 1e-5, Yb, Z, mean, rstd, ws)
    torch.cuda.synchronize()
    assert torch.all(Z[:, 0] == -inf) and torch.all(Z[:, 3] == -inf) and torch.all(Z[:, 1] == inf) and torch.all(Z[:, 2] == inf)


@pytest.mark.parametrize("M,K,N", SHAPES)
def test_a_nan_pre_activation_passes_no_gradient(M, K, N):
    print(f"[special] nan {M}x{K}x{N}", flush=True)
    d = data(M, K, N)
    d["b"][:4] = 0.0
    rows = (3, M - 1)
    # NaNs of either sign (the sign a sum of NaNs takes is the hardware's)
    bad = torch.tensor([0x7fc0, -64], dtype=torch.int16, device="cuda").view(torch.bfloat16)
    for r, v in zip(rows, bad):
        d["X"][r, 0] = v
    _, dX, _, db = relu(d, M, K, N)
    for r in rows:
        assert torch.all(dX[r] == 0)
    assert torch.isfinite(dX.float()).all() and torch.isfinite(db).all()


# gate, up and down products in 128 x 128 tiles; on few rows; on padded copies (D as it is, D through a copy of X, down product
# split); on 256 x 256 tiles, the down product whole, split and in 128 x 128 tiles
FFN = [(4500, 384, 1100), (4097, 771, 1003), (4608, 256, 640), (16, 256, 264), (150, 100, 130),
       (5827, 672, 1144), (4526, 1077, 1120), (2037, 1039, 3834), (5832, 1536, 1024), (1540, 2560, 3840), (3383, 512, 1280)]


@pytest.mark.parametrize("M,D,H", FFN)
def test_an_infinite_row_of_the_feed_forward_block(M, D, H):
    print(f"[special] ffn {M}x{D}x{H}", flush=True)
    t = I.generate_ffn("bf16", M, D, H, seed=9950 + M)
    # all weights positive: an infinite element of X makes every sum of its row +infinity, gate, activation and output alike
    d = {k: (v.abs() + 2.0 ** -10 if k != "X" else v).to("cuda", torch.bfloat16) for k, v in t.items()}
    Y = torch.empty(M, D, device="cuda", dtype=torch.bfloat16)
    ws = torch.empty(max(256, api.fdl_llama_ffn_workspace_bytes("bf16", M, D, H)), dtype=torch.uint8, device="cuda")
    rows = [5, M - 1]
    for r in rows:
        d["X"][r, 1] = float("inf")
    api.fdl_llama_ffn_forward("bf16", d["X"], d["Wg"], d["Wu"], d["Wd"], Y, ws)
    torch.cuda.synchronize()
    assert torch.all(Y[rows] == float("inf"))
    rest = [r for r in range(M) if r not in rows]
    assert torch.isfinite(Y[rest].float()).all()
