"""The bias of the 256 x 256 tiles' forward product, which a workgroup fetches at the top of a tile: several tiles per workgroup and the
shortest reduction, one pipeline round, with a bias that differs from column to column by more than the products do; and, on every
kernel that forms a forward product, a bias far above the products, added once, to the finished sum."""
import pytest
import torch

from paper_2509_14279_amd import api, inputs as I

pytestmark = pytest.mark.gpu


# whole tiles, more of them, ragged rows, padded columns, two rounds
@pytest.mark.parametrize("M,K,N", [(12032, 128, 6144), (16384, 128, 8448), (12100, 128, 6144), (8760, 128, 5167), (12032, 256, 6144)])
def test_bias_of_every_tile(M, K, N):
    print(f"[bias] {M}x{K}x{N}", flush=True)
    t = I.generate(I.custom("bf16", M, K, N, seed=M + N))
    X, W = (t[k].to("cuda", torch.bfloat16) for k in ("X", "W"))
    b = (torch.arange(N, device="cuda", dtype=torch.float32) * 37 % 1024 + 8.25)
    Y = torch.empty(M, N, device="cuda", dtype=torch.bfloat16)
    ws = torch.empty(max(256, api.fdl_linear_relu_workspace_bytes("bf16", M, K, N)), dtype=torch.uint8, device="cuda")
    api.fdl_linear_relu_forward("bf16", X, W, b, Y, ws)
    torch.cuda.synchronize()
    ref = torch.clamp(X.float() @ W.float().t() + b, min=0)
    # half a unit of bf16, and the fp32 sums of both sides: K + 1 additions of at most 2^-24 of a partial sum each
    terms = X.float().abs() @ W.float().abs().t() + b
    bound = ref * 2.0 ** -8 + 2 * (K + 1) * 2.0 ** -24 * terms
    assert torch.all((Y.float() - ref).abs() <= bound)


# 256 x 256 tiles: as they are, ragged rows, padded on X as it is and as a copy, split, split and ragged or padded; 128 x 128, whole and
# split; few rows; generic (test_routes_host.py)
EVERY = [(12032, 1024, 6144), (8425, 768, 1536), (8760, 128, 5167), (4529, 157, 6144), (1280, 3072, 3584), (1337, 3072, 3328),
         (2062, 2651, 2073), (4700, 256, 768), (512, 4096, 2048), (32, 2048, 1003), (4864, 151, 70)]


@pytest.mark.parametrize("M,K,N", EVERY)
def test_a_large_bias_is_rounded_once(M, K, N):
    print(f"[bias] once {M}x{K}x{N}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(M + K + N)
    # small integers: their products' sums are exact in fp32 in any order (16 K < 2^24), so that the one rounding of sum + bias, then of
    # the result to bf16, is all that a value may show; the bias has 24 bits
    X, W = (torch.randint(-4, 5, s, device="cuda", generator=g).to(torch.bfloat16) for s in ((M, K), (N, K)))
    b = torch.randn(N, device="cuda", generator=g) * 2.0 ** 12 + 0.1
    S = X.float() @ W.float().t()
    assert torch.equal(S[:64].double(), X[:64].double() @ W.double().t())
    ref = (S + b).to(torch.bfloat16)
    Y, Z = (torch.empty(M, N, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    mean, rstd, ones, zeros = (torch.full((n,), v, device="cuda") for n, v in ((M, 0.0), (M, 0.0), (N, 1.0), (N, 0.0)))
    ws = torch.empty(max(256, api.fdl_workspace_bytes("bf16", M, K, N), api.fdl_linear_relu_workspace_bytes("bf16", M, K, N)),
                     dtype=torch.uint8, device="cuda")
    api.fdl_forward("bf16", X, W, b, ones, zeros, 1e-5, Y, Z, mean, rstd, ws)
    torch.cuda.synchronize()
    assert torch.equal(Z, ref)
    api.fdl_linear_relu_forward("bf16", X, W, b, Y, ws)
    dY = torch.ones(M, N, device="cuda", dtype=torch.bfloat16)
    dX, dW, db = torch.empty_like(X), torch.empty_like(W), torch.empty(N, device="cuda")
    api.fdl_linear_relu_backward("bf16", dY, X, W, b, dX, dW, db, ws)
    torch.cuda.synchronize()
    assert torch.equal(Y, ref.clamp(min=0))
    assert torch.equal(db, (ref > 0).sum(0).float())       # (counts: exact)
