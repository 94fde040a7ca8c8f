"""The bias of the 256 x 256 tiles' forward product, which a workgroup fetches a tile ahead: several tiles per workgroup and the
shortest reduction, one pipeline round, with a bias that differs from column to column by more than the products do."""
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
