"""fp32 storage, layers small enough for 32 x 32 tiles whose reduction a workgroup's wavefronts share: Linear+ReLU (every operand
orientation, every epilogue, the column sums) at the tiles' and steps' edges, against fp64."""
import pytest
import torch

from paper_2509_14279_amd import api, inputs as I

pytestmark = pytest.mark.gpu


# one element; a tile and its neighbours; reductions of less than, exactly and more than a step of 16, a round of 256; the largest
@pytest.mark.parametrize("M,K,N", [(1, 1, 1), (3, 2, 5), (31, 16, 33), (32, 15, 32), (33, 17, 31), (64, 63, 65), (17, 256, 40),
                                   (40, 257, 17), (100, 300, 129), (255, 255, 257), (256, 256, 256), (300, 300, 700), (777, 333, 300),
                                   (512, 512, 512), (1000, 200, 300), (1500, 300, 256), (1024, 64, 1023)])
def test_linear_relu_of_small_layers(M, K, N):
    print(f"[small f64] {M}x{K}x{N}", flush=True)
    t = {k: v.to("cuda") for k, v in I.generate(I.custom("f32", M, K, N, seed=M + 3 * K + N)).items()}
    X, W, b, dY = (t[k].contiguous() for k in ("X", "W", "b", "dY"))
    ws = torch.full((max(256, api.fdl_linear_relu_workspace_bytes("f32", M, K, N)),), 0xA5, dtype=torch.uint8, device="cuda")
    Y, dX, dW, db = (torch.full(s, float("nan"), device="cuda") for s in ((M, N), (M, K), (N, K), (N,)))
    api.fdl_linear_relu_forward("f32", X, W, b, Y, ws)
    api.fdl_linear_relu_backward("f32", dY, X, W, b, dX, dW, db, ws)
    torch.cuda.synchronize()
    x, w, d = X.double(), W.double(), dY.double()
    z = x @ w.t() + b.double()
    g = torch.where(z > 0, d, torch.zeros_like(d))
    # fp64 sums (an ulp of 2^-53 per term, with room), rounded to fp32 once
    for got, ref, terms in ((Y, z.clamp(min=0), x.abs() @ w.abs().t() + b.double().abs()), (dX, g @ w, g.abs() @ w.abs()),
                            (dW, g.t() @ x, g.abs().t() @ x.abs()), (db, g.sum(0), g.abs().sum(0))):
        assert torch.all((got.double() - ref).abs() <= 2.0 ** -23 * ref.abs() + 2.0 ** -40 * terms + 1e-45)
