"""Normalisation of rows of exactly 4096 and 8192 columns, which four or eight wavefronts share: one row, a workgroup's remainder, more
rows than are in flight at once, and (stand-alone norms) input and output of as many bytes as the memory-side cache, half as many more,
twice as many."""
import pytest
import torch

from paper_2509_14279_amd import api, inputs as I

pytestmark = pytest.mark.gpu
EPS = 1e-5


def near(got, ref, rel, what):
    err = (got.double() - ref).abs()
    assert torch.all(err <= rel * ref.abs() + 1e-7), (what, err.max().item())


@pytest.mark.parametrize("N", [4096, 8192])
@pytest.mark.parametrize("M", [1, 37, 1025, 5001])
def test_stand_alone_norms(M, N):
    print(f"[even rows] norm {M}x{N}", flush=True)
    t = {k: v.to("cuda") for k, v in I.generate_norm("bf16", M, N, seed=M + N).items()}
    A, gamma, beta = t["A"].bfloat16(), t["gamma"], t["beta"]
    Y, R = torch.empty_like(A), torch.empty_like(A)
    mean, rstd = torch.empty(M, device="cuda"), torch.empty(M, device="cuda")
    api.fdl_layernorm_forward("bf16", A, gamma, beta, EPS, Y, mean, rstd)
    api.fdl_rmsnorm_forward("bf16", A, gamma, EPS, R)
    torch.cuda.synchronize()
    a = A.double()
    mu, rs = a.mean(1), (a.var(1, unbiased=False) + EPS).rsqrt()
    # fp32 sums of N terms in short chains: 2^-20 is 16 of their roundings; the outputs are rounded to bf16 once (2^-9)
    near(mean, mu, 2.0 ** -20, "mean")
    near(rstd, rs, 2.0 ** -20, "rstd")
    x = (a - mu[:, None]) * rs[:, None] * gamma.double()
    assert torch.all((Y.double() - (x + beta.double())).abs() <= 2.0 ** -8 * (x + beta.double()).abs() + 2.0 ** -18 * (x.abs() + beta.abs() + 1))
    near(R, a * (a.square().mean(1, keepdim=True) + EPS).rsqrt() * gamma.double(), 2.0 ** -8, "rms")


@pytest.mark.parametrize("M,N", [(1, 4096), (1024, 4096), (1025, 4096), (4096, 4096), (4500, 4096), (3, 8192), (2000, 8192)])
def test_normalised_gelu(M, N):
    print(f"[even rows] block {M}x{N}", flush=True)
    t = {k: v.to("cuda") for k, v in I.generate(I.custom("bf16", M, 8, N, seed=M + N), with_dY=False).items()}
    X, W = t["X"].bfloat16(), t["W"].bfloat16()
    ws = torch.empty(api.fdl_workspace_bytes("bf16", M, 8, N), dtype=torch.uint8, device="cuda")
    Y, Z = (torch.empty(M, N, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    mean, rstd = torch.empty(M, device="cuda"), torch.empty(M, device="cuda")
    api.fdl_forward("bf16", X, W, t["b"], t["gamma"], t["beta"], EPS, Y, Z, mean, rstd, ws)
    torch.cuda.synchronize()
    z = Z.double()
    a = z * torch.erfc(z * -(0.5 ** 0.5)) * 0.5
    mu, rs = a.mean(1), (a.var(1, unbiased=False) + EPS).rsqrt()
    near(mean, mu, 2.0 ** -22, "mean")          # fp64 sums of fp32 values, rounded to fp32 once
    near(rstd, rs, 2.0 ** -22, "rstd")
    x, b = (a - mu[:, None]) * rs[:, None] * t["gamma"].double(), t["beta"].double()
    assert torch.all((Y.double() - (x + b)).abs() <= 2.0 ** -8 * (x + b).abs() + 2.0 ** -18 * (x.abs() + b.abs() + 1))


# input and output together: 256 MB less a row; 256 MB, from which on loads and stores go past the caches; 384 MB less a row; 384 MB, from
# which on each die has a stretch of the rows; a row more; 512 MB and a little
@pytest.mark.parametrize("N,M", [(n, m) for n in (4096, 8192) for m in ((1 << 28) // (4 * n) - 1, (1 << 28) // (4 * n), (3 << 27) // (4 * n) - 1,
                                                                       (3 << 27) // (4 * n), (3 << 27) // (4 * n) + 1, (1 << 28) // (2 * n) + 5)])
def test_rows_past_the_caches_have_the_same_bits(N, M):
    t = {k: v.to("cuda") for k, v in I.generate_norm("bf16", 300, N, seed=N).items()}
    A, gamma, beta = t["A"].bfloat16(), t["gamma"], t["beta"]
    print(f"[even rows] {M}x{N}", flush=True)

    def run(A):
        Y, R, m, r = torch.empty_like(A), torch.empty_like(A), torch.empty(len(A), device="cuda"), torch.empty(len(A), device="cuda")
        api.fdl_layernorm_forward("bf16", A, gamma, beta, EPS, Y, m, r)
        api.fdl_rmsnorm_forward("bf16", A, gamma, EPS, R)
        return Y, R, m, r

    big = run(A.repeat((M + 299) // 300, 1)[:M].contiguous())
    for whole, part in zip(big, run(A)):
        for i in (0, 300, M // 300 * 300 - 300):
            assert torch.equal(whole[i:i + 300].view(torch.uint8), part[:len(whole[i:i + 300])].view(torch.uint8))
        tail = M % 300
        assert torch.equal(whole[M - tail:].view(torch.uint8), part[:tail].view(torch.uint8))


# rows of the block run in one of three forms by their number (the last, from 384 MB of input and output on, not where it normalises in
# place); small integers, whose products' sums are exact, give every batch the same pre-activations, and sums in fp64 leave the statistics'
# fp32 roundings the same
@pytest.mark.parametrize("N,batches", [(4096, (1, 1000, 1024, 1025, 4095, 4096, 5000, 24575, 24576, 24583)), (8192, (1, 700, 2000, 12287, 12288, 12290))])
def test_rows_of_the_block_do_not_depend_on_the_rows_beside_them(N, batches):
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    X = torch.randint(-3, 4, (max(batches), 8), device="cuda", generator=g).to(torch.bfloat16)
    W = (torch.randint(-3, 4, (N, 8), device="cuda", generator=g) / 8).to(torch.bfloat16)
    b, gamma, beta = (torch.randn(N, device="cuda", generator=g) * 0.1 + c for c in (0.0, 1.0, 0.0))

    def run(M):
        ws = torch.empty(api.fdl_workspace_bytes("bf16", M, 8, N), dtype=torch.uint8, device="cuda")
        Y, Z = (torch.empty(M, N, device="cuda", dtype=torch.bfloat16) for _ in range(2))
        mean, rstd = torch.empty(M, device="cuda"), torch.empty(M, device="cuda")
        api.fdl_forward("bf16", X[:M].contiguous(), W, b, gamma, beta, EPS, Y, Z, mean, rstd, ws)
        return Y, Z, mean, rstd

    most = run(max(batches))
    for M in batches:
        print(f"[even rows] block {M} of {N}", flush=True)
        for got, ref in zip(run(M), most):
            assert torch.equal(got.view(torch.uint8), ref[:M].contiguous().view(torch.uint8))
    M = max(batches)
    Y = torch.empty(M, N, device="cuda", dtype=torch.bfloat16)
    ws = torch.empty(max(256, api.fdl_forward_inference_workspace_bytes("bf16", M, 8, N)), dtype=torch.uint8, device="cuda")
    api.fdl_forward_inference("bf16", X, W, b, gamma, beta, EPS, Y, ws)
    assert torch.equal(Y.view(torch.uint8), most[0].view(torch.uint8))
