"""The row kernels at the edges of their row lengths: one wavefront, a pair of wavefronts or a workgroup per row, streamed
rows; rows that end inside a 16-byte vector; matrices of one row and of more rows than one pass holds.  Same bars as the
other parity tests (tests/harness.py), against the fp64 oracles."""
import numpy as np
import pytest
import torch

from oracle import fdl_oracle as O
from oracle import siblings_oracle as S
from paper_2509_14279_amd import api, inputs as I
import harness as H

pytestmark = pytest.mark.gpu

BF16_WIDTHS = [7, 129, 136, 504, 511, 512, 513, 1025, 1727, 2049, 4095, 4097, 8191, 8193, 8208, 16383, 16384, 16391, 32760, 32768, 32771]
F32_WIDTHS = [3, 257, 1023, 1026, 4097, 8192, 16383, 16388]
WIDTHS = [("bf16", n) for n in BF16_WIDTHS] + [("f32", n) for n in F32_WIDTHS]


@pytest.mark.parametrize("dtype,N", WIDTHS)
@pytest.mark.parametrize("M", [1, 1037])
def test_stand_alone_norms(dtype, N, M):
    print(f"[rows] {dtype} {M}x{N}", flush=True)
    t = I.generate_norm(dtype, M, N, seed=8000 + N + M)
    n = {k: v.numpy().astype(np.float64) for k, v in t.items()}
    dt = I.storage_torch_dtype(dtype)
    A = t["A"].to("cuda", dt)
    out = {"Y": H.Guarded((M, N), dt), "mean": H.Guarded((M,), torch.float32), "rstd": H.Guarded((M,), torch.float32),
           "R": H.Guarded((M, N), dt)}
    gamma, beta = t["gamma"].to("cuda"), t["beta"].to("cuda")
    api.fdl_layernorm_forward(dtype, A, gamma, beta, 1e-5, out["Y"].view, out["mean"].view, out["rstd"].view)
    api.fdl_rmsnorm_forward(dtype, A, gamma, 1e-5, out["R"].view)
    torch.cuda.synchronize()
    for k, g in out.items():
        assert g.intact(), f"kernel wrote outside the {k} buffer"
    ref = S.layernorm_forward(n["A"], n["gamma"], n["beta"], 1e-5)
    H.check(dtype, "Y", H.to_f64(out["Y"].view), ref["Y"])
    H.check(dtype, "mean", H.to_f64(out["mean"].view), ref["mean"])
    H.check(dtype, "R", H.to_f64(out["R"].view), S.rmsnorm_forward(n["A"], n["gamma"], 1e-5)["Y"])


@pytest.mark.parametrize("dtype,M,N", [("bf16", 37, 8193), ("bf16", 530, 16384), ("bf16", 65, 11570), ("bf16", 70, 16392),
                                       ("bf16", 2600, 1030), ("bf16", 300, 4093), ("f32", 70, 4100), ("f32", 33, 8190),
                                       ("f32", 2600, 515), ("f32", 40, 16390), ("bf16", 530, 32768),
                                       ("bf16", 33, 30003), ("bf16", 20, 32776),
                                       # segments of 4096 (bf16) and 2048 (fp32) columns: a last one of one element, of part
                                       # of a wavefront, whole; rows that share a workgroup in odd and even numbers; one row
                                       ("bf16", 1, 36865), ("bf16", 700, 32769), ("bf16", 2300, 40960), ("bf16", 33, 37000),
                                       # narrow rows: sixteen lanes each (to 128 and 64 columns), an element per thread in
                                       # the backward pass (to 256, where they are ragged or padded)
                                       ("bf16", 2600, 15), ("bf16", 33000, 17), ("bf16", 1037, 33), ("bf16", 37, 127),
                                       ("bf16", 300, 128), ("bf16", 70, 129), ("bf16", 70, 505), ("bf16", 33000, 504), ("bf16", 37, 511), ("bf16", 515, 255), ("f32", 2600, 17),
                                       # several rows per workgroup in the backward pass: a wavefront each, two each, at
                                       # their edges; row counts that leave wavefronts without a row
                                       ("bf16", 1, 64), ("bf16", 3, 65), ("bf16", 5, 256), ("bf16", 1037, 257), ("bf16", 1039, 512),
                                       ("bf16", 5, 513), ("bf16", 1037, 1016), ("bf16", 3, 1024), ("f32", 3, 256),
                                       ("f32", 1037, 257), ("f32", 1039, 512), ("f32", 5, 511), ("f32", 1, 63),
                                       ("f32", 33000, 7), ("f32", 500, 64), ("f32", 70, 65), ("f32", 41, 255),
                                       ("f32", 1, 18433), ("f32", 600, 16385), ("f32", 1300, 18432), ("f32", 37, 20001)])
def test_forward_and_backward_of_the_block(dtype, M, N):
    cfg = I.custom(dtype, M, 16, N, seed=8100 + M + N)
    print(f"[rows] {cfg.name}", flush=True)
    t = I.generate(cfg)
    got = H.run_fdl(cfg, t)
    n = {k: v.numpy().astype(np.float64) for k, v in t.items()}
    ref = O.forward_backward(n["X"], n["W"], n["b"], n["gamma"], n["beta"], n["dY"], cfg.eps)
    for k in H.OUTPUTS + ("mean",):
        H.check(dtype, k, H.to_f64(got[k]), ref[k])


# (the last four: rows that start at any element, spread over more wavefronts while they are few)
@pytest.mark.parametrize("N,M", [(4104, 5000), (8200, 5000), (12345, 5000), (16384, 5000), (16392, 5000), (20001, 5000),
                                 (32768, 5000), (1500, 4000), (3001, 2000), (5003, 1000), (8191, 1000)])
def test_rows_do_not_depend_on_the_rows_beside_them(N, M):
    # rows shared by two, four and eight wavefronts: a workgroup that walks several rows must give each the bits it has when
    # every workgroup holds one row (at most 256 rows: one trip)
    t = I.generate_norm("bf16", 256, N, seed=8200 + N)
    A = t["A"].to("cuda", torch.bfloat16)
    A = torch.cat([A.roll(k, 0) * (1.0 + k / 8) for k in range(20)])[:M].contiguous()
    gamma, beta = t["gamma"].to("cuda"), t["beta"].to("cuda")

    def run(A):
        m = A.shape[0]
        out = [torch.empty_like(A), torch.empty_like(A), torch.empty(m, device="cuda"), torch.empty(m, device="cuda")]
        api.fdl_rmsnorm_forward("bf16", A, gamma, 1e-5, out[0])
        api.fdl_layernorm_forward("bf16", A, gamma, beta, 1e-5, *out[1:])
        return out

    for whole, parts in zip(run(A), zip(*[run(A[i:i + 256].contiguous()) for i in range(0, M, 256)])):
        assert torch.equal(whole.view(torch.uint8), torch.cat(parts).view(torch.uint8))


@pytest.mark.parametrize("M,K,N", [(300, 100, 1000), (300, 77, 4095), (300, 64, 8200), (200, 64, 12345), (200, 64, 16384),
                                   (100, 64, 30001), (100, 64, 32769), (40, 32, 65536)])
def test_statistics_of_nearly_constant_rows(M, K, N):
    # Z is 8 with a spread of one bf16 step (1/16) and less: GELU(z) = z to fp32, sums of such values are exact, and squared
    # deviations of few distinct sizes make every rounding of a long chain go the same way.  The saved mean is the rounded
    # exact one (2^-24); 1/rstd^2 carries at most the chain of a vector's eight squares (8 roundings) and rstd its own
    # rounding: 5 x 2^-24.
    cfg = I.custom("bf16", M, K, N, seed=8300 + M + N)
    t = I.generate(cfg, with_dY=False)
    t["W"] = (t["W"] * 0.02).to(torch.bfloat16).float()
    t["b"] = t["b"] + 8.0
    got = H.run_fdl(cfg, t, backward=False)
    A = O.gelu(H.to_f64(got["Z"]))
    mean, rstd = A.mean(axis=1), (A.var(axis=1) + cfg.eps) ** -0.5
    assert np.abs(H.to_f64(got["mean"]) / mean - 1).max() <= 2.0 ** -24 * 1.001
    assert np.abs(H.to_f64(got["rstd"]) / rstd - 1).max() <= 5 * 2.0 ** -24


# (a wavefront per row, two; 6656 and 11520 rows leave wavefronts without a pair of rows on the last round)
BLOCKED = [(2560, 2560, 512), (5120, 1024, 1024), (12288, 3584, 512), (6656, 1024, 512), (11520, 512, 768)]


@pytest.mark.parametrize("M,K,N", BLOCKED)
def test_blocked_gradients_of_narrow_rows(M, K, N):
    # dZ in 32 x 32 blocks, written by a wavefront or two per row (test_routes_host.py: all but the first)
    cfg = I.custom("bf16", M, K, N, seed=8200 + N)
    t = I.generate(cfg)
    got = H.run_fdl(cfg, t)
    n = {k: v.numpy().astype(np.float64) for k, v in t.items()}
    ref = O.forward_backward(n["X"], n["W"], n["b"], n["gamma"], n["beta"], n["dY"], cfg.eps)
    for k in H.OUTPUTS + ("Z", "mean"):
        H.check("bf16", k, H.to_f64(got[k]), ref[k])
