"""GELU and its derivative in fp64 (fp32 storage): arguments on, beside and half way between the nodes of the kernels' table,
at its end and past it, in each form of the row kernels.  One row with K = 1, X = 1, W = z, b = 0 makes the pre-activations the
numbers z themselves and dW the row's dZ, element by element.

Bounds: one rounding to fp32 (2^-24) of the result, and 1e-12 of the sum of the magnitudes that cancel in it (the saved fp32
statistics are taken as they are; sums of up to 20000 fp64 terms, and the oracle's erfc, which rounds its argument: 2e-13 of
Phi(-38)); where the result is below the smallest normal fp32 number, half the spacing there (2^-150)."""
import numpy as np
import pytest
import torch

from oracle import fdl_oracle as O
from paper_2509_14279_amd import inputs as I
import harness as H

pytestmark = pytest.mark.gpu


def arguments(N):
    """N arguments: magnitudes around nodes (multiples of 1/64) and midpoints from 0 to beyond 13.25, both signs."""
    k = np.concatenate([np.arange(0, 200), np.arange(200, 849, 7), np.arange(840, 850)]) / 64.0
    e = np.float32(1e-6)
    a = np.concatenate([k, k + e, np.maximum(k - e, 0), k + 1 / 128, k + 1 / 128 + e, [1e-30, 1e-8, 14.5, 20.0, 38.0, 100.0]])
    z = np.concatenate([a, -a]).astype(np.float32)
    z = np.random.default_rng(N).permutation(z)
    return np.resize(z, N)


# sixteen lanes per row; one, two, four vectors per thread; 1024 threads; segments; the backward kernels' forms likewise
@pytest.mark.parametrize("N", [47, 200, 1000, 1537, 2048, 3001, 4096, 7000, 16001, 20000])
def test_gelu_and_its_derivative(N):
    z = arguments(N)
    rng = np.random.default_rng(N + 1)
    t = {"X": torch.ones(1, 1), "W": torch.from_numpy(z)[:, None].contiguous(), "b": torch.zeros(N),
         "gamma": torch.from_numpy((1 + 0.3 * rng.standard_normal(N)).astype(np.float32)),
         "beta": torch.from_numpy((0.3 * rng.standard_normal(N)).astype(np.float32)),
         "dY": torch.from_numpy(rng.standard_normal((1, N)).astype(np.float32))}
    cfg = I.custom("f32", 1, 1, N, seed=0)
    got = {k: H.to_f64(v) for k, v in H.run_fdl(cfg, t).items()}
    Z = z.astype(np.float64)
    assert np.array_equal(got["Z"][0], Z)
    A, mean, rstd = O.gelu(Z), got["mean"][0], got["rstd"][0]
    exact_mean = A.mean()
    exact_rstd = 1.0 / np.sqrt(A.var() + cfg.eps)
    u = 2.0 ** -24
    assert abs(mean - exact_mean) <= u * abs(exact_mean) + 1e-12 * np.abs(A).max()
    assert abs(rstd - exact_rstd) <= (u + 1e-12) * exact_rstd
    g64 = {k: t[k].numpy().astype(np.float64) for k in ("gamma", "beta", "dY")}
    Y = (A - exact_mean) * exact_rstd * g64["gamma"] + g64["beta"]
    S = (np.abs(A) + abs(exact_mean)) * exact_rstd * np.abs(g64["gamma"]) + np.abs(g64["beta"])
    # (the segments' second kernel normalises with the same fp64 statistics)
    assert np.all(np.abs(got["Y"][0] - Y) <= u * np.abs(Y) + 1e-12 * S)
    ah = (A - mean) * rstd
    g = g64["dY"][0] * g64["gamma"]
    c1, c2 = g.mean(), (g * ah).mean()
    d = O.gelu_grad(Z)
    dZ = rstd * (g - c1 - ah * c2) * d
    S = rstd * (np.abs(g) + np.abs(g).mean() + np.abs(ah) * np.abs(g * ah).mean()) * (np.abs(O.Phi(Z)) + np.abs(Z * O.phi(Z)))
    assert np.all(np.abs(got["dW"][:, 0] - dZ) <= u * np.abs(dZ) + 1e-12 * S + 2.0 ** -150)
    assert np.all(np.abs(got["dgamma"] - g64["dY"][0] * ah) <= u * np.abs(g64["dY"][0] * ah) + 1e-12 * np.abs(g64["dY"][0]) * (np.abs(A) + abs(mean)) * rstd)


# (one vector, two, eight elements per thread; a wavefront's rows; the two kernels for long rows)
@pytest.mark.parametrize("N", [47, 200, 1000, 1537, 4096, 5000, 20000])
def test_gradients_far_out(N):
    """GELU'(z) = Phi(z) + z phi(z) below -13 is small, not zero: times a large upstream gradient it is an ordinary number."""
    rng = np.random.default_rng(N + 2)
    z = rng.standard_normal(N).astype(np.float32)
    far = rng.permutation(N)[:N // 3]
    z[far] = -np.concatenate([np.linspace(13.2, 13.3, len(far) - len(far) // 2), np.linspace(13.3, 17.0, len(far) // 2)])
    t = {"X": torch.ones(1, 1), "W": torch.from_numpy(z)[:, None].contiguous(), "b": torch.zeros(N), "gamma": torch.ones(N),
         "beta": torch.zeros(N), "dY": torch.from_numpy((1e30 * rng.standard_normal((1, N))).astype(np.float32))}
    cfg = I.custom("f32", 1, 1, N, seed=0)
    got = {k: H.to_f64(v) for k, v in H.run_fdl(cfg, t).items()}
    Z, mean, rstd = z.astype(np.float64), got["mean"][0], got["rstd"][0]
    ah, g = (O.gelu(Z) - mean) * rstd, t["dY"].numpy().astype(np.float64)[0]
    factor = rstd * (g - g.mean() - ah * (g * ah).mean())
    S = rstd * (np.abs(g) + np.abs(g).mean() + np.abs(ah) * np.abs(g * ah).mean())
    dZ = factor * O.gelu_grad(Z)
    assert np.abs(dZ[far]).min() > 0 and np.abs(dZ[far]).max() > 1e-8
    d = np.abs(O.Phi(Z)) + np.abs(Z * O.phi(Z))
    assert np.all(np.abs(got["dW"][:, 0] - dZ) <= 2.0 ** -24 * np.abs(dZ) + 1e-12 * S * d + 2.0 ** -150)


# (the forms of the row kernels as above)
@pytest.mark.parametrize("N", [47, 200, 1000, 1537, 4096, 5000, 20000])
def test_very_large_arguments(N):
    """Phi is 0 or 1 for any finite argument that is large, also where its square leaves no digit of it: GELU(z) is 0 or z, and the
    normalised row is that of the few elements of the largest magnitude."""
    rng = np.random.default_rng(N + 3)
    z = rng.standard_normal(N).astype(np.float32)
    at = rng.permutation(N)[:9]
    z[at] = [1e25, -1e25, 1e30, -1e30, 3e9, -3e9, -3.4e38, 2e30, -1e15]
    t = {"X": torch.ones(1, 1), "W": torch.from_numpy(z)[:, None].contiguous(), "b": torch.zeros(N), "gamma": torch.ones(N),
         "beta": torch.zeros(N), "dY": torch.from_numpy(rng.standard_normal((1, N)).astype(np.float32))}
    cfg = I.custom("f32", 1, 1, N, seed=0)
    got = {k: H.to_f64(v) for k, v in H.run_fdl(cfg, t).items()}
    Z, mean, rstd = z.astype(np.float64), got["mean"][0], got["rstd"][0]
    A, u = O.gelu(Z), 2.0 ** -24
    assert A[at[0]] == Z[at[0]] and A[at[6]] == 0
    exact_mean, exact_rstd = A.mean(), 1.0 / np.sqrt(A.var() + cfg.eps)
    assert abs(mean - exact_mean) <= (u + 1e-12) * exact_mean and abs(rstd - exact_rstd) <= (u + 1e-12) * exact_rstd
    Y = (A - exact_mean) * exact_rstd
    assert np.all(np.abs(got["Y"][0] - Y) <= u * np.abs(Y) + 1e-12 * (np.abs(A) + exact_mean) * exact_rstd)
    ah, g = (A - mean) * rstd, t["dY"].numpy().astype(np.float64)[0]
    dZ = rstd * (g - g.mean() - ah * (g * ah).mean()) * O.gelu_grad(Z)
    S = rstd * (np.abs(g) + np.abs(g).mean() + np.abs(ah) * np.abs(g * ah).mean()) * (np.abs(O.Phi(Z)) + np.abs(Z * O.phi(Z)))
    assert np.isfinite(dZ).all()
    assert np.all(np.abs(got["dW"][:, 0] - dZ) <= u * np.abs(dZ) + 1e-12 * S + 2.0 ** -150)


def test_infinities_and_nan():
    # as the library's erfc and exp: GELU(-inf) and whatever a row with a NaN or an infinity gives are NaN, rows beside it are not
    for bad in (np.inf, -np.inf, np.nan):
        cfg = I.custom("f32", 3, 1, 130, seed=3)
        t = I.generate(cfg)
        t["X"][1, 0] = bad
        got = {k: H.to_f64(v) for k, v in H.run_fdl(cfg, t).items()}
        assert np.isnan(got["Y"][1]).all() and np.isnan(got["dX"][1]).all()
        assert np.isfinite(got["Y"][[0, 2]]).all() and np.isfinite(got["dX"][[0, 2]]).all()
    # GELU(inf) is infinite, and so is the mean of a row that has it and no NaN
    cfg = I.custom("f32", 1, 1, 130, seed=3)
    t = I.generate(cfg)
    t["X"][0, 0] = 1.0
    t["W"][7, 0] = np.inf
    assert H.to_f64(H.run_fdl(cfg, t)["mean"])[0] == np.inf
