"""Precision of the 16 x 16 tile kernels where their sums could cancel or drift, against
the fp64 oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1410_4984_amd as gpps  # noqa: E402
from paper_1410_4984_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def t(a, dtype):
    return torch.tensor(a, dtype=dtype, device=DEV)


def grads(inp, dtype):
    g = gpps.psi_grads(t(inp["mu"], dtype), t(inp["S"], dtype), t(inp["Z"], dtype), inp["sigma_f2"], inp["l"],
                       inp["dL_dpsi0"], t(inp["dL_dPsi1"], dtype), t(inp["dL_dPsi2"], dtype), path="generic")
    torch.cuda.synchronize()
    return {k: v.double().cpu().numpy() for k, v in g.items()}


def rel(a, b):
    a, b = np.ravel(a), np.ravel(np.asarray(b, np.float64))
    return np.linalg.norm(a - b) / np.linalg.norm(b)


# Variances far above l^2 and inducing inputs a lengthscale apart: dZ and dl are sums of
# W (z_m' - z_m), sqrt(S) / l (up to 600 here) times smaller than the sums of W (mu - z)
# whose difference they are.  The exponents are up to 6 log(1 + 2 S / l^2) = 85 in
# magnitude, so their rounding leaves 85 2^-24 = 5e-6 of W in fp32 and 1e-14 in fp64; four
# times that, and in fp64 the oracle's own 5e-14 besides.
@pytest.mark.parametrize("dtype,tol", [(torch.float32, 2e-5), (torch.float64, 1e-13)])
@pytest.mark.parametrize("Q,l,groups", [(10, 0.005, 1), (12, 0.002, 1), (10, 0.05, 16), (20, 0.05, 1)])
def test_short_lengthscales_under_wide_variances(Q, l, groups, dtype, tol):
    print(f"[Q={Q} l={l} groups={groups} {dtype}]", flush=True)
    rng = np.random.default_rng(Q + groups)
    N, M = 300, 64
    c = 0.3 * rng.standard_normal((groups, Q)) if groups == 1 else rng.standard_normal((groups, Q))
    Z = (c[:, None, :] + l * rng.standard_normal((groups, M // groups, Q))).reshape(M, Q)
    A = rng.standard_normal((M, M))
    inp = synth.to_f32({"mu": c.mean(0) + 0.7 * rng.standard_normal((N, Q)), "S": rng.uniform(0.5, 2.0, (N, Q)),
                        "Z": Z[rng.permutation(M)], "l": np.full(Q, l), "sigma_f2": 1.25, "dL_dpsi0": 0.75,
                        "dL_dPsi1": rng.standard_normal((N, M)), "dL_dPsi2": 0.5 * (A + A.T)})
    ref = oracle.psi_grads(inp["mu"], inp["S"], inp["Z"], inp["sigma_f2"], inp["l"], inp["dL_dpsi0"],
                           inp["dL_dPsi1"], inp["dL_dPsi2"])
    got = grads(inp, dtype)
    err = {k: rel(got[k], v) for k, v in ref.items()}
    print({k: f"{e:.1e}" for k, e in err.items()}, flush=True)
    assert max(err.values()) <= tol, err


# Equal rows: every addition to dZ, dl and dsf2 may round the same way, the k-th of n by up
# to k / n 2^-p of their sum, so n additions in one go by n / 2 2^-p.  The kernels add 128
# rows, then the chunk's groups of 128 (at most 20 here), then the chunks (512 / 8 and 8):
# below 128 2^-p with the terms' own scalings.  One row's gradient times N is the reference:
# the terms are the same.
@pytest.mark.parametrize("dtype,ulp", [(torch.float32, 2.0 ** -24), (torch.float64, 2.0 ** -53)])
@pytest.mark.parametrize("N,M,Q", [(40000, 2048, 5), (65536, 300, 20), (131, 40, 6), (257, 200, 4)])
def test_gradient_sums_of_many_equal_rows(N, M, Q, dtype, ulp):
    print(f"[equal rows N={N} M={M} Q={Q} {dtype}]", flush=True)
    rng = np.random.default_rng(N + M)
    row = {"mu": 0.3 * rng.standard_normal((1, Q)), "S": rng.uniform(0.1, 0.5, (1, Q))}
    Z, l = t(0.5 * rng.standard_normal((M, Q)), dtype), rng.uniform(0.8, 1.6, Q)
    G1, G2 = t(rng.uniform(0.5, 1.0, (1, M)), dtype), t(rng.uniform(0.5, 1.0, (M, M)) / M, dtype)
    out = []
    for n in (1, N):
        g = gpps.psi_grads(*(t(row[k], dtype).repeat(n, 1) for k in ("mu", "S")), Z, 1.25, l, 0.0,
                           G1.repeat(n, 1), G2, path="generic")
        torch.cuda.synchronize()
        out.append({k: g[k].double().cpu().numpy() for k in ("dZ", "dl", "dsigma_f2")})
    err = {k: np.abs(out[1][k] / (N * out[0][k]) - 1.0).max() / ulp for k in out[0]}
    print({k: f"{e:.0f} ulp" for k, e in err.items()}, flush=True)
    assert max(err.values()) <= 128, err


# The exponent of Psi2 where few rows count, of a size of 32 .. 64 in powers of two here: it is
# rounded once at that size, 0.29 ulp ln 2 = 1.4e-15 of Psi2, and the roundings at half of it
# and below shall add no more than that again.  Reference in extended precision.
def test_exponent_rounding_f64(Q=30, tol=2e-15):
    N, M, L = 200, 64, np.longdouble
    errs = []
    for seed in range(6):
        inp = synth.random_inputs(N, M, Q, seed=seed)
        mu, S, Z, l = (inp[k].astype(L) for k in ("mu", "S", "Z", "l"))
        C = -(((Z[:, None] - Z[None]) / l) ** 2).sum(-1) / 4
        ref = np.zeros((M, M), L)
        for n in range(N):
            lp2 = 2 * np.log(L(inp["sigma_f2"])) - np.log1p(2 * S[n] / l**2).sum() / 2
            d = mu[n] - (Z[:, None] + Z[None]) / 2
            ref += np.exp(lp2 + C - (d * d / (l**2 + 2 * S[n])).sum(-1))
        f64 = torch.float64
        P2 = gpps.psi_stats(t(inp["mu"], f64), t(inp["S"], f64), t(inp["Z"], f64), inp["sigma_f2"], inp["l"])[2]
        errs.append(float(np.linalg.norm(P2.cpu().numpy() - ref) / np.linalg.norm(ref)))
    print([f"{e:.1e}" for e in errs], flush=True)
    assert np.sqrt(np.mean(np.square(errs))) <= tol, errs


# Statistics of so many inducing inputs that the forward's tasks take a few chunks each and
# more than one round of workgroups (M from about 1000 on, with the region's room for it or
# without), against the oracle; tolerances of the parity tests.
@pytest.mark.parametrize("dtype,tol", [(torch.float32, 1e-4), (torch.float64, 1e-12)])
@pytest.mark.parametrize("N,M,Q", [(40, 2048, 5), (37, 1500, 6), (18, 3000, 9), (9, 1030, 33)])
def test_statistics_in_several_rounds(N, M, Q, dtype, tol):
    print(f"[several rounds N={N} M={M} Q={Q} {dtype}]", flush=True)
    inp = synth.to_f32(synth.random_inputs(N, M, Q, seed=M))
    ws = torch.full((gpps.workspace_bytes(dtype, N, M, Q),), 0x7F, dtype=torch.uint8, device=DEV)
    got = gpps.psi_stats(t(inp["mu"], dtype), t(inp["S"], dtype), t(inp["Z"], dtype), inp["sigma_f2"], inp["l"],
                         workspace=ws, path="generic")
    ref = oracle.psi_stats(inp["mu"], inp["S"], inp["Z"], inp["sigma_f2"], inp["l"])
    for k, a, b in zip(("psi0", "Psi1", "Psi2"), got, ref):
        assert rel(a.double().cpu().numpy(), b) <= tol, k
    assert torch.equal(got[2], got[2].T)


# Both sides of the lines at which the gradients at Q = 3 and 4 go to the tile kernels or stay
# with the vector ones (fp32: M = 170, 384 and 512; fp64: always tiles), and Q = 2, which
# stays; upstream not symmetric; against the oracle, tolerances of the parity tests.
@pytest.mark.parametrize("dtype,tol", [(torch.float32, 1e-4), (torch.float64, 1e-12)])
@pytest.mark.parametrize("M", [7, 128, 129, 170, 171, 384, 385, 512, 513])
@pytest.mark.parametrize("Q", [2, 3, 4])
def test_gradients_around_the_dispatch_lines(M, Q, dtype, tol):
    print(f"[dispatch lines M={M} Q={Q} {dtype}]", flush=True)
    inp = synth.to_f32(synth.random_inputs(33, M, Q, seed=M + Q))
    inp["dL_dPsi2"] = np.float32(inp["dL_dPsi2"] + np.triu(np.ones((M, M)), 1))
    got = grads(inp, dtype)
    ref = oracle.psi_grads(inp["mu"], inp["S"], inp["Z"], inp["sigma_f2"], inp["l"], inp["dL_dpsi0"],
                           inp["dL_dPsi1"], inp["dL_dPsi2"])
    for k, v in ref.items():
        assert rel(got[k], v) <= tol, k
