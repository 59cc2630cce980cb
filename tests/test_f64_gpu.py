"""The double-precision matrix-core kernels against the fp64 oracle, at the sizes
where they can go wrong: every register width (Q at both ends of each), partial
and single 16-blocks of M, waves with one column block and without any, several
column groups, z staged in windows, one row and odd row counts, and rows whose
exponents leave the fast exponential's range.

Tolerance 1e-12 (relative Frobenius): the exponents here are below 100 in
magnitude, so a rounding of each is below 100 2^-53 = 1.1e-14, and a sum of Q <= 64
such terms in another order below 64 times that.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1410_4984_amd as gpps  # noqa: E402
from paper_1410_4984_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TOL = 1e-12


def t(a):
    return None if a is None else torch.tensor(a, dtype=torch.float64, device=DEV)


def call(inp, G1=True, G2=True):
    N, Q = inp["mu"].shape
    M = inp["Z"].shape[0]
    ws = torch.full((gpps.workspace_bytes(torch.float64, N, M, Q),), 0x7F, dtype=torch.uint8, device=DEV)
    mu, S, Z = t(inp["mu"]), t(inp["S"]), t(inp["Z"])
    psi0, P1, P2 = gpps.psi_stats(mu, S, Z, inp["sigma_f2"], inp["l"], workspace=ws)
    ws.fill_(0x7F)
    g = gpps.psi_grads(mu, S, Z, inp["sigma_f2"], inp["l"], inp["dL_dpsi0"],
                       t(inp["dL_dPsi1"]) if G1 else None, t(inp["dL_dPsi2"]) if G2 else None,
                       workspace=ws)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in dict(psi0=psi0, Psi1=P1, Psi2=P2, **g).items()}


def reference(inp, G1=True, G2=True):
    N, M = inp["mu"].shape[0], inp["Z"].shape[0]
    r0, R1, R2 = oracle.psi_stats(inp["mu"], inp["S"], inp["Z"], inp["sigma_f2"], inp["l"])
    g = oracle.psi_grads(inp["mu"], inp["S"], inp["Z"], inp["sigma_f2"], inp["l"], inp["dL_dpsi0"],
                         inp["dL_dPsi1"] if G1 else np.zeros((N, M)),
                         inp["dL_dPsi2"] if G2 else np.zeros((M, M)))
    return dict(psi0=r0, Psi1=R1, Psi2=R2, **g)


def check(got, ref, what):
    for k, v in ref.items():
        a, v = got[k].ravel(), np.asarray(v, np.float64).ravel()
        e = np.linalg.norm(a - v) / max(np.linalg.norm(v), 1e-300)
        assert e <= TOL, (what, k, e)
    assert np.array_equal(got["Psi2"], got["Psi2"].T)


@pytest.mark.parametrize("N,M,Q", [
    (1, 1, 5), (2, 15, 3), (3, 16, 4), (5, 17, 8), (17, 33, 9), (33, 32, 12), (19, 48, 13), (40, 49, 16),
    (31, 100, 17), (21, 129, 20), (18, 130, 2), (9, 257, 21), (12, 300, 24), (7, 100, 25), (6, 512, 30),
    (11, 97, 32), (10, 70, 33), (5, 600, 40), (8, 50, 41), (9, 33, 48), (7, 40, 49), (5, 65, 64),
    (3, 1100, 20), (300, 10, 10)])
def test_f64_edges(N, M, Q):
    print(f"[f64 N={N} M={M} Q={Q}]", flush=True)
    inp = synth.random_inputs(N, M, Q, seed=N + M + Q)
    inp["dL_dPsi2"] = inp["dL_dPsi2"] + np.triu(np.ones((M, M)), 1)  # not symmetric
    check(call(inp), reference(inp), (N, M, Q))


@pytest.mark.parametrize("G1,G2", [(True, False), (False, True), (False, False)])
def test_f64_null_upstream(G1, G2):
    inp = synth.random_inputs(23, 40, 7, seed=3)
    check(call(inp, G1, G2), reference(inp, G1, G2), (G1, G2))


def test_f64_far_rows():
    # exponents of 1e8 and beyond contribute nothing; an infinite mean gives a zero row of
    # Psi1 and no contribution to Psi2, as the closed forms do
    inp = synth.random_inputs(37, 40, 7, seed=4)
    inp["mu"][3] += 1e5
    inp["mu"][36, 2] = -1e8
    check(call(inp), reference(inp), "far")
    inp["mu"][5, 1] = np.inf
    got, ref = call(inp), reference(inp)
    for k in ("Psi1", "Psi2"):
        assert np.linalg.norm(got[k] - ref[k]) <= TOL * np.linalg.norm(ref[k]), k
    assert np.isnan(got["dmu"][5]).any() and np.isfinite(got["dmu"][4]).all()


def test_f64_nan_propagates():
    inp = synth.random_inputs(37, 40, 7, seed=5)
    inp["mu"][7, 3] = np.nan
    got = call(inp)
    assert np.isnan(got["Psi1"][7]).all() and np.isfinite(got["Psi1"][8]).all()
    assert np.isnan(got["Psi2"]).all() and np.isnan(got["dmu"][7]).all() and np.isnan(got["dZ"]).all()
    assert np.isfinite(got["dmu"][6]).all()
    inp = synth.random_inputs(37, 40, 7, seed=5)
    inp["Z"][17, 2] = np.nan
    got = call(inp)
    bad = np.zeros((40, 40), bool)
    bad[17] = bad[:, 17] = True
    assert np.array_equal(np.isnan(got["Psi2"]), bad)
    assert np.array_equal(np.isnan(got["Psi1"]).all(0), bad[17] & (np.arange(40) == 17))


def test_f64_accumulates_over_chunks():
    inp = synth.random_inputs(150, 50, 10, seed=6)
    whole = call(inp)
    mu, S, Z = t(inp["mu"]), t(inp["S"]), t(inp["Z"])
    G1, G2 = t(inp["dL_dPsi1"]), t(inp["dL_dPsi2"])
    out = gout = None
    rows = []
    for a, b in ((0, 61), (61, 150)):
        n = b - a
        P1 = torch.empty((n, 50), dtype=torch.float64, device=DEV)
        o = None if out is None else (out[0], P1, out[2])
        out = gpps.psi_stats(mu[a:b], S[a:b], Z, inp["sigma_f2"], inp["l"], accumulate=out is not None, out=o)
        go = None if gout is None else dict(gout, dmu=torch.empty((n, 10), dtype=torch.float64, device=DEV),
                                            dS=torch.empty((n, 10), dtype=torch.float64, device=DEV))
        gout = gpps.psi_grads(mu[a:b], S[a:b], Z, inp["sigma_f2"], inp["l"],
                              inp["dL_dpsi0"], G1[a:b], G2,
                              accumulate=gout is not None, out=go)
        rows.append((gout["dmu"], gout["dS"]))
    got = {"Psi2": out[2], "psi0": out[0], "dZ": gout["dZ"], "dl": gout["dl"], "dsigma_f2": gout["dsigma_f2"],
           "dmu": torch.cat([r[0] for r in rows]), "dS": torch.cat([r[1] for r in rows])}
    for k, v in got.items():
        v = v.cpu().numpy().ravel()
        assert np.linalg.norm(v - whole[k].ravel()) <= TOL * np.linalg.norm(whole[k]), k
