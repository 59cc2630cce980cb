"""The single-precision 16 x 16 tile kernels of the generic path against the fp64
oracle, at the sizes where they can go wrong: every register width (Q at both ends of
each), partial and single 16-blocks of M, waves with one column block and without any,
several column groups, z staged in windows, chunk counts at the edges of the reduce's
splits, one row and odd row counts, shapes past the matrix-core path's limits, calls
that its range guard hands over, and rows whose exponents leave the fast
exponential's range.

Tolerances: those of the fp32 parity tests (an exponent here is below 100 in
magnitude, so its rounding is below 100 2^-24 = 6e-6; a gradient sums terms of both
signs).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1410_4984_amd as gpps  # noqa: E402
from paper_1410_4984_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TOL = {"psi0": 1e-6, "Psi1": 1e-5, "Psi2": 1e-4, "dmu": 1e-4, "dS": 1e-4, "dZ": 1e-4,
       "dsigma_f2": 1e-4, "dl": 1e-4}


def t(a):
    return torch.tensor(a, dtype=torch.float32, device=DEV)


def call(inp, path="generic"):
    N, Q = inp["mu"].shape
    M = inp["Z"].shape[0]
    ws = torch.full((gpps.workspace_bytes(torch.float32, N, M, Q),), 0x7F, dtype=torch.uint8, device=DEV)
    mu, S, Z = t(inp["mu"]), t(inp["S"]), t(inp["Z"])
    psi0, P1, P2 = gpps.psi_stats(mu, S, Z, inp["sigma_f2"], inp["l"], workspace=ws, path=path)
    ws.fill_(0x7F)
    g = gpps.psi_grads(mu, S, Z, inp["sigma_f2"], inp["l"], inp["dL_dpsi0"], t(inp["dL_dPsi1"]),
                       t(inp["dL_dPsi2"]), workspace=ws, path=path)
    torch.cuda.synchronize()
    return {k: v.double().cpu().numpy() for k, v in dict(psi0=psi0, Psi1=P1, Psi2=P2, **g).items()}


def check(got, inp, what):
    r0, R1, R2 = oracle.psi_stats(inp["mu"], inp["S"], inp["Z"], inp["sigma_f2"], inp["l"])
    ref = dict(psi0=r0, Psi1=R1, Psi2=R2,
               **oracle.psi_grads(inp["mu"], inp["S"], inp["Z"], inp["sigma_f2"], inp["l"],
                                  inp["dL_dpsi0"], inp["dL_dPsi1"], inp["dL_dPsi2"]))
    for k, v in ref.items():
        a, v = got[k].ravel(), np.asarray(v, np.float64).ravel()
        e = np.linalg.norm(a - v) / max(np.linalg.norm(v), 1e-300)
        assert e <= TOL[k], (what, k, e)
    assert np.array_equal(got["Psi2"], got["Psi2"].T)


@pytest.mark.parametrize("N,M,Q", [
    (1, 1, 5), (3, 130, 4), (2, 260, 3), (5, 17, 8), (17, 33, 9), (33, 32, 12), (19, 48, 13), (40, 49, 16),
    (31, 100, 17), (21, 129, 20), (9, 257, 21), (12, 300, 24), (7, 100, 25), (6, 512, 30), (64, 16, 6),
    (68, 16, 6), (1025, 16, 6), (11, 97, 32), (10, 70, 33), (5, 600, 40), (8, 50, 41), (9, 33, 48), (7, 40, 49),
    (5, 65, 64), (3, 1100, 20), (300, 10, 10), (70, 520, 5)])
def test_f32_tile_edges(N, M, Q):
    print(f"[f32 N={N} M={M} Q={Q}]", flush=True)
    inp = synth.to_f32(synth.random_inputs(N, M, Q, seed=N + M + Q))
    inp["dL_dPsi2"] = np.float32(inp["dL_dPsi2"] + np.triu(np.ones((M, M)), 1))  # not symmetric
    check(call(inp), inp, (N, M, Q))


@pytest.mark.parametrize("N,M,Q", [(400, 513, 6), (301, 300, 33), (260, 90, 63)])
def test_f32_tiles_past_the_matrix_core_limits(N, M, Q):
    inp = synth.to_f32(synth.random_inputs(N, M, Q, seed=N))
    got, forced = call(inp, path=None), call(inp)
    for k, v in forced.items():
        assert np.array_equal(got[k], v), k
    check(got, inp, (N, M, Q))
    with pytest.raises(gpps.GppsError) as e:
        call(inp, path="mfma")
    assert e.value.status == 8


def test_f32_tiles_behind_the_range_guard():
    # short lengthscales: the matrix-core path's fp16 operands do not hold them
    inp = synth.to_f32(synth.random_inputs(2000, 100, 10, seed=8, l_range=(0.02, 0.03), z_scale=2.0))
    N, M, Q = 2000, 100, 10
    ws = torch.empty(gpps.workspace_bytes(torch.float32, N, M, Q), dtype=torch.uint8, device=DEV)
    gpps.psi_stats(t(inp["mu"]), t(inp["S"]), t(inp["Z"]), inp["sigma_f2"], inp["l"], workspace=ws)
    assert gpps.route_taken(ws, torch.float32, N, M, Q) == 1
    got, ref = call(inp, path=None), call(inp)
    for k, v in ref.items():
        assert np.array_equal(got[k], v), k
    check(got, inp, "guard")


def test_f32_far_rows():
    # exponents of 1e8 and beyond contribute nothing; NaN stays within its row
    inp = synth.to_f32(synth.random_inputs(37, 40, 7, seed=4))
    inp["mu"][3] += 1e5
    inp["mu"][36, 2] = -1e8
    check(call(inp), inp, "far")
    inp["mu"][7, 3] = np.nan
    got = call(inp)
    assert np.isnan(got["Psi1"][7]).all() and np.isfinite(got["Psi1"][8]).all()
    assert np.isnan(got["Psi2"]).all() and np.isnan(got["dmu"][7]).all() and np.isfinite(got["dmu"][6]).all()
