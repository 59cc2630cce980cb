"""Calls on both sides of the smallest ones, which take the generic kernels without a path
flag: N (M^2 + 1000) (Q + 6) <= 1.5e7 (at M = 10, Q = 2 up to N = 1,704).  The route word
tells them (2) from calls that the range guard handed over (1), and both sides agree
with the fp64 oracle to the fp32 parity tolerances."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1410_4984_amd as gpps  # noqa: E402
from paper_1410_4984_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu

TOL = {"psi0": 1e-6, "Psi1": 1e-5, "Psi2": 1e-4, "dmu": 1e-4, "dS": 1e-4, "dZ": 1e-4,
       "dsigma_f2": 1e-4, "dl": 1e-4}


# far: half the data 300 lengthscales away, which the guard rejects
@pytest.mark.parametrize("N,path,far,route", [
    (1704, None, False, 2), (1704, None, True, 2), (1, None, False, 2), (1704, "mfma", False, 0),
    (1704, "mfma", True, 1), (1704, "generic", False, -1), (1705, None, False, 0), (1705, None, True, 1)])
def test_route_and_results_around_the_smallest_calls(N, path, far, route):
    print(f"[small calls N={N} {path} far={far}: route {route}]", flush=True)
    M, Q = 10, 2
    inp = synth.random_inputs(N, M, Q, seed=N, l_range=(0.8, 1.2))
    if far:
        inp["mu"][: N // 2] += 300.0
    inp = synth.to_f32(inp)
    d = {k: torch.tensor(v, dtype=torch.float32, device="cuda:0") for k, v in inp.items()
         if isinstance(v, np.ndarray)}
    ws = torch.full((gpps.workspace_bytes(torch.float32, N, M, Q),), 0xFF, dtype=torch.uint8, device="cuda:0")
    psi0, P1, P2 = gpps.psi_stats(d["mu"], d["S"], d["Z"], inp["sigma_f2"], inp["l"], workspace=ws, path=path)
    assert gpps.route_taken(ws, torch.float32, N, M, Q) == route
    ws.fill_(0xFF)
    g = gpps.psi_grads(d["mu"], d["S"], d["Z"], inp["sigma_f2"], inp["l"], inp["dL_dpsi0"], d["dL_dPsi1"],
                       d["dL_dPsi2"], workspace=ws, path=path)
    assert gpps.route_taken(ws, torch.float32, N, M, Q) == route
    got = dict(psi0=psi0, Psi1=P1, Psi2=P2, **g)
    r0, R1, R2 = oracle.psi_stats(inp["mu"], inp["S"], inp["Z"], inp["sigma_f2"], inp["l"])
    ref = dict(psi0=r0, Psi1=R1, Psi2=R2,
               **oracle.psi_grads(inp["mu"], inp["S"], inp["Z"], inp["sigma_f2"], inp["l"],
                                  inp["dL_dpsi0"], inp["dL_dPsi1"], inp["dL_dPsi2"]))
    for k, v in ref.items():
        a, v = got[k].double().cpu().numpy().ravel(), np.asarray(v, np.float64).ravel()
        assert np.linalg.norm(a - v) <= TOL[k] * max(np.linalg.norm(v), 1e-300), k
