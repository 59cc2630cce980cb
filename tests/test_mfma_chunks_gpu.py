"""Row chunks of the matrix-core kernels where a grid is not filled by chunks of their usual
length: the tile gradient's one and two rounds (Q >= 31), the forwards with several tasks or
two ranges per chunk, the symmetric gradient at the widest Q of one block; ragged last
chunks.  Against the fp64 oracle, tolerances of the fp32 parity tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1410_4984_amd as gpps  # noqa: E402
from paper_1410_4984_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu

TOL = {"psi0": 1e-6, "Psi1": 1e-5, "Psi2": 1e-4, "dmu": 1e-4, "dS": 1e-4, "dZ": 1e-4,
       "dsigma_f2": 1e-4, "dl": 1e-4}


@pytest.mark.parametrize("N,M,Q", [(3000, 60, 62), (4999, 60, 40), (8001, 32, 33), (301, 96, 48), (1000, 130, 36),
                                   (2000, 130, 31), (333, 400, 25), (700, 300, 12), (13001, 20, 30), (41, 256, 62)])
def test_short_row_chunks(N, M, Q):
    print(f"[short chunks N={N} M={M} Q={Q}]", flush=True)
    inp = synth.to_f32(synth.random_inputs(N, M, Q, seed=N))
    d = {k: torch.tensor(v, dtype=torch.float32, device="cuda:0") for k, v in inp.items()
         if isinstance(v, np.ndarray)}
    ws = torch.full((gpps.workspace_bytes(torch.float32, N, M, Q),), 0x7F, dtype=torch.uint8, device="cuda:0")
    psi0, P1, P2 = gpps.psi_stats(d["mu"], d["S"], d["Z"], inp["sigma_f2"], inp["l"], workspace=ws, path="mfma")
    g = gpps.psi_grads(d["mu"], d["S"], d["Z"], inp["sigma_f2"], inp["l"], inp["dL_dpsi0"], d["dL_dPsi1"],
                       d["dL_dPsi2"], workspace=ws, path="mfma")
    assert gpps.route_taken(ws, torch.float32, N, M, Q) == 0
    r0, R1, R2 = oracle.psi_stats(inp["mu"], inp["S"], inp["Z"], inp["sigma_f2"], inp["l"])
    ref = dict(psi0=r0, Psi1=R1, Psi2=R2,
               **oracle.psi_grads(inp["mu"], inp["S"], inp["Z"], inp["sigma_f2"], inp["l"],
                                  inp["dL_dpsi0"], inp["dL_dPsi1"], inp["dL_dPsi2"]))
    for k, v in ref.items():
        a, v = dict(psi0=psi0, Psi1=P1, Psi2=P2, **g)[k].double().cpu().numpy().ravel(), np.ravel(v)
        assert np.linalg.norm(a - v) <= TOL[k] * np.linalg.norm(v), k
