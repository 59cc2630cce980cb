"""The largest N a launch of one workgroup per 64 rows takes: kernels that do a second job in
workgroups of their own must still take it."""
import pytest

torch = pytest.importorskip("torch")

import paper_1410_4984_amd as gpps  # noqa: E402

pytestmark = pytest.mark.gpu


# 2^24 - 1 row blocks of 256 threads fill a launch (2^32 threads) to the last workgroup, which
# leaves none for the symmetric part of dL/dPsi2 and the column sums beside them.  With
# M = Q = 1 and L = Psi2 = sum_n k(x_n, z)^2, dX_n = -2 k^2 (x_n - z) / l^2 to a few
# roundings of an exponent below 32 (1e-14), and dZ = -sum_n dX_n; that sum has at most
# 2^24 / 2048 64 = 5e5 terms in a row: 5e5 2^-53 = 6e-11 of their absolute values.
def test_known_gradients_at_the_row_block_limit():
    N, z, l = 2 ** 30 - 64, 0.25, 1.5
    if torch.cuda.mem_get_info()[0] < 96 << 30:
        pytest.skip("needs 96 GB of device memory")
    print(f"[launch limit N={N}]", flush=True)
    f64 = torch.float64
    X = torch.randn(N, 1, generator=torch.Generator(device="cuda:0").manual_seed(1), device="cuda:0", dtype=f64)
    Z = torch.full((1, 1), z, device="cuda:0", dtype=f64)
    g = gpps.psi_grads(X, None, Z, 1.0, [l], 0.0, None, torch.ones(1, 1, device="cuda:0", dtype=f64))
    torch.cuda.synchronize()
    total = scale = 0.0
    for i in range(0, N, 1 << 27):
        d = X[i:i + (1 << 27), 0] - z
        want = -2.0 * torch.exp(-(d / l) ** 2) * d / l ** 2
        err = float((g["dmu"][i:i + (1 << 27), 0] - want).abs().max())
        assert err <= 1e-14, (i, err)
        total, scale = total - float(want.sum()), scale + float(want.abs().sum())
    assert abs(float(g["dZ"]) - total) <= 6e-11 * scale
    del X, g, d, want
    torch.cuda.empty_cache()
