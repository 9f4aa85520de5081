"""The rule of the mixed-precision projector products (split kernels from 96
projectors, 129 columns, and d = 15,000 or d k n_proj = 1.5e9) on both sides of
each edge, and the tiles of the split kernels at sizes past it: d off a multiple
of 32, a partial last 256 tile of projectors, columns and rows, several column
tiles.

With V_eff = 0 the product is Lambda / 2 X + P diag(h) P^T X exactly.  Tolerance
relative to the output's maximum: two roundings of the inputs to FP32, one of
the product, sums of at most d = 16,000 terms whose rounding errors add like a
random walk (sqrt(16000) u = 7.5e-6): 2e-5 in FP32, 1e-11 in FP64.
"""
import numpy as np
import pytest

from paper_1404_3773_amd import ces

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,N,n_proj,k", [
    (21, 35, 96, 129), (21, 35, 95, 129), (21, 35, 96, 128), (21, 35, 257, 257), (20, 40, 130, 300),
    (22, 30, 96, 129), (17, 30, 432, 400), (17, 30, 433, 400), (9, 12, 300, 300)])
def test_products_match_float64(L, N, n_proj, k):
    print("case", L, N, n_proj, k, flush=True)
    B = ces.Basis(L - 1, N, 10.0, 4, 2, 2 * L)
    rng = np.random.default_rng(n_proj + k)
    P = rng.standard_normal((n_proj, B.d)) / np.sqrt(B.d)
    h = rng.standard_normal(n_proj)
    X = rng.standard_normal((k, B.d))
    H = ces.Ham(B, torch.zeros(B.n_grid, dtype=torch.float64, device="cuda"),
                torch.from_numpy(P).cuda(), h)
    z = B.tables()[0]
    kin = np.concatenate([np.tile(0.5 * (z[l] / 10.0) ** 2, 2 * l + 1) for l in range(L)])
    ref = X * kin + (X @ P.T * h) @ P
    for prec, tol in ((ces.CES_PREC_MIXED, 2e-5), (ces.CES_PREC_FP64, 1e-11)):
        Y = torch.full((k, B.d), float("nan"), dtype=torch.float64, device="cuda")
        H.apply_H(torch.from_numpy(X).cuda(), Y, prec, H.workspace(k, prec))
        err = np.max(np.abs(Y.cpu().numpy() - ref)) / np.max(np.abs(ref))
        print("  prec", prec, "err %.2e" % err, flush=True)
        assert err < tol
