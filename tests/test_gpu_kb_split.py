"""Mixed-precision projector products at the edges of their tiles: column and
projector counts on both sides of the 96 / 128 rule and of a 256 tile, a
partial last 32-step of either contraction, odd d (rows padded to 32), several
split-K chunks, one of them short.

With V_eff = 0 the product is Lambda / 2 X + P diag(h) P^T X exactly.  Tolerance
relative to the output's maximum: inputs rounded to FP32 (two roundings), a
product error of one FP32 rounding, sums of at most d = 12,000 terms in FP32
whose rounding errors add like a random walk (sqrt(12000) u = 7e-6): 2e-5.
"""
import numpy as np
import pytest

from paper_1404_3773_amd import ces

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,N,n_proj,k", [
    (9, 11, 96, 129), (9, 11, 95, 129), (9, 11, 96, 128), (9, 11, 257, 257), (10, 12, 300, 130),
    (20, 30, 129, 256), (20, 30, 13, 4), (20, 30, 700, 513)])
def test_projector_products_match_float64(L, N, n_proj, k):
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
        Y = torch.empty((k, B.d), dtype=torch.float64, device="cuda")
        H.apply_H(torch.from_numpy(X).cuda(), Y, prec, H.workspace(k, prec))
        err = np.max(np.abs(Y.cpu().numpy() - ref)) / np.max(np.abs(ref))
        print("  prec", prec, "err %.2e" % err, flush=True)
        assert err < tol
