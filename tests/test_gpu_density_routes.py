"""The density's two kernels at the edges of their rule, against the oracle: the
largest L of a wave per row and the first past it in each precision (FP64 L =
56, 57; FP32 L = 88, 89), several column tiles on fewer than 1024 rows and on
more, one column tile on few rows, ragged columns, an odd n_phi and the largest
(99 KB of LDS).

Tolerance relative to the maximum: 1e-11 in FP64 (sums of at most 2048 + 600
terms, conditioning of a few hundred), 5e-5 where psi is formed in FP32.
"""
import numpy as np
import pytest

from oracle import basis as ob
from oracle import density as od
from paper_1404_3773_amd import ces

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,N,n_r,n_th,n_ph,k", [
    (56, 2, 9, 114, 224, 19), (57, 2, 9, 114, 229, 33), (57, 2, 3, 114, 228, 16),
    (88, 2, 2, 90, 176, 5), (89, 2, 2, 90, 178, 37), (96, 2, 1, 20, 192, 3),
    (9, 4, 56, 18, 41, 34), (9, 4, 57, 18, 72, 34), (9, 4, 5, 18, 2048, 20), (3, 3, 4, 6, 7, 50)])
def test_density_matches_oracle(L, N, n_r, n_th, n_ph, k):
    print("case", L, N, n_r, n_th, n_ph, k, flush=True)
    bs = ob.make_basis(L, N, 9.0, n_r, n_th, n_ph)
    B = ces.Basis(L - 1, N, 9.0, n_r, n_th, n_ph)
    H = ces.Ham(B, torch.zeros(B.n_grid, dtype=torch.float64, device="cuda"))
    rng = np.random.default_rng(L + n_ph)
    X = rng.standard_normal((B.d, k))
    occ = rng.random(k)
    ref = od.density_grid(bs, X, occ).ravel()
    Xd = torch.from_numpy(X.T.copy()).cuda()
    for prec, tol in ((ces.CES_PREC_FP64, 1e-11), (ces.CES_PREC_MIXED, 5e-5)):
        rho = torch.full((B.n_grid,), float("nan"), dtype=torch.float64, device="cuda")
        H.density(Xd, torch.from_numpy(occ).cuda(), rho, None, prec, H.workspace(k, prec))
        err = float(np.max(np.abs(rho.cpu().numpy() - ref)) / np.max(np.abs(ref)))
        print("  prec", prec, "err %.2e" % err, flush=True)
        assert err < tol
