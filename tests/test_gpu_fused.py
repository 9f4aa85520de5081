"""The fused angular stage (L <= 16) and the first sizes past it against the
oracle: L on both sides of an 8-row step and of 16, theta rows in one group and
several, ragged groups, odd n_theta, phi grids finer and coarser than the
stage's own 4 L points (V_eff is resampled), one part of A and two, n_r past the
two-part limit, ragged column tiles.

Tolerance: the H X tolerances of the other tests (FP64 1e-11 relative to the
maximum for sums of N + n_r + n_theta + 8 L < 400 terms; 5e-5 in FP32).
"""
import numpy as np
import pytest

from oracle import basis as ob
from oracle import hamiltonian as oh
from paper_1404_3773_amd import ces

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,N,n_r,n_th,n_ph,k", [
    (1, 3, 5, 1, 1, 1), (2, 4, 6, 4, 3, 17), (3, 4, 6, 5, 40, 16), (8, 6, 12, 16, 32, 5),
    (9, 6, 12, 18, 17, 33), (9, 6, 20, 19, 37, 48), (15, 4, 9, 31, 60, 16), (16, 4, 9, 33, 64, 3),
    (16, 5, 100, 40, 31, 20), (17, 4, 9, 34, 68, 18)])
def test_apply_H_matches_oracle(L, N, n_r, n_th, n_ph, k):
    print("case", L, N, n_r, n_th, n_ph, k, flush=True)
    bs = ob.make_basis(L, N, 9.0, n_r, n_th, n_ph)
    B = ces.Basis(L - 1, N, 9.0, n_r, n_th, n_ph)
    rng = np.random.default_rng(L * 100 + n_ph)
    V = rng.standard_normal((n_r, n_th, n_ph))
    X = rng.standard_normal((B.d, k))
    H = ces.Ham(B, torch.from_numpy(V.ravel()).cuda())
    H.set_veff(torch.from_numpy(2.0 * V.ravel()).cuda())
    H.set_veff(torch.from_numpy(V.ravel()).cuda())
    ref = oh.apply_H_real(bs, V, X)
    Xd = torch.from_numpy(X.T.copy()).cuda()
    for prec, tol in ((ces.CES_PREC_FP64, 1e-11), (ces.CES_PREC_MIXED, 5e-5)):
        Y = torch.full_like(Xd, float("nan"))
        H.apply_H(Xd, Y, prec, H.workspace(k, prec))
        err = np.max(np.abs(Y.cpu().numpy().T - ref)) / np.max(np.abs(ref))
        print("  prec", prec, "err %.2e" % err, flush=True)
        assert err < tol
