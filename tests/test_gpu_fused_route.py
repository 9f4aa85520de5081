"""H X with L <= 16 on both sides of the rule between the fused angular kernel
and the three kernels, against the oracle: the work limits of 2048 (FP64) and
3072 (FP32) on grids with theta nodes as L needs them, grids with many more, the
L that are fused at any width and those that are not, in both precisions, after
the potential has been replaced.  The two forms of V_eff are of one potential: a
narrow and a wide block of the same columns agree.

Tolerance: the H X tolerances of the other tests relative to the maximum (FP64
1e-11 for sums of N + n_r + n_theta + 8 L < 400 terms; 5e-5 in FP32).
"""
import numpy as np
import pytest

from oracle import basis as ob
from oracle import hamiltonian as oh
from paper_1404_3773_amd import ces

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,N,n_r,n_th,n_ph,k", [
    (9, 3, 24, 18, 36, 336), (9, 3, 24, 18, 36, 337), (9, 3, 24, 18, 35, 512), (9, 3, 24, 18, 36, 513), (1, 3, 1, 1, 1, 2000), (1, 2, 16, 9, 40, 1700), (1, 2, 36, 2, 4, 256),
    (1, 2, 36, 2, 4, 257), (3, 2, 100, 6, 12, 180),
    (5, 3, 60, 10, 20, 1000), (6, 2, 60, 12, 24, 1000), (7, 2, 12, 30, 29, 1100),
    (10, 2, 30, 40, 40, 128), (10, 2, 30, 40, 40, 160), (11, 2, 40, 23, 44, 400),
    (12, 2, 40, 25, 50, 350), (16, 2, 30, 64, 33, 144), (16, 2, 40, 32, 64, 300)])
def test_apply_H_matches_oracle(L, N, n_r, n_th, n_ph, k):
    print("case", L, N, n_r, n_th, n_ph, k, flush=True)
    bs = ob.make_basis(L, N, 9.0, n_r, n_th, n_ph)
    B = ces.Basis(L - 1, N, 9.0, n_r, n_th, n_ph)
    rng = np.random.default_rng(L * 100 + n_ph)
    V = rng.standard_normal((n_r, n_th, n_ph))
    X = rng.standard_normal((B.d, k))
    H = ces.Ham(B, torch.zeros(B.n_grid, dtype=torch.float64, device="cuda"))
    H.set_veff(torch.from_numpy(V.ravel()).cuda())
    some = np.r_[0:3, k // 2, k - 17:k]      # the oracle's columns
    ref = oh.apply_H_real(bs, V, X[:, some])
    Xd = torch.from_numpy(X.T.copy()).cuda()
    for prec, tol in ((ces.CES_PREC_FP64, 1e-11), (ces.CES_PREC_MIXED, 5e-5)):
        Y = torch.full_like(Xd, float("nan"))
        H.apply_H(Xd, Y, prec, H.workspace(k, prec))
        Yn = Y.cpu().numpy().T
        assert np.isfinite(Yn).all()
        err = np.max(np.abs(Yn[:, some] - ref)) / np.max(np.abs(ref))
        Z = torch.empty_like(Xd[:20])
        H.apply_H(Xd[:20], Z, prec, H.workspace(20, prec))
        dif = float((Z - Y[:20]).abs().max() / Y.abs().max())
        print("  prec", prec, "err %.2e, narrow against wide %.2e" % (err, dif), flush=True)
        assert err < tol and dif < tol
