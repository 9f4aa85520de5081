"""The streamed radial forward contraction (n_r > 96) as a step of the filter's
recurrence (result over the oldest block, all three operands in the epilogue),
on both sides of the workgroup counts its forms are chosen by: FP32 on 64-column
workgroups from 2048 (L = 46, one group; L = 40, two) and just below, FP64 from
800 and below, FP64 of up to 32 columns from 1024 and below; ragged columns and
n_r off a multiple of the k-step, with and without projectors.

Reference: the recurrence in float64 with the oracle's H X on some columns.
Tolerance relative to the output's maximum: FP64 1e-11; mixed 2e-5 for each of
the three FP32 products.
"""
import numpy as np
import pytest

from oracle import basis as ob
from oracle import hamiltonian as oh
from paper_1404_3773_amd import ces

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,N,n_r,n_proj,k", [
    (46, 3, 98, 2, 61), (45, 3, 98, 0, 61), (40, 66, 98, 3, 128), (29, 4, 101, 2, 64),
    (28, 4, 101, 0, 64), (33, 5, 97, 2, 30), (31, 5, 97, 0, 30), (5, 40, 225, 2, 49)])
def test_filter_matches_oracle(L, N, n_r, n_proj, k):
    print("case", L, N, n_r, n_proj, k, flush=True)
    n_th, n_ph = min(2 * L, 24), 2 * L - 1
    bs = ob.make_basis(L, N, 9.0, n_r, n_th, n_ph)
    B = ces.Basis(L - 1, N, 9.0, n_r, n_th, n_ph)
    rng = np.random.default_rng(L + k)
    V = rng.standard_normal((n_r, n_th, n_ph))
    X = rng.standard_normal((B.d, k))
    P = rng.standard_normal((n_proj, B.d)) / np.sqrt(B.d)
    h = rng.standard_normal(n_proj)
    H = ces.Ham(B, torch.from_numpy(V.ravel()).cuda(),
                torch.from_numpy(P).cuda() if n_proj else None, h if n_proj else None)
    some = [0, 1, k // 2, k - 1]
    top = 0.6 * float(B.tables()[0].max() / 9.0) ** 2
    a, b, a0 = 0.5, top, -1.0

    def hx(v):
        return oh.apply_H_real(bs, V, v) + P.T @ (h[:, None] * (P @ v))

    e, c = (b - a) / 2, (b + a) / 2
    s1 = s = e / (a0 - c)
    prev, cur = X[:, some], (hx(X[:, some]) - c * X[:, some]) * (s1 / e)
    for _ in range(2):
        sn = 1 / (2 / s1 - s)
        prev, cur = cur, (hx(cur) - c * cur) * (2 * sn / e) - prev * (s * sn)
        s = sn
    for prec, tol in ((ces.CES_PREC_FP64, 1e-11), (ces.CES_PREC_MIXED, 6e-5)):
        Y = torch.from_numpy(X.T.copy()).cuda()
        H.cheb_filter(Y, 3, a, b, a0, prec, H.workspace(k, prec))
        Yn = Y.cpu().numpy().T
        assert np.isfinite(Yn).all()
        err = np.max(np.abs(Yn[:, some] - cur)) / np.max(np.abs(cur))
        print("  prec", prec, "err %.2e" % err, flush=True)
        assert err < tol
