"""The last product of a filter writes the caller's block itself: degrees with
no, one and two recurrence buffers behind the result, the one-chunk and the
streamed radial form, a row pitch above d, and FP64 in a mixed-precision
workspace (column chunks).

Reference: the three-term recurrence in float64 with FP64 products.  Tolerance
relative to the output's maximum: FP64 1e-11; mixed 2e-5 for each of the at
most three FP32 products.
"""
import pytest

from paper_1404_3773_amd import ces

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def recurrence(H, X, degree, a, b, a0):
    w = H.workspace(X.shape[0])

    def hx(V):
        Y = torch.empty_like(V)
        H.apply_H(V, Y, ces.CES_PREC_FP64, w)
        return Y

    e, c = (b - a) / 2, (b + a) / 2
    s1 = s = e / (a0 - c)
    prev, cur = X, (hx(X) - c * X) * (s1 / e)
    for _ in range(2, degree + 1):
        sn = 1 / (2 / s1 - s)
        prev, cur = cur, (hx(cur) - c * cur) * (2 * sn / e) - prev * (s * sn)
        s = sn
    return cur


@pytest.mark.parametrize("degree", [1, 2, 3])
@pytest.mark.parametrize("L,N,n_r,n_proj,k", [(9, 11, 16, 5, 7), (18, 30, 100, 0, 33),
                                              (18, 70, 106, 9, 20)])
def test_last_step_writes_the_block(L, N, n_r, n_proj, k, degree):
    print("case", L, N, n_r, n_proj, k, degree, flush=True)
    B = ces.Basis(L - 1, N, 10.0, n_r, 2 * L, 4 * L)
    g = torch.Generator().manual_seed(L + N + degree)
    V = torch.rand(B.n_grid, dtype=torch.float64, generator=g).cuda()
    P = (torch.randn((n_proj, B.d), dtype=torch.float64, generator=g).cuda() / B.d ** 0.5
         if n_proj else None)
    H = ces.Ham(B, V, P, [0.5] * n_proj if n_proj else None)
    X = torch.randn((k, B.d), dtype=torch.float64, generator=g).cuda()
    ref = recurrence(H, X, degree, 1.0, 9.0, 0.2)
    scale = ref.abs().max()
    for prec, wprec, tol in ((ces.CES_PREC_FP64, ces.CES_PREC_FP64, 1e-11),
                             (ces.CES_PREC_FP64, ces.CES_PREC_MIXED, 1e-11),
                             (ces.CES_PREC_MIXED, ces.CES_PREC_MIXED, 6e-5)):
        buf = torch.full((k, B.d + 3), 7.0, dtype=torch.float64, device="cuda")
        Y = buf[:, :B.d]
        Y.copy_(X)
        H.cheb_filter(Y, degree, 1.0, 9.0, 0.2, prec, H.workspace(k, wprec))
        err = float((Y - ref).abs().max() / scale)
        print("  prec", prec, "workspace", wprec, "err %.2e" % err, flush=True)
        assert err < tol
        assert bool((buf[:, B.d:] == 7.0).all())
