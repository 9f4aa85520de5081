"""The streamed radial forward contraction (n_r > 96) on its workgroups of 64
and of 32 columns: column counts on both sides of each rule (one 32-column
group, padding of 64-column groups, number of workgroups), N on both sides of
its 4-wave tiles, n_r not a multiple of the k-step.

Reference: the FP64 product of the same columns taken 16 at a time (32-column
workgroups).  Tolerance relative to the output's maximum: FP64 1e-13 (the same
sums in another order), mixed 1e-6 (FP32 rounding of an H X whose parts are of
the output's size).
"""
import pytest

from paper_1404_3773_amd import ces

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,N,n_r,n_proj,k", [
    (18, 20, 97, 3, 33), (18, 64, 99, 0, 64), (18, 65, 101, 5, 97), (40, 66, 98, 4, 128),
    (40, 30, 100, 0, 113), (40, 130, 131, 2, 66)])
def test_wide_blocks_match_narrow_ones(L, N, n_r, n_proj, k):
    print("case", L, N, n_r, n_proj, k, flush=True)
    B = ces.Basis(L - 1, N, 10.0, n_r, 2 * L, 4 * L)
    g = torch.Generator().manual_seed(L * N + k)
    V = torch.rand(B.n_grid, dtype=torch.float64, generator=g).cuda()
    P = (torch.randn((n_proj, B.d), dtype=torch.float64, generator=g).cuda() / B.d ** 0.5
         if n_proj else None)
    H = ces.Ham(B, V, P, [0.5] * n_proj if n_proj else None)
    X = torch.randn((k, B.d), dtype=torch.float64, generator=g).cuda()
    for prec, tol in ((ces.CES_PREC_FP64, 1e-13), (ces.CES_PREC_MIXED, 1e-6)):
        Y, Z = torch.empty_like(X), torch.empty_like(X)
        H.apply_H(X, Y, prec, H.workspace(k, prec))
        for c in range(0, k, 16):
            n = min(16, k - c)
            H.apply_H(X[c:c + n], Z[c:c + n], ces.CES_PREC_FP64, H.workspace(n))
        err = float((Y - Z).abs().max() / Z.abs().max())
        print("  prec", prec, "err %.2e" % err, flush=True)
        assert err < tol
