"""Scratch of the projector products: blocks with projectors just below the
fixed 256 MiB of ces_apply_H_noalloc are taken (at these sizes more than 24 MiB
of split-K partial sums in a region of their own would not fit), and a
workspace holds at most 32 chunks of partial sums per projector and column.

The product runs the kernels of ces_apply_H, so the two agree bit for bit; with
V_eff = 0 the result is Lambda / 2 X + P diag(h) P^T X, tolerances relative to
the output's maximum as for the other products: FP64 1e-11, FP32 2e-5 (sums of
at most d = 57,660 terms, u sqrt(d) = 1.4e-5).
"""
import numpy as np
import pytest

from paper_1404_3773_amd import ces

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FP64, MIXED = ces.CES_PREC_FP64, ces.CES_PREC_MIXED


def handle(L, N, grid, n_proj):
    B = ces.Basis(L - 1, N, 14.0, *grid)
    g = torch.Generator(device="cuda").manual_seed(n_proj)
    P = torch.randn((n_proj, B.d), dtype=torch.float64, device="cuda", generator=g) / B.d ** 0.5
    V = torch.zeros(B.n_grid, dtype=torch.float64, device="cuda")
    return B, P, ces.Ham(B, V, P, np.linspace(-1.0, 1.0, n_proj)), g


@pytest.mark.parametrize("L,N,grid,n_proj,k,prec", [
    (31, 60, (90, 62, 124), 52, 96, MIXED),
    (25, 40, (60, 50, 100), 100, 128, FP64),
    (25, 40, (60, 50, 100), 100, 208, MIXED)])
def test_noalloc_near_its_limit_with_projectors(L, N, grid, n_proj, k, prec):
    print("case", L, N, n_proj, k, prec, flush=True)
    B, P, H, g = handle(L, N, grid, n_proj)
    X = torch.randn((k, B.d), dtype=torch.float64, device="cuda", generator=g)
    Y, Z = torch.empty_like(X), torch.full_like(X, float("nan"))
    H.apply_H(X, Y, prec, H.workspace(k, prec))
    H.apply_H_noalloc(X, Z, prec)
    assert torch.equal(Y, Z)
    z = B.tables()[0]
    kin = torch.as_tensor(np.concatenate([np.tile(0.5 * (z[l] / 14.0) ** 2, 2 * l + 1)
                                          for l in range(L)])).cuda()
    h = torch.as_tensor(np.linspace(-1.0, 1.0, n_proj)).cuda()
    ref = X * kin + (X @ P.T.contiguous() * h) @ P
    err = float((Z - ref).abs().max() / ref.abs().max())
    print("  err %.2e" % err, flush=True)
    assert err < (1e-11 if prec == FP64 else 2e-5)


@pytest.mark.parametrize("L,N,grid,n_proj,k", [
    (31, 60, (90, 62, 124), 52, 32), (25, 40, (60, 50, 100), 100, 128),
    (41, 73, (20, 12, 82), 300, 400)])
def test_workspace_of_the_projector_products(L, N, grid, n_proj, k):
    B, P, H, _ = handle(L, N, grid, n_proj)
    H0 = ces.Ham(B, torch.zeros(B.n_grid, dtype=torch.float64, device="cuda"))
    kp = (k + 15) // 16 * 16
    for prec in (FP64, MIXED):
        extra = H.workspace_size(k, prec) - H0.workspace_size(k, prec)
        print("case", L, n_proj, k, prec, "bytes", extra, flush=True)
        # C and Z = P C, the partial sums, and the regions' alignment
        assert extra <= 8 * n_proj * kp + 8 * B.d * kp + 32 * 8 * n_proj * kp + 4096
