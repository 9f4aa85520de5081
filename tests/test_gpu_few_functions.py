"""One and two grid functions to coefficients and back: one function on grids
of few and many rows, two on both sides of the 3000 rows from which they go one
by one, n_r on and off a multiple of 16, an odd n_phi, an L past the folded
Legendre stages, a kinetic-energy cutoff that leaves l without functions, row
pitches above d, and a mixed-precision workspace.

Tolerance relative to the maximum: the FP64 1e-11 of the other transforms.
"""
import numpy as np
import pytest

from oracle import basis as ob
from oracle import hamiltonian as oh
from paper_1404_3773_amd import ces

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,N,n_r,n_th,n_ph,k", [
    (1, 2, 3, 1, 1, 1), (6, 5, 17, 12, 25, 1), (25, 5, 16, 50, 100, 1), (33, 3, 70, 67, 67, 1),
    (5, 4, 100, 30, 20, 2), (5, 4, 13, 230, 20, 2), (25, 3, 60, 50, 99, 2), (9, 40, 200, 18, 36, 2)])
@pytest.mark.parametrize("prec", [ces.CES_PREC_FP64, ces.CES_PREC_MIXED])
def test_transforms_match_oracle(L, N, n_r, n_th, n_ph, k, prec):
    print("case", L, N, n_r, n_th, n_ph, k, prec, flush=True)
    bs = ob.make_basis(L, N, 9.0, n_r, n_th, n_ph)
    B = ces.Basis(L - 1, N, 9.0, n_r, n_th, n_ph)
    H = ces.Ham(B, torch.zeros(B.n_grid, dtype=torch.float64, device="cuda"))
    rng = np.random.default_rng(L * 1000 + n_ph)
    X = rng.standard_normal((B.d, k))
    f = rng.standard_normal((n_r, n_th, n_ph, k))
    work = H.workspace(k, prec)
    buf = torch.full((k, B.d + 3), 7.0, dtype=torch.float64, device="cuda")
    Xd = buf[:, :B.d]
    Xd.copy_(torch.from_numpy(X.T.copy()))
    fd = torch.full((k, B.n_grid), float("nan"), dtype=torch.float64, device="cuda")
    H.to_grid(Xd, fd, work)
    ref = np.moveaxis(oh.to_grid_real(bs, X), 3, 0).reshape(k, -1)
    assert np.max(np.abs(fd.cpu().numpy() - ref)) < 1e-11 * np.max(np.abs(ref))
    fd.copy_(torch.from_numpy(np.moveaxis(f, 3, 0).reshape(k, -1).copy()))
    H.from_grid(fd, Xd, work)
    ref = oh.from_grid_real(bs, f).T
    assert np.max(np.abs(Xd.cpu().numpy() - ref)) < 1e-11 * np.max(np.abs(ref))
    assert bool((buf[:, B.d:] == 7.0).all())


def test_a_cutoff_basis_keeps_its_layout():
    """Kinetic-energy cutoff: the one-function transforms agree with the block
    transforms of three functions (rounding apart)."""
    B = ces.Basis(11, 8, 9.0, 20, 24, 48, e_cut=1.0)
    assert min(B.Nl) == 0 and max(B.Nl) < 8
    H = ces.Ham(B, torch.zeros(B.n_grid, dtype=torch.float64, device="cuda"))
    g = torch.Generator().manual_seed(5)
    X = torch.randn((3, B.d), dtype=torch.float64, generator=g).cuda()
    f3, X3 = torch.empty((3, B.n_grid), dtype=torch.float64, device="cuda"), torch.empty_like(X)
    H.to_grid(X, f3, H.workspace(3))
    H.from_grid(f3, X3, H.workspace(3))
    f1, X1 = torch.empty_like(f3[:1]), torch.empty_like(X[:1])
    H.to_grid(X[1:2], f1, H.workspace(1))
    H.from_grid(f3[1:2], X1, H.workspace(1))
    assert float((f1 - f3[1:2]).abs().max()) < 1e-11 * float(f3.abs().max())
    assert float((X1 - X3[1:2]).abs().max()) < 1e-11 * float(X3.abs().max())
