"""Phi transforms of grid functions, the density and the one-function transforms
against the oracle at the edges of their tiles: n_phi odd, even, a multiple of
32 and off it, fewer than 16 point pairs; L on both sides of a 16-row tile and
of an 8-row step; one and several column tiles, ragged; workgroups that split
one row's sum (few rows) and waves that own one; a trig table in LDS and one
too large for it.

Tolerance: the FP64 sums have n_phi + n_theta + n_r + N < 600 terms and outputs
are compared relative to their maximum, so rounding stays below 600 u = 7e-14
times the transforms' conditioning (a few hundred for random inputs); 1e-11 as
for every other FP64 transform, 5e-5 where psi is formed in FP32.
"""
import numpy as np
import pytest

from oracle import basis as ob
from oracle import density as od
from oracle import hamiltonian as oh
from paper_1404_3773_amd import ces

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [
    # L, N, n_r, n_theta, n_phi, k
    (1, 3, 5, 2, 4, 1),
    (2, 3, 4, 3, 5, 17),
    (8, 6, 9, 16, 32, 16),
    (9, 5, 8, 18, 33, 33),
    (16, 5, 20, 32, 64, 5),
    (17, 4, 70, 35, 67, 3),
    (33, 3, 18, 40, 66, 19),
    (81, 2, 2, 82, 324, 2),
]


def rel(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_grid_transforms_and_density_match_oracle(shape):
    L, N, n_r, n_th, n_ph, k = shape
    print("case", shape, flush=True)
    bs = ob.make_basis(L, N, 9.0, n_r, n_th, n_ph)
    B = ces.Basis(L - 1, N, 9.0, n_r, n_th, n_ph)
    H = ces.Ham(B, torch.zeros(B.n_grid, dtype=torch.float64, device="cuda"))
    rng = np.random.default_rng(L * 1000 + n_ph)
    X = rng.standard_normal((B.d, k))
    f = rng.standard_normal((n_r, n_th, n_ph, k))
    occ = rng.random(k)
    work = H.workspace(k)
    # odd leading dimensions and bases: the grid columns are 8-byte aligned only
    Xd = torch.from_numpy(X.T.copy()).cuda()
    buf = torch.empty(k * B.n_grid + 1, dtype=torch.float64, device="cuda")
    fd = buf[1:].view(k, B.n_grid)
    H.to_grid(Xd, fd, work)
    ref = np.moveaxis(oh.to_grid_real(bs, X), 3, 0).reshape(k, -1)
    assert rel(fd.cpu().numpy(), ref) < 1e-11
    fd.copy_(torch.from_numpy(np.moveaxis(f, 3, 0).reshape(k, -1).copy()))
    Xb = torch.empty_like(Xd)
    H.from_grid(fd, Xb, work)
    assert rel(Xb.cpu().numpy().T, oh.from_grid_real(bs, f)) < 1e-11
    rho_ref = od.density_grid(bs, X, occ)
    tau_ref = od.density_coefficients(bs, rho_ref)
    rho = torch.empty(B.n_grid, dtype=torch.float64, device="cuda")
    tau = torch.empty(B.d, dtype=torch.float64, device="cuda")
    for prec, tol in ((ces.CES_PREC_FP64, 1e-11), (ces.CES_PREC_MIXED, 5e-5)):
        H.density(Xd, torch.from_numpy(occ).cuda(), rho, tau, prec, H.workspace(k, prec))
        assert rel(rho.cpu().numpy(), rho_ref.ravel()) < tol
        assert rel(tau.cpu().numpy(), tau_ref) < tol


# (the oracle's Hartree sum takes minutes at L = 81)
@pytest.mark.parametrize("shape", SHAPES[:-2], ids=lambda s: "x".join(map(str, s)))
def test_one_function_potential_matches_oracle(shape):
    """ks_potential's forward and inverse transforms run with the radial nodes
    as columns; its pieces must compose to the transforms of ces_hartree."""
    L, N, n_r, n_th, n_ph, _ = shape
    print("case", shape, flush=True)
    bs = ob.make_basis(L, N, 9.0, n_r, n_th, n_ph)
    B = ces.Basis(L - 1, N, 9.0, n_r, n_th, n_ph)
    H = ces.Ham(B, torch.zeros(B.n_grid, dtype=torch.float64, device="cuda"))
    rng = np.random.default_rng(L * 1000 + n_ph)
    rho, ion, vext = (rng.standard_normal((n_r, n_th, n_ph)) for _ in range(3))
    dev = [torch.from_numpy(a.ravel().copy()).cuda() for a in (rho, ion, vext)]
    work = H.workspace(1)
    v = torch.empty(B.n_grid, dtype=torch.float64, device="cuda")
    vh = torch.empty_like(v)
    tau = torch.empty(B.d, dtype=torch.float64, device="cuda")
    H.ks_potential(dev[0], dev[1], dev[2], v, work, tau=tau)
    H.hartree(tau, vh, work)
    tau_ref = od.density_coefficients(bs, rho - ion)
    assert rel(tau.cpu().numpy(), tau_ref) < 1e-11
    vh_ref = od.hartree_grid(bs, tau_ref)
    assert rel(vh.cpu().numpy(), vh_ref.ravel()) < 1e-11
    v_ref = vext + vh_ref - np.cbrt(3.0 / np.pi * np.maximum(rho, 0.0))
    assert rel(v.cpu().numpy(), v_ref.ravel()) < 1e-11
