"""The three-way bf16 split of the mixed-precision projector products at the ends
of FP32's range: blocks scaled by powers of two down to where the third part
falls under bf16's subnormals, and up; and an infinite entry.

With V_eff = 0 the product is Lambda / 2 X + P diag(h) P^T X; large h makes the
projector term the output's size.  Tolerance: 2e-5 of the maximum as for other
sums of d = 16,000 terms, plus what the split may drop of values below 2^-110: 2^-134
of each element of X (times |P|, |h|, |P| summed) and of C.
"""
import numpy as np
import pytest

from paper_1404_3773_amd import ces

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

L, N, NPROJ, K = 20, 40, 130, 140


def problem():
    B = ces.Basis(L - 1, N, 10.0, 4, 2, 2 * L)
    rng = np.random.default_rng(3)
    P = rng.standard_normal((NPROJ, B.d)) / np.sqrt(B.d)
    h = 300.0 * rng.standard_normal(NPROJ)
    X = rng.standard_normal((K, B.d))
    H = ces.Ham(B, torch.zeros(B.n_grid, dtype=torch.float64, device="cuda"),
                torch.from_numpy(P).cuda(), h)
    return B, P, h, X, H


def product(B, H, X):
    Y = torch.empty((K, B.d), dtype=torch.float64, device="cuda")
    H.apply_H(torch.from_numpy(X).cuda(), Y, ces.CES_PREC_MIXED,
              H.workspace(K, ces.CES_PREC_MIXED))
    return Y.cpu().numpy()


def test_scaled_blocks():
    B, P, h, X, H = problem()
    z = B.tables()[0]
    kin = np.concatenate([np.tile(0.5 * (z[l] / 10.0) ** 2, 2 * l + 1) for l in range(L)])
    ref = X * kin + (X @ P.T * h) @ P
    lost = 2.0 ** -134 * (np.abs(P.T) @ (np.abs(h) * np.abs(P).sum(axis=1) + 1.0)).max()
    for e in (0, -60, -104, -110, -114, -118, 60, 90):
        err = np.max(np.abs(product(B, H, X * 2.0 ** e) * 2.0 ** -e - ref))
        print("scale 2^%d err %.2e of the maximum" % (e, err / np.max(np.abs(ref))), flush=True)
        assert err < 2e-5 * np.max(np.abs(ref)) + lost * 2.0 ** -e


def test_an_infinite_entry_stays_in_its_column():
    B, P, h, X, H = problem()
    Y = product(B, H, X)
    X[3, 7] = np.inf
    Z = product(B, H, X)
    assert np.isnan(Z[3]).all()
    keep = np.arange(K) != 3
    assert np.array_equal(Z[keep], Y[keep])
