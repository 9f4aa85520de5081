"""FP64 projector products on the 128 x 128 tiles of long contractions: full
and ragged tiles in both directions, columns on both sides of the rule (an
even number of 64-column tiles), odd d (the general kernel).

With V_eff = 0 the product is Lambda / 2 X + P diag(h) P^T X exactly; sums of
about 100,000 FP64 terms: 1e-11 relative to the output's maximum.
"""
import numpy as np
import pytest

from paper_1404_3773_amd import ces

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,n_proj,k", [
    (80, 96, 65), (80, 129, 128), (80, 130, 129), (80, 97, 200), (78, 256, 256), (79, 97, 100)])
def test_wide_fp64_projector_product(N, n_proj, k):
    print("case", N, n_proj, k, flush=True)
    B = ces.Basis(36, N, 10.0, 4, 2, 74)
    g = torch.Generator().manual_seed(n_proj + k)
    P = torch.randn((n_proj, B.d), dtype=torch.float64, generator=g).cuda() / np.sqrt(B.d)
    h = torch.randn(n_proj, dtype=torch.float64, generator=g)
    X = torch.randn((k, B.d), dtype=torch.float64, generator=g).cuda()
    H = ces.Ham(B, torch.zeros(B.n_grid, dtype=torch.float64, device="cuda"), P, h.numpy())
    z = B.tables()[0]
    kin = np.concatenate([np.tile(0.5 * (z[l] / 10.0) ** 2, 2 * l + 1) for l in range(37)])
    ref = X * torch.from_numpy(kin).cuda() + (X @ P.T * h.cuda()) @ P
    Y = torch.empty_like(X)
    H.apply_H(X, Y, ces.CES_PREC_FP64, H.workspace(k))
    err = float((Y - ref).abs().max() / ref.abs().max())
    print("  err %.2e" % err, flush=True)
    assert err < 1e-11
