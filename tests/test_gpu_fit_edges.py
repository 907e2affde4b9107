"""The fit at the edges of its blocks (64-row diagonal blocks, two of them a solve step, panels
of 16 in the factorisation, 64 or 128 columns a solve workgroup, 65,536-column chunks): row
counts around 16, 64 and 128, single and ragged columns, two chunks, FP32 xi, against the oracle."""
import numpy as np
import pytest

from gpu_common import note, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_mu,n_g,n_orb", [(1, 1, 3), (1, 70, 3), (15, 31, 12), (63, 63, 40),
                                            (64, 129, 40), (65, 200, 40), (127, 300, 40),
                                            (128, 1000, 40), (129, 16500, 40), (193, 333, 60),
                                            (7, 70000, 12)])
def test_fit_edges(n_mu, n_g, n_orb):
    import torch
    from oracle import fit as of
    from paper_2607_17314_amd import _lib as L
    from paper_2607_17314_amd import api
    rng = np.random.default_rng(1000 * n_mu + n_g)
    phi4 = rng.normal(size=(4, n_orb, n_g))
    xyz, w = rng.normal(size=(3, n_g)), 0.5 + rng.random(n_g)
    piv = rng.choice(n_g, n_mu, replace=False)
    ref = of.fit(phi4, w, piv)
    grid, p = api.DeviceGrid.from_host(xyz, w), torch.as_tensor(phi4).cuda()
    note(f"fit n_mu={n_mu} n_g={n_g} n_orb={n_orb}")
    xi, xig, _, chol, _ = api.fit_ex(p, grid, piv, keep_chol=True)
    # Gram matrices of condition below 100 (n_orb^2 on the diagonal against terms of about
    # n_orb beside it), sums of at most 193 products
    assert rel_err(xi.cpu().numpy(), ref.xi) < 1e-11
    assert rel_err(xig.cpu().numpy(), ref.xigrad) < 1e-11
    xi32, xig2, _, chol2, _ = api.fit_ex(p, grid, piv, xi_prec=L.XTC_FP32, keep_chol=True)
    assert torch.equal(xi32, xi.float()) and torch.equal(xig2, xig) and torch.equal(chol2, chol)
