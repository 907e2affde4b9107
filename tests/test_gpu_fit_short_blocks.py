"""The kept factors of fits whose last diagonal block has fewer than 64 rows (the panels past
them are left out): L and the inverses of its 64 x 64 diagonal blocks, zero past the rows."""
import numpy as np
import pytest

from gpu_common import note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_mu", [2, 5, 16, 17, 32, 33, 48, 49, 64, 65, 80, 81, 113])
def test_factor_of_a_short_block(n_mu):
    import torch
    from paper_2607_17314_amd import api
    rng = np.random.default_rng(n_mu)
    n_g, n_orb = 150, 40
    phi4 = rng.normal(size=(4, n_orb, n_g))
    xyz, w = rng.normal(size=(3, n_g)), 0.5 + rng.random(n_g)
    piv = rng.choice(n_g, n_mu, replace=False)
    note(f"factor n_mu={n_mu}")
    grid = api.DeviceGrid.from_host(xyz, w)
    chol = api.fit_ex(torch.as_tensor(phi4).cuda(), grid, piv, xi=False, xigrad=False, keep_chol=True)[3].cpu().numpy()
    P = phi4[:, :, piv]
    for s in range(4):
        L = np.linalg.cholesky((P[0].T @ P[0]) * (P[s].T @ P[s]))
        got = np.tril(chol[s, :n_mu * n_mu].reshape(n_mu, n_mu))
        inv = chol[s, n_mu * n_mu:].reshape(-1, 64, 64)
        # condition below 100, at most 113 products a sum
        assert np.abs(got - L).max() < 1e-11 * np.abs(L).max()
        for b in range(inv.shape[0]):
            nb = min(64, n_mu - 64 * b)
            ref = np.linalg.inv(L[64 * b:64 * b + nb, 64 * b:64 * b + nb])
            assert np.abs(inv[b, :nb, :nb] - ref).max() < 1e-11 * np.abs(ref).max()
            assert not inv[b, nb:].any() and not inv[b, :, nb:].any()
