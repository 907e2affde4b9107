"""The FP64 matrix products at the edges of their tiles, through the orbital values
phi4[c] = C^T ao4[c] (four products per launch) with seeded coefficients: row and column
counts on both sides of 64 and 128, one row, one column, inner dimensions below one k-tile
(10), between tiles (56, 60) and enough tiles for each of the three shapes."""
import numpy as np
import pytest

from gpu_common import note, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("which", ["h2_tiny", "h4", "h6_small"])
@pytest.mark.parametrize("n_orb,n_g", [(1, 1), (1, 4097), (63, 64), (64, 65), (65, 127), (127, 129),
                                       (128, 128), (129, 33000), (200, 9000), (257, 17001)])
def test_orbital_products_at_tile_edges(request, which, n_orb, n_g):
    import torch
    from oracle import orbitals
    from paper_2607_17314_amd import api
    wl = request.getfixturevalue(which)
    rng = np.random.default_rng(n_orb + n_g)
    note(f"orbital products {which}: n_orb={n_orb} n_g={n_g} n_ao={wl.n_ao}")
    xyz = np.ascontiguousarray(rng.normal(scale=2.0, size=(3, n_g)))
    C = rng.normal(size=(wl.n_ao, n_orb))
    n_occ = min(3, n_orb)
    grid = api.DeviceGrid.from_host(xyz, np.ones(n_g))
    phi4, rho = api.eval_orbitals(wl.basis, grid, C, n_occ)
    torch.cuda.synchronize()
    # a sample of the columns, the last ones among them
    at = np.unique(np.concatenate([rng.integers(0, n_g, 200), np.arange(max(0, n_g - 130), n_g)]))
    ref = orbitals.eval_orbitals(wl.basis, C, np.ascontiguousarray(xyz[:, at]))
    # sums of at most 60 products, each factor good to a few units in the last place
    assert rel_err(phi4.cpu().numpy()[:, :, at], ref) < 1e-13
    assert rel_err(rho.cpu().numpy()[at], orbitals.density(ref, n_occ)) < 1e-13
