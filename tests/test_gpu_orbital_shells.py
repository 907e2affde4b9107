"""Orbital values over shells of every angular momentum the library takes (0 to 6), in orders
and numbers that leave the shell groups of a launch uneven, on one point to more than a chunk."""
import numpy as np
import pytest

from gpu_common import note, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ls", [[0], [6], [0, 1, 2, 3, 4, 5, 6], [2, 0, 5, 1, 1, 6, 3, 0, 4, 2, 1]])
@pytest.mark.parametrize("n_g", [1, 257, 33000])
def test_every_angular_momentum(ls, n_g):
    import torch
    from oracle import orbitals
    from paper_2607_17314_amd import api
    from workloads.basis import Basis
    rng = np.random.default_rng(len(ls) + n_g)
    n_prim = rng.integers(1, 4, len(ls))
    start = np.concatenate([[0], np.cumsum(n_prim)]).astype(np.int32)
    basis = Basis(rng.normal(size=(3, 3)), rng.integers(0, 3, len(ls)).astype(np.int32),
                  np.array(ls, np.int32), start, 0.3 + rng.random(start[-1]), rng.normal(size=start[-1]))
    n_ao = sum((l + 1) * (l + 2) // 2 for l in ls)
    xyz, C = rng.normal(size=(3, n_g)), rng.normal(size=(n_ao, 7))
    note(f"orbital shells l={ls} n_g={n_g} n_ao={n_ao}")
    phi4, rho = api.eval_orbitals(basis, api.DeviceGrid.from_host(xyz, np.ones(n_g)), C, 3)
    at = np.unique(np.concatenate([rng.integers(0, n_g, 200), np.arange(max(0, n_g - 130), n_g)]))
    ref = orbitals.eval_orbitals(basis, C, np.ascontiguousarray(xyz[:, at]))
    # sums of at most 130 signed products, each factor good to a few units in the last place
    assert rel_err(phi4.cpu().numpy()[:, :, at], ref) < 1e-12
    assert rel_err(rho.cpu().numpy()[at], orbitals.density(ref, 3)) < 1e-12
