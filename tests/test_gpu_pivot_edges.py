"""Pivot selection around the sizes of its candidate search and planned batches: grids of
fewer points than candidates, around 64 and 512 points, one orbital, more pivots than one
planned batch, exact ties (repeated points) and an early rank-deficient stop, against the
oracle's selection index for index."""
import numpy as np
import pytest

from gpu_common import note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_g,n_orb,n_mu,repeat", [(1, 1, 1, False), (7, 2, 3, False), (63, 3, 5, False),
                                                   (64, 4, 9, True), (65, 5, 14, False),
                                                   (511, 12, 70, False), (513, 12, 60, True),
                                                   (1500, 14, 97, False), (2100, 16, 120, True)])
def test_selection_matches_oracle(n_g, n_orb, n_mu, repeat):
    import torch
    from oracle import pivots
    from paper_2607_17314_amd import api
    rng = np.random.default_rng(n_g + n_orb)
    phi4, w = rng.normal(size=(4, n_orb, n_g)), rng.random(n_g) + 0.1
    if repeat:   # every third point repeats its predecessor: exact ties, the lower index first
        phi4[:, :, 2::3] = phi4[:, :, 1:-1:3][:, :, :phi4[:, :, 2::3].shape[2]]
        w[2::3] = w[1:-1:3][:w[2::3].shape[0]]
    ref = pivots.select_fused(phi4, w, n_mu)
    gaps = [g for g in ref.scalar_state.gaps + ref.grad_state.gaps if g != 0.0]
    note(f"select n_g={n_g} n_orb={n_orb} n_mu={n_mu} repeat={repeat}: smallest gap but ties "
         f"{min(gaps) if gaps else 0.0:.1e}")
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    got, info, st = api.select_points(t(phi4), api.DeviceGrid.from_host(np.zeros((3, n_g)), w), n_mu)
    assert np.array_equal(got, ref.pivots)
    assert int(info[0]) == len(ref.scalar) and int(info[1]) == len(ref.grad)


def test_selection_stops_at_the_numerical_rank():
    """Three orbitals span six pair products: the scalar channel ends there."""
    import torch
    from oracle import pivots
    from paper_2607_17314_amd import api
    rng = np.random.default_rng(5)
    n_g, n_mu = 300, 40
    phi4, w = np.zeros((4, 3, n_g)), rng.random(n_g) + 0.1
    phi4[:, :, :] = rng.normal(size=(4, 3, n_g))
    ref = pivots.select_fused(phi4, w, n_mu)
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    got, info, st = api.select_points(t(phi4), api.DeviceGrid.from_host(np.zeros((3, n_g)), w), n_mu)
    assert st > 0 and len(got) < n_mu
    assert len(got) == len(ref.pivots) and int(info[0]) == len(ref.scalar) == 6
