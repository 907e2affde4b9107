"""The Gauss-Newton step at the edges of its parts (block reductions up to 16 parameters, 4 x 4
blocks of C above, tiles of walkers, a thread per row of the factorisation), against the oracle."""
import numpy as np
import pytest

from gpu_common import note, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_params", [1, 16, 17, 18, 64, 127, 128])
@pytest.mark.parametrize("n_walkers", [2, 63, 129, 1025])
def test_gn_step_edges(n_params, n_walkers):
    import torch
    from oracle import vmc
    from paper_2607_17314_amd import api
    rng = np.random.default_rng(n_params * 31 + n_walkers)
    E = rng.normal(size=n_walkers)
    E[0] += 40.0   # clipped where there are walkers enough
    dE = rng.normal(size=(n_walkers, n_params))
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    note(f"Gauss-Newton n_walkers={n_walkers} n_params={n_params}")
    ref, _, _, st = vmc.gn_step(E, dE, 2.0, 0.5)
    delta, stats = api.vmc_gn_step(t(E), t(dE), 2.0, 0.5)
    # C + lambda of condition below 100, sums of at most 1,025 terms
    assert rel_err(np.asarray(torch.as_tensor(delta).cpu()), ref) < 1e-11
