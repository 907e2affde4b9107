"""FP64 stage 1 at the edges of its tiles (128- or 96-row by 32-bra tiles, 16-ket steps):
grids below one ket step and around multiples of 16 and 32, row counts around a tile with
the two density rows, bra ranges, and powers of rbar in both polynomial lengths with and
without an o = 1 term, against the oracle on seeded rows."""
import numpy as np
import pytest

from gpu_common import note, rel_err

pytestmark = pytest.mark.gpu

U3, ULAP, D4, FIELD, ESCALE = 2, 4, 16, 32, 64


@pytest.mark.parametrize("powers", [[2, 4, 6, 8], [1, 2, 5], [1, 3, 13]])
@pytest.mark.parametrize("n_g,n_mu,bra", [(5, 3, None), (16, 16, None), (31, 30, (7, 24)),
                                          (33, 9, (1, 33)), (48, 1, None), (130, 94, None),
                                          (193, 95, (32, 161)), (257, 126, None), (161, 127, None)])
def test_stage1_edges(powers, n_g, n_mu, bra):
    import torch
    from oracle import contract as oc
    from paper_2607_17314_amd import api
    from workloads import Correlator, FORM_EE
    rng = np.random.default_rng(n_g * 7 + n_mu)
    corr = Correlator(FORM_EE, np.array([[0, 0, o] for o in powers], np.int32),
                      rng.uniform(-0.5, 0.5, (1, len(powers))), 0.9)
    xyz, w = rng.normal(size=(3, n_g)), rng.random(n_g)
    xi, rho = rng.normal(size=(n_mu, n_g)), rng.random(n_g)
    piv = rng.choice(n_g, n_mu, replace=False)
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    for ch in (U3 | D4 | FIELD | ESCALE, U3 | ULAP | D4 | FIELD | ESCALE):
        note(f"stage 1 n_g={n_g} n_mu={n_mu} bra={bra} powers={powers} channels={ch}")
        got = api.kernel_contract(api.DeviceGrid.from_host(xyz, w), corr, t(xi), None, t(rho), piv,
                                  ch, 0, bra=bra)
        ref = oc.contract(xyz, w, corr, xi, None, rho[piv], rho, ch, bra_range=bra)
        for k in ("u3", "ulap", "D4", "field"):
            if ref.get(k) is not None:
                # double sums of at most 257 x 257 signed terms, each good to a few 1e-16
                assert rel_err(got[k].cpu().numpy(), ref[k]) < 1e-11, k
        # E3, E4 (here from u3 and D4; the device's from the density rows) and E3x, E4x
        for i in (0, 1, 3, 4):
            assert abs(got["escale"][i] - ref["escale"][i]) <= 1e-10 * abs(ref["escale"]).max(), i
