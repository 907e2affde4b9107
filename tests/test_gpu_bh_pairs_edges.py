"""BH pair values, split and FP64, at the edges of their tiles (32 bra points, ket steps of 16,
16 nuclei at a time): nucleus counts around 16, the most allowed, two types in turn, grids
below one tile and ragged ones, bra ranges, against the oracle."""
import numpy as np
import pytest

from gpu_common import note, rel_err

pytestmark = pytest.mark.gpu

U3, D4, FIELD = 2, 16, 32
MNO = [(m, n, o) for m in range(4) for n in range(m + 1) for o in range(4) if m + n + o > 0]


@pytest.mark.parametrize("n_nuc", [1, 3, 16, 17, 24])
@pytest.mark.parametrize("n_g,n_mu,bra", [(5, 3, None), (64, 9, (3, 36)), (65, 30, None),
                                          (161, 33, (31, 160))])
def test_bh_pair_value_edges(n_nuc, n_g, n_mu, bra):
    import torch
    from oracle import contract as oc
    from paper_2607_17314_amd import _lib as L
    from paper_2607_17314_amd import api
    from workloads import Correlator, FORM_BH
    rng = np.random.default_rng(100 * n_nuc + n_g)
    mno = np.array(MNO, np.int32)
    types = min(n_nuc, 2)
    corr = Correlator(FORM_BH, mno, rng.uniform(-0.5, 0.5, (types, len(mno))) / n_nuc, 0.9,
                      np.array([1.0, 1.3])[:types], 2.0 * rng.normal(size=(n_nuc, 3)),
                      (np.arange(n_nuc) % types).astype(np.int32))
    xyz, w = rng.normal(size=(3, n_g)), rng.random(n_g)
    xi, rho = rng.random((n_mu, n_g)), rng.random(n_g)
    piv = rng.choice(n_g, n_mu, replace=False)
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    ch = U3 | D4 | FIELD
    note(f"BH pair values n_nuc={n_nuc} n_g={n_g} n_mu={n_mu} bra={bra}")
    ref = oc.contract(xyz, w, corr, xi, None, rho[piv], rho, ch, bra_range=bra)
    # a split product is good to 2^-21: u3 sums positive terms, D4 signed ones of at most 161
    # kets (a loss of about sqrt(161)); the field comes from the FP64 pair values
    for prec, tols in ((L.XTC_SPLIT_F16, (1e-6, 1e-5, 1e-11)), (0, (1e-11, 1e-11, 1e-11))):
        got = api.kernel_contract(api.DeviceGrid.from_host(xyz, w), corr, t(xi), None, t(rho), piv,
                                  ch, bra=bra, precision=prec)
        for k, tol in zip(("u3", "D4", "field"), tols):
            assert rel_err(got[k].cpu().numpy(), ref[k]) < tol, (prec, k)
