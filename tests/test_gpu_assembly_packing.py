"""The four-index assembly on both sides of the rule that packs the pairs of its projections (more
64 x 64 tiles than 256, N_mu rows by n_orb^2 columns), ragged sizes, against the oracle's tensors;
and the one-body pieces, which are formed from the same factors."""
import numpy as np
import pytest

from gpu_common import note, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_mu,with_x", [(3, 9, True), (45, 447, True), (33, 895, False),   # 224, 252 tiles
                                           (49, 449, False), (33, 965, True)])                # 304, 288
def test_assembly_on_both_sides_of_the_packing_rule(n, n_mu, with_x):
    import torch
    from oracle import assembly as oa
    from paper_2607_17314_amd import api
    rng = np.random.default_rng(31 * n + n_mu)
    phi4 = rng.normal(size=(4, n, n_mu))
    u1, u3, D1, D4 = (rng.normal(size=s) for s in ((3, n_mu, n_mu),) + ((n_mu, n_mu),) * 3)
    X2, X3 = (rng.normal(size=(n, n, n_mu)) for _ in range(2))
    X2, X3 = (X2 + X2.transpose(1, 0, 2), X3 + X3.transpose(1, 0, 2)) if with_x else (None, None)
    t = lambda a: None if a is None else torch.as_tensor(np.ascontiguousarray(a)).cuda()
    tiles = -(-n_mu // 64) * -(-n * n // 64)
    note(f"assembly n_orb={n} n_mu={n_mu} X={with_x}: {tiles} tiles")
    args = [t(a) for a in (phi4, u1, u3, D1, D4, X2, X3)]
    piv = np.arange(n_mu)
    kt, du = oa.k_tensor(phi4, piv, u1, u3), oa.du_tensor(phi4, piv, D1, D4, X2, X3)
    ref = {"K": kt, "dU": du, "W": oa.w_tensor(kt, du)}
    asm = api.Assembly(*args, outputs=7)
    alone = {k: api.Assembly(*args, outputs=bit) for k, bit in (("K", 1), ("dU", 2), ("W", 4))}
    for p0, p1 in ((0, 2), (n - 1, n)):
        got = asm.panel(p0, p1)
        for k in ("K", "dU", "W"):
            # two nested sums of at most 4 x 965 signed products each, rounded to 1e-16 per product
            assert rel_err(got[k].cpu().numpy(), ref[k][p0:p1].transpose(0, 2, 1, 3)) < 1e-12, k
            assert torch.equal(alone[k].panel(p0, p1)[k], got[k])
    dh, f, e0 = api.one_body(*args, n_occ=2, e_nuc=0.5)
    rdh = oa.delta_h(du, 2)
    assert rel_err(dh.cpu().numpy(), rdh) < 1e-12
    assert rel_err(f.cpu().numpy(), oa.fock_xtc(rdh, ref["W"], 2)) < 1e-12
    assert abs(e0 - oa.e0_xtc(rdh, 2, 0.5)) < 1e-12 * abs(rdh).max()
