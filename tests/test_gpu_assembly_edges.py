"""The four-index assembly at sizes around its packing and tiles: one, two and odd orbital
counts, fewer pivots than a k-tile, each output alone and together, with and without X,
whole and one-orbital panels, against the oracle's tensors."""
import numpy as np
import pytest

from gpu_common import note, rel_err

pytestmark = pytest.mark.gpu

K, DU, W = 1, 2, 4


@pytest.mark.parametrize("outputs", [K, DU, W, K | DU | W])
@pytest.mark.parametrize("n,n_mu,with_x", [(1, 1, True), (2, 5, False), (7, 16, True), (11, 17, True),
                                           (13, 40, False), (23, 33, True)])
def test_assembly_edges(outputs, n, n_mu, with_x):
    import torch
    from oracle import assembly as oa
    from paper_2607_17314_amd import api
    rng = np.random.default_rng(31 * n + n_mu)
    phi4 = rng.normal(size=(4, n, n_mu))
    u1, u3, D1, D4 = (rng.normal(size=s) for s in ((3, n_mu, n_mu),) + ((n_mu, n_mu),) * 3)
    X2, X3 = (rng.normal(size=(n, n, n_mu)) for _ in range(2))
    X2, X3 = (X2 + X2.transpose(1, 0, 2), X3 + X3.transpose(1, 0, 2)) if with_x else (None, None)
    t = lambda a: None if a is None else torch.as_tensor(np.ascontiguousarray(a)).cuda()
    note(f"assembly n_orb={n} n_mu={n_mu} X={with_x} outputs={outputs}")
    asm = api.Assembly(t(phi4), t(u1), t(u3), t(D1), t(D4), t(X2), t(X3), outputs=outputs)
    piv = np.arange(n_mu)
    kt, du = oa.k_tensor(phi4, piv, u1, u3), oa.du_tensor(phi4, piv, D1, D4, X2, X3)
    ref = {"K": kt, "dU": du, "W": oa.w_tensor(kt, du)}
    for p0, p1 in ((0, n), (n - 1, n)):
        got = asm.panel(p0, p1)
        for k, bit in (("K", K), ("dU", DU), ("W", W)):
            if outputs & bit:   # panel [p - p0][r][q][s], tensor [p][q][r][s]
                want = ref[k][p0:p1].transpose(0, 2, 1, 3)
                # two nested sums of at most 120 products each
                assert rel_err(got[k].cpu().numpy(), want) < 1e-12, k
            else:
                assert got[k] is None
