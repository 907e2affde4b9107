"""Non-finite inputs are not hidden by the kernels."""
import numpy as np
import pytest

from gpu_common import note

pytestmark = pytest.mark.gpu

U1, U3, ULAP, D4, FIELD, ESCALE = 1, 2, 4, 16, 32, 64


def _case(n_g, n_mu, powers):
    from workloads import Correlator, FORM_EE
    rng = np.random.default_rng(n_g + n_mu)
    corr = Correlator(FORM_EE, np.array([[0, 0, o] for o in powers], np.int32),
                      rng.uniform(-0.5, 0.5, (1, len(powers))), 0.9)
    return (corr, rng.normal(size=(3, n_g)), rng.random(n_g), rng.normal(size=(n_mu, n_g)),
            rng.random(n_g), rng.choice(n_g, n_mu, replace=False))


def _dev(a):
    import torch
    return torch.as_tensor(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("powers", [[2, 4], [1, 2, 5], [3, 13]])
@pytest.mark.parametrize("at", [0, 70, 129])
def test_nan_coordinate_reaches_every_channel(powers, at):
    """Every sum holds a pair with the point, whose distance is NaN: |grad u|^2 and the
    Laplacian come out NaN like the gradient channels, and so does the adjoint."""
    from paper_2607_17314_amd import api
    corr, xyz, w, xi, rho, piv = _case(130, 9, powers)
    xyz[1, at] = np.nan
    grid = api.DeviceGrid.from_host(xyz, w)
    note(f"NaN coordinate at {at}, powers {powers}")
    for ch in (U3 | FIELD | ESCALE, U3 | ULAP | FIELD | ESCALE):
        got = api.kernel_contract(grid, corr, _dev(xi), None, _dev(rho), piv, ch, 0)
        for k in ("u3", "ulap", "field"):
            if got[k] is not None:
                assert bool(got[k].isnan().all()), k
        assert np.isnan(got["escale"][[0, 3, 4]]).all()
    cot = {"u3": _dev(np.ones((9, 9)))}
    dtheta, dd = api.grad(grid, corr, _dev(xi), None, _dev(rho), piv, cot, want_d=True)
    assert bool(dtheta.isnan().all()) and bool(dd.isnan().all())


@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("at", [3, 60, 120, 128, 129])
def test_nonfinite_vector_at_a_point_of_zero_weight(at, value):
    """0 * inf and 0 * NaN are NaN in the ket sums of every tile, the first and the last among
    them; the other vectors are untouched."""
    from oracle import contract as oc
    from paper_2607_17314_amd import api
    corr, xyz, w, xi, rho, piv = _case(130, 9, [2, 4])
    bra = (32, 56)   # the point is among the kets alone
    w[at] = 0.0
    note(f"xi[4] = {value} at point {at} of weight 0")
    ref = oc.contract(xyz, w, corr, xi, None, rho[piv], rho, U3, bra_range=bra)["u3"]
    xi[4, at] = value
    got = api.kernel_contract(api.DeviceGrid.from_host(xyz, w), corr, _dev(xi), None, _dev(rho), piv,
                              U3, 0, bra=bra)["u3"].cpu().numpy()
    assert np.isnan(got[:, 4]).all()
    keep = np.arange(9) != 4
    # sums of at most 130 x 24 products, each good to a few 1e-16
    assert np.abs(got[:, keep] - ref[:, keep]).max() < 1e-11 * np.abs(ref).max()


@pytest.mark.parametrize("at", [0, 4, 6, 255, 256, 699])
@pytest.mark.parametrize("where", ["value", "gradient"])
def test_nan_orbital_loses_no_other_point(at, where):
    """A NaN orbital value or derivative at one point takes that point out of the channels that
    it enters; the others are selected as without it. The points 5 and 7 carry the largest
    residuals, next to a NaN."""
    from oracle import pivots
    from paper_2607_17314_amd import api
    rng = np.random.default_rng(at)
    n_g, n_mu = 700, 40
    phi4, w = rng.normal(size=(4, 9, n_g)), rng.random(n_g) + 0.1
    phi4[:, :, 5] *= 9.0
    phi4[:, :, 7] *= 5.0
    w[[5, 7]] = 1.1
    clean = phi4.copy()
    if where == "value":   # enters both channels
        phi4[0, 3, at] = np.nan
        clean[:, :, at] = 0.0
    else:                  # enters the gradient channel alone
        phi4[2, 3, at] = np.nan
        clean[1:, :, at] = 0.0
    ref = pivots.select_fused(clean, w, n_mu).pivots
    note(f"NaN orbital {where} at point {at}")
    got, _, st = api.select_points(_dev(phi4), api.DeviceGrid.from_host(np.zeros((3, n_g)), w), n_mu)
    assert st == 0 and np.array_equal(got, ref)
