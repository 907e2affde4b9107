"""Products whose left operand has rows 2^22 elements apart and more take 64-bit offsets within a
tile, closer ones 32-bit offsets: u3 of a few bra points on grids just below and above that size
(xi's row stride is the number of grid points), against the double sum itself."""
import numpy as np
import pytest

from gpu_common import note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_g", [(1 << 22) - 1, (1 << 22) + 5])
def test_u3_over_four_million_points(n_g):
    import torch
    from paper_2607_17314_amd import api
    from workloads import Correlator, FORM_EE
    n_mu, b0, b1 = 65, 100, 133   # a whole 64-row tile and one row, two k-tiles and one point
    corr = Correlator(FORM_EE, np.array([[0, 0, 2], [0, 0, 3]], np.int32), np.array([[0.4, -0.3]]), 0.9)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    f64 = dict(dtype=torch.float64, device="cuda", generator=gen)
    xyz, w = 3.0 * torch.randn((3, n_g), **f64), torch.rand(n_g, **f64)
    xi, rho = torch.randn((n_mu, n_g), **f64), torch.rand(n_g, **f64)
    note(f"u3 on {n_g} points, row stride {'above' if n_g >= 1 << 22 else 'below'} 2^22")
    got = api.kernel_contract(api.DeviceGrid(xyz, w), corr, xi, None, rho, np.arange(n_mu), 2, 0,
                              bra=(b0, b1))["u3"]
    panel = torch.zeros((n_mu, b1 - b0), dtype=torch.float64, device="cuda")
    for s in range(0, n_g, 1 << 18):
        k = slice(s, min(n_g, s + (1 << 18)))
        r = sum((xyz[c, k][:, None] - xyz[c, b0:b1][None]) ** 2 for c in range(3)).sqrt()
        t = 1.0 / (1.0 + 0.9 * r)
        e = 0.9 * r * t
        up = 0.9 * t * t * (2 * 0.4 * e - 3 * 0.3 * e * e)
        panel += (xi[:, k] * w[k]) @ (up * up)
    ref = (xi[:, b0:b1] * w[b0:b1]) @ panel.T
    # sums of 4.2 million terms of random sign: the rounding of the running sum adds about
    # 2^-53 sqrt(4.2e6) = 2e-13 of the result
    assert float((got - ref).abs().max() / ref.abs().max()) < 1e-11
