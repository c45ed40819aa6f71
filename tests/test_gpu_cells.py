"""Cell steps at the edges of their expressions against the oracle.

Potentials at the switch and the removable singularities of the rate
expressions and one ulp beside them, far outside the physiological range, and
at the limit where the kernels hold V (2,400 mV; 3,000 mV).  An exponential's
argument x carries a rounding of |x| 2^-53, and the largest here is 665: 1e-13
relative, some ten such factors to a product: bar 1e-11, of each current's own
size or 1.
"""
import numpy as np
import pytest

import oracle.orc as orc

pytestmark = pytest.mark.gpu

POINTS = {
    "tt": (-40.0, 15.0, -85.23, -56.86, 0.0, 60.0, 200.0, -200.0, 1000.0, -1000.0, 2400.0, -2400.0),
    "crn": (-40.0, -47.13, -14.1, 3.3328, 19.9, -10.0, 7.9, -81.18, 0.0, 60.0, 200.0, -200.0, 1000.0,
            -1000.0, 3000.0, -3000.0),
}


@pytest.mark.parametrize("n", [1, 257])
@pytest.mark.parametrize("kind", ["tt", "crn"])
def test_cell_step_edges(kind, n):
    import torch
    from paper_2510_12011_amd import sim
    s = sim.Simulation(0)
    s.set_ionic(kind)
    at = np.array(POINTS[kind])
    at = np.concatenate([at, np.nextafter(at, 1e4), np.nextafter(at, -1e4)])
    for first in range(0, at.size if n == 1 else 1):
        V = np.resize(np.roll(at, -first), n)
        _, u = orc.ionic_init(kind, n)
        u = np.ascontiguousarray(u * np.linspace(0.9, 1.1, n))
        u_or = u.copy()
        i_or = orc.ionic_step(kind, V, u_or, 0.01)
        Vd, ud = torch.tensor(V, device="cuda:0"), torch.tensor(u, device="cuda:0")
        i_gpu = s.ionic_step(0.01, Vd, ud).cpu().numpy()
        np.testing.assert_allclose(ud.cpu().numpy(), u_or, rtol=1e-11, atol=1e-15)
        np.testing.assert_allclose(i_gpu, i_or, rtol=1e-11, atol=1e-11)


@pytest.mark.parametrize("kind", ["tt", "crn"])
def test_nan_stays(kind):
    """A NaN potential or state is not clipped away."""
    import torch
    from paper_2510_12011_amd import sim
    s = sim.Simulation(0)
    s.set_ionic(kind)
    V, u = orc.ionic_init(kind, 3)
    V[1] = np.nan
    u[2, 2] = np.nan          # the myoplasm's calcium
    Vd, ud = torch.tensor(V, device="cuda:0"), torch.tensor(u, device="cuda:0")
    i_gpu = s.ionic_step(0.01, Vd, ud).cpu().numpy()
    assert np.isfinite(i_gpu[0]) and np.isnan(i_gpu[1:]).all()
    u_gpu = ud.cpu().numpy()
    assert np.isfinite(u_gpu[:, 0]).all() and np.isnan(u_gpu[6:9, 1]).all() and np.isnan(u_gpu[2, 2])
