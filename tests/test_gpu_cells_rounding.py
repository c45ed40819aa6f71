"""Rounding of the ten Tusscher-Panfilov m gate's step, the gate whose formula has the most
roundings.  The expressions as published, evaluated with numpy in FP64, are the
measure: over cells with V over its range, the kernel's relative rms error
against 80-bit arithmetic may be no more than 5% above theirs (the rms of 60,000
cells scatters by 1%).
"""
import numpy as np
import pytest

import oracle.orc as orc

pytestmark = pytest.mark.gpu


def _m_step(V, m, dt):
    T = V.dtype.type
    one = T(1)
    inf = one / (one + np.exp((T(-56.86) - V) / T(9.03))) ** 2
    tau = (one / (one + np.exp((T(-60) - V) / T(5)))) * (
        T(0.1) / (one + np.exp((V + T(35)) / T(5))) + T(0.1) / (one + np.exp((V - T(50)) / T(200))))
    return inf - (inf - m) * np.exp(-T(dt) / tau)


@pytest.mark.parametrize("dt", [0.005, 0.01, 0.02])
def test_m_gate_rounding(dt):
    import torch
    from paper_2510_12011_amd import sim
    n = 60_000
    rng = np.random.default_rng(5)
    V = rng.uniform(-90.0, 40.0, n)
    _, u = orc.ionic_init("tt", n)
    u = np.ascontiguousarray(u)
    u[9] = rng.uniform(0.001, 0.999, n)
    m = u[9].copy()
    s = sim.Simulation(0)
    s.set_ionic("tt")
    ud = torch.tensor(u, device="cuda:0")
    s.ionic_step(dt, torch.tensor(V, device="cuda:0"), ud)
    exact = _m_step(V.astype(np.longdouble), m.astype(np.longdouble), dt)
    rms = lambda a: float(np.sqrt(np.mean(((a - exact) / exact).astype(float) ** 2)))
    got, direct = rms(ud[9].cpu().numpy()), rms(_m_step(V, m, dt))
    print("rms", got, "as published, FP64", direct)
    assert got <= 1.05 * direct
