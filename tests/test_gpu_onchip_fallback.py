"""One workgroup of the single-launch solve stops looking for the others' sums.

Whichever exchange it is, and whether the first workgroup has finished by then
or not, the run's results are the streaming kernels': a step is either solved
by the launch or, as a whole, again.  The last exchange of a solve of k
iterations is the second of iteration k - 1 in FP64 (1 + 8 (k - 1) + 1) and the
second of the residual replacement after it with the FP32 iteration (1 + 8 k + 3).

Bars as in test_gpu_onchip.py, of V and of the states it drives (1e-11 FP64,
1e-8 FP32 iteration, of the norm).  Times are ends of steps: one step apart where
V lies on the threshold.
"""
import functools

import numpy as np
import pytest

from paper_2510_12011_amd import inputs

pytestmark = pytest.mark.gpu

BAR = {"fp64": 1e-11, "mixed": 1e-8}


FIRST = 220   # steps before the one whose solve is disturbed


def _run(precision, steps, polls, give_up=None):
    from paper_2510_12011_amd import sim
    spec = inputs.tiny_cube(n=20)                 # 9,261 nodes, 19 workgroups
    s = sim.from_spec(spec, precision=precision)
    s.set_tuning(onchip_polls=polls)
    s.run(FIRST)
    s.set_tuning(onchip_give_up=give_up)
    _, st = s.run(steps)
    return s.get_state(), s.iterations(steps), st


@functools.lru_cache(maxsize=None)
def _reference(precision, steps):
    return _run(precision, steps, 0)


def _same(got, ref, bar, dt):
    (a, it, st), (b, jt, su) = got, ref
    assert st == su == 0
    assert np.abs(it - jt).max() <= 1
    for k in ("V", "Vprev", "u"):
        assert np.linalg.norm(a[k] - b[k]) <= bar * np.linalg.norm(b[k]), k
    for k in ("lat", "lrt"):
        fin = np.isfinite(b[k])
        assert (np.isfinite(a[k]) == fin).all(), k
        assert np.abs(a[k][fin] - b[k][fin]).max(initial=0.0) <= 1.001 * dt, k


@pytest.mark.parametrize("group,wait", [(0, 0), (7, 0), (7, 1), (18, 1)])
@pytest.mark.parametrize("where", ["first", "middle", "last", "last_of_run"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_one_workgroup_stops_looking(precision, where, group, wait):
    steps = 1 if where == "last_of_run" else 30
    ref = _reference(precision, steps)
    assert np.isfinite(ref[0]["lat"]).any() and ref[1][0] > 2
    k = int(ref[1][0])
    last = 1 + 8 * (k - 1) + 1 if precision == "fp64" else 1 + 8 * k + 3
    exchange = {"first": 1, "middle": 1 + 8 * (k - 2)}.get(where, last)
    print("[case]", precision, where, group, wait, "exchange", exchange, flush=True)
    got = _run(precision, steps, 3000, (exchange, group, wait))
    _same(got, ref, BAR[precision], 0.01)


@pytest.mark.parametrize("group", [0, 2, 5])
def test_one_workgroup_of_a_batch_stops_looking(group):
    """It looks once at each exchange: the first at which another is later than it."""
    from paper_2510_12011_amd import sim
    out = []
    for tuning in (dict(onchip_polls=3000, onchip_give_up=(1, group, 0)), dict(onchip_polls=0)):
        one = [inputs.small_box(nx=n, ny=9, nz=8, lx=0.15 * n, ly=1.4, lz=1.2, seed=n) for n in (12, 20)]
        spec = inputs.BatchSpec(name="boxes", chi=one[0].chi, cm=one[0].cm, theta=0.5, ionic="ms", dt=0.02,
                                n_steps=40,
                                instances=[inputs.Instance(o.mesh, 0.17, 0.019, o.stimuli) for o in one])
        print("[case] batch", group, tuning, flush=True)
        s = sim.batch_from_spec(spec)
        s.set_tuning(**tuning)
        _, st = s.run(40)
        out.append((s.get_state(), np.asarray(s.instance_iterations(40)), st))
    _same(*out, BAR["mixed"], 0.02)


def test_tuning_range():
    from paper_2510_12011_amd import _lib as L, sim
    s = sim.Simulation(0)
    for value, ok in ((0, True), (0xffffff, True), (-1, False), (1 << 24, False)):
        r = L.lib().mdx_set_tuning(s._h, L.MDX_TUNE_ONCHIP_GIVE_UP, value)
        assert r == (L.MDX_OK if ok else L.MDX_ERR_INVALID_ARG)


@pytest.mark.parametrize("first", [5, 18, 20, 22, 35])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_goes_on_after_an_error_of_another_call(precision, first):
    """A run that ends with an error that another call of the thread left behind,
    its solve being in flight; from the state before it the next run is right."""
    from paper_2510_12011_amd import _lib as L, sim
    spec = inputs.tiny_cube(n=20)
    s, w = (sim.from_spec(spec, precision=precision) for _ in range(2))
    w.set_tuning(onchip_polls=0)
    s.run(first)
    state = s.get_state()
    print("[case]", precision, first, s.iterations(first), flush=True)
    assert L.lib().hipSetDevice(99) != 0        # no such device: an error for the caller
    with pytest.raises(L.MdxError) as e:
        s.run(10)
    assert e.value.status == L.MDX_ERR_DEVICE
    out = []
    for t in (s, w):
        t.set_state(**state)
        _, st = t.run(20)
        out.append((t.get_state(), t.iterations(20), st))
    print("  iterations", out[0][1], out[1][1], flush=True)
    _same(*out, BAR[precision], 0.01)
