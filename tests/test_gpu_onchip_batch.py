"""The batch's single-launch solve against the streaming kernels.

Both iterate with FP32 matrix values and replace the residual in FP64; the
order of the dot products' sums differs, so alpha may round to the neighbouring
FP32 value, which moves a step's correction (some 1e-2 of V) by 6e-8 of itself:
bar 1e-8 of the norm.  The stopping tests are on the same norms: counts may
differ by one where a norm lies on the threshold.
"""
import functools

import numpy as np
import pytest

from paper_2510_12011_amd import inputs

pytestmark = pytest.mark.gpu


def _boxes(shapes):
    inst = []
    for k, (nx, ny, nz) in enumerate(shapes):
        one = inputs.small_box(nx=nx, ny=ny, nz=nz, lx=0.15 * nx, ly=0.15 * ny, lz=0.15 * nz, seed=k)
        inst.append(inputs.Instance(one.mesh, 0.17, 0.019 * (1 + k), one.stimuli))
    return inputs.BatchSpec(name="boxes", instances=inst, chi=one.chi, cm=one.cm, theta=0.5, ionic="ms",
                            dt=0.02, n_steps=40)


# one instance in one workgroup; instances of one to several workgroups, with
# rows of 7, 15 and (unstructured) up to 33 entries; 1, 2, 3, 4 and 10 rows a
# thread
COHORTS = {
    "one_box": lambda: _boxes([(6, 5, 4)]),
    "boxes": lambda: _boxes([(7, 7, 7), (12, 9, 8), (3, 3, 2), (7, 8, 7)]),
    "boxes_r4": lambda: _boxes([(70, 56, 50), (70, 56, 50), (9, 8, 7)]),
    "surfaces": lambda: inputs.batch_surfaces(3, levels=(4, 5), axes_mm=(20.0, 40.0), stim_radius=2.0),
    "surfaces_r10": lambda: inputs.batch_surfaces(8, levels=(7, 7), axes_mm=(20.0, 40.0),
                                                  stim_radius=2.0),
    "shells": lambda: inputs.batch_shells(5, 20_000, n_min=500, n_max=9_000),
    "shells_r2": lambda: inputs.batch_shells(10, 160_000, n_min=4_000, n_max=60_000),
}


@functools.lru_cache(maxsize=1)
def _cohort(name):
    return COHORTS[name]()


def _run(spec, steps=40, **tuning):
    from paper_2510_12011_amd import sim
    print("[case]", spec.name, spec.n_nodes, tuning, flush=True)
    s = sim.batch_from_spec(spec)
    s.set_tuning(**tuning)
    v, st = s.run(steps, out_every=steps // 2)
    return np.concatenate([np.asarray(x).ravel() for x in v]), np.asarray(s.instance_iterations(steps)), st


def _close(a, b):
    assert np.linalg.norm(a[0] - b[0]) <= 1e-8 * np.linalg.norm(b[0])
    assert np.abs(a[1] - b[1]).max() <= 1
    assert a[2] == b[2]


@pytest.mark.parametrize("name", list(COHORTS))
def test_matches_streaming_kernels(name):
    spec = _cohort(name)
    ref = _run(spec, onchip_polls=0, graph=True)
    got = _run(spec)
    print("  rel", np.linalg.norm(got[0] - ref[0]) / np.linalg.norm(ref[0]), "iterations",
          ref[1].sum(), got[1].sum(), flush=True)
    _close(got, ref)
    again = _run(spec, graph=True)
    assert np.array_equal(again[0], got[0])


@pytest.mark.parametrize("name", ["boxes", "boxes_r4", "surfaces", "shells", "shells_r2"])
def test_adds_rows_as_the_tuned_layout(name):
    """The layout that the autotuner installs sets the order of a row's FP32
    sum: against the streaming kernels with that layout, chosen by hand."""
    from paper_2510_12011_amd import sim
    spec = _cohort(name)
    s = sim.batch_from_spec(spec)
    r = s.autotune(reps=5)
    v, st = s.run(40, out_every=20)
    print("  tuned", r["fmt"], r["lanes_per_row"], flush=True)
    got = np.concatenate([np.asarray(x).ravel() for x in v]), np.asarray(s.instance_iterations(40)), st
    ref = _run(spec, fmt=r["fmt"], lanes_per_row=r["lanes_per_row"], tiles_per_group=r["tiles_per_group"])
    print("  rel", np.linalg.norm(got[0] - ref[0]) / np.linalg.norm(ref[0]), flush=True)
    _close(got, ref)


def test_cap_and_periodic_replacement():
    """Every solve stopped at the cap, and a replacement every 2 iterations."""
    for rtol, max_iter, rr in ((1e-14, 4, 50), (1e-9, 1000, 2)):
        spec = _boxes([(7, 7, 7), (12, 9, 8), (3, 3, 2)])
        spec.rtol, spec.max_iter, spec.rr_interval = rtol, max_iter, rr
        a, b = _run(spec, 20), _run(spec, 20, onchip_polls=0)
        _close(a, b)


def test_gives_up_and_falls_back():
    """A launch that may look for the other workgroups' sums only once: the
    step is solved again by the streaming kernels."""
    spec = _boxes([(12, 9, 8), (9, 8, 7)])
    _close(_run(spec, 20, onchip_polls=1), _run(spec, 20, onchip_polls=0))


def test_layout_tunings_select_streaming():
    """A layout chosen by hand is run: bitwise the streaming kernels' result."""
    spec = _boxes([(7, 7, 7), (3, 3, 2)])
    a = _run(spec, 20, fmt="sell", lanes_per_row=2)
    b = _run(spec, 20, fmt="sell", lanes_per_row=2, onchip_polls=0)
    assert np.array_equal(a[0], b[0])
