"""The single-launch solve against the streaming kernels it stands in for.

The two run the same recurrences; what differs is the order in which the dot
products' partial sums are added (FP64), so
* FP64: alpha and beta differ by some 1e-15 relative, V by far less than the
  solver tolerance 1e-10 lets the iterates move: bar 1e-11;
* FP32 iteration: alpha may round to the neighbouring FP32 value, which moves
  the correction by 6e-8 of itself, and a step's correction is at most some
  1e-2 of V: bar 1e-8.
The stopping test is on the same norms: counts may differ by one where a norm
lies on the threshold.
"""
import numpy as np
import pytest

from paper_2510_12011_amd import inputs

pytestmark = pytest.mark.gpu

# (name, spec, precision, steps): one block; a block boundary inside the mesh
# (512 rows a block); 8-entry and 16-entry rows; 2, 4, 7 and 10 rows a thread;
# and blocks whose last pass is nearly empty
CASES = {
    "one_block": (lambda: inputs.small_box(), "fp64", 40),
    "one_block_mixed": (lambda: inputs.small_box(), "mixed", 40),
    "two_blocks": (lambda: inputs.small_box(nx=7, ny=8, nz=7), "fp64", 40),   # 576 rows
    "surface_642": (lambda: inputs.small_surface(level=3), "fp64", 60),
    "surface_mixed": (lambda: inputs.atrium_surface(7), "mixed", 30),          # R = 2
    "surface_655k": (lambda: inputs.atrium_surface(8), "fp64", 20),            # R = 6
    "cube_fp64": (lambda: inputs.tiny_cube(n=20), "fp64", 60),
    "slab_h0.1_fp64": (lambda: inputs.slab(0.1), "fp64", 20),                  # R = 4
    "slab_h0.08_mixed": (lambda: inputs.slab_precision(0.08), "mixed", 20),    # R = 7
    "shell_mixed": (lambda: inputs.shell_run(1_200_000), "mixed", 10),         # R = 10
}


def _run(spec, precision, steps, **tuning):
    from paper_2510_12011_amd import sim
    s = sim.from_spec(spec, precision=precision, prepare=False)
    s.set_tuning(**tuning)
    s.prepare(spec.dt)
    v, st = s.run(steps, out_every=steps)
    return v[0], s.iterations(steps), st, s.times()[0]


@pytest.mark.parametrize("name", CASES)
def test_matches_streaming_kernels(name):
    build, precision, steps = CASES[name]
    spec = build()
    print("[case]", name, flush=True)
    v, it, st, lat = _run(spec, precision, steps)
    w, jt, su, mat = _run(spec, precision, steps, onchip_polls=0)
    assert st == su == 0
    err = np.linalg.norm(v - w) / np.linalg.norm(w)
    print(name, "rel", err, "iterations", it.sum(), jt.sum(), flush=True)
    assert err <= (1e-11 if precision == "fp64" else 1e-8)
    assert np.abs(it - jt).max() <= 1
    assert (np.isfinite(lat) == np.isfinite(mat)).all()


def test_iteration_cap_and_periodic_replacement():
    """Every solve stopped at the cap, and a replacement every 3 iterations."""
    from paper_2510_12011_amd import sim
    for rtol, max_iter, rr in ((1e-14, 4, 50), (1e-9, 1000, 3)):
        out = []
        for polls in (20000, 0):
            spec = inputs.slab_precision(0.5)
            spec.rtol, spec.max_iter, spec.rr_interval = rtol, max_iter, rr
            print("[case] cap", max_iter, "rr", rr, "polls", polls, flush=True)
            s = sim.from_spec(spec, precision="mixed", prepare=False)
            s.set_tuning(onchip_polls=polls)
            s.prepare(spec.dt)
            v, st = s.run(30, out_every=30)
            out.append((v[0], st, s.iterations(30)))
        (v, st, it), (w, su, jt) = out
        assert st == su and (it == jt).all()
        assert np.linalg.norm(v - w) <= 1e-8 * np.linalg.norm(w)


def test_gives_up_and_falls_back():
    """A launch that may look for the other workgroups' sums only once: the
    step is solved again by the streaming kernels (or the run reports that the
    launch was interrupted), never with a wrong result."""
    from paper_2510_12011_amd import _lib as L
    spec = inputs.tiny_cube(n=20)
    w, jt, su, _ = _run(spec, "fp64", 30, onchip_polls=0)
    print("[case] one poll", flush=True)
    try:
        v, it, st, _ = _run(spec, "fp64", 30, onchip_polls=1)
    except L.MdxError as e:
        assert e.status == L.MDX_ERR_DEVICE
        return
    assert st == 0
    assert np.linalg.norm(v - w) <= 1e-11 * np.linalg.norm(w)
    assert np.abs(it - jt).max() <= 1


def test_simulations_in_turn_share_the_device():
    """Two simulations advanced alternately, and from two threads at once."""
    import threading

    import torch
    from paper_2510_12011_amd import sim
    spec = inputs.tiny_cube(n=20)
    w, *_ = _run(spec, "fp64", 40)
    sims = []
    for _ in range(2):
        with torch.cuda.stream(torch.cuda.Stream()):
            sims.append(sim.from_spec(spec))
    print("[case] alternately", flush=True)
    for _ in range(4):
        for s in sims:
            s.run(5)
    print("[case] two threads", flush=True)
    out = [None, None]

    def go(k):
        out[k] = sims[k].run(20, out_every=20)[0][0]

    th = [threading.Thread(target=go, args=(k,)) for k in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for v in out:
        assert np.array_equal(v, w)
