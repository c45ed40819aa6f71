"""Simulations in several threads: their single-launch solves may be in flight
together as far as the CUs reach, and wait for each other beyond that.  Results
are bitwise those of each simulation alone: nobody gives up.
"""
import threading
import time

import numpy as np
import pytest

from paper_2510_12011_amd import inputs

pytestmark = pytest.mark.gpu


def _sim(spec, **kw):
    import torch
    from paper_2510_12011_amd import sim
    with torch.cuda.stream(torch.cuda.Stream()):
        if isinstance(spec, inputs.BatchSpec):
            return sim.batch_from_spec(spec)
        return sim.from_spec(spec, **kw)


def _threads(calls):
    out = [None] * len(calls)

    def go(k):
        try:
            out[k] = calls[k]()
        except Exception as e:      # shown by the caller
            out[k] = e

    th = [threading.Thread(target=go, args=(k,)) for k in range(len(calls))]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for o in out:
        if isinstance(o, Exception):
            raise o
    return out


def test_a_small_solve_does_not_wait_for_another():
    """A launch of 19 workgroups that lasts (one of them stops looking at the
    first exchange, once its own looks and the others' are used up) leaves the
    device to other simulations': to one of four at least, since streams may share
    a hardware queue."""
    spec = inputs.tiny_cube(n=20)
    sims = [_sim(spec) for _ in range(5)]
    for s in sims:
        s.run(5)
    sims[0].set_tuning(onchip_polls=1_000_000, onchip_give_up=(1, 3, 1))

    def run(k):
        time.sleep(0.03 if k else 0.0)
        t = time.perf_counter()
        sims[k].run(3)
        return time.perf_counter() - t

    print("[case] one lasts", flush=True)
    took = _threads([lambda k=k: run(k) for k in range(5)])
    print(took, flush=True)
    assert took[0] > 0.1      # the launch did last
    assert min(took[1:]) < 0.05


# (simulations, steps): together more CUs than the device has; a batch beside
# single meshes
MIXES = {
    "tiny": ([("tiny", "fp64")] * 6, 40),
    "large": ([("slab", "fp64"), ("slab", "mixed"), ("tiny", "mixed")], 10),
    "batch": ([("shells", None), ("tiny", "fp64"), ("surface", "mixed")], 30),
}


def _spec(name):
    return {"tiny": lambda: inputs.tiny_cube(n=20), "slab": lambda: inputs.slab(0.1),
            "surface": lambda: inputs.atrium_surface(7),
            "shells": lambda: inputs.batch_shells(4, 40_000, n_min=500, n_max=20_000)}[name]()


@pytest.mark.parametrize("name", list(MIXES))
def test_threads_give_the_same_bits(name):
    sims, steps = MIXES[name]
    alone = []
    for kind, precision in sims:
        s = _sim(_spec(kind), **({"precision": precision} if precision else {}))
        alone.append(np.concatenate([np.ravel(v) for v in s.run(steps, out_every=steps)[0]]))
        s.close()
    ss = [_sim(_spec(kind), **({"precision": precision} if precision else {})) for kind, precision in sims]
    print("[case]", name, flush=True)
    got = _threads([lambda s=s: s.run(steps, out_every=steps) for s in ss])
    for (v, st), ref in zip(got, alone):
        assert st == 0
        assert np.array_equal(np.concatenate([np.ravel(x) for x in v]), ref)


def test_persistent_batch_beside_single_launches():
    """The persistent batched iteration fills the device and waits for all of its
    workgroups too: it and the single launches take turns."""
    spec = inputs.batch_shells(4, 40_000, n_min=500, n_max=20_000)
    b = _sim(spec)
    b.set_tuning(persistent=True)
    ref = np.concatenate([np.ravel(v) for v in b.run(20, out_every=20)[0]])
    b.prepare(spec.dt)
    b.set_tuning(persistent=True)
    s = [_sim(inputs.tiny_cube(n=20)) for _ in range(2)]
    print("[case] persistent", flush=True)
    out = _threads([lambda: b.run(20, out_every=20)] + [lambda t=t: t.run(60, out_every=60) for t in s])
    assert np.array_equal(np.concatenate([np.ravel(v) for v in out[0][0]]), ref)
    assert np.array_equal(out[1][0], out[2][0])
