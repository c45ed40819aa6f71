"""Single-launch solves with every kernel shape that the other tests do not reach
(rows a thread follow from the mesh's size, the row's length from its kind),
against the streaming kernels from the same state.

Bars as in test_gpu_onchip.py: 1e-11 of the norm in FP64, 1e-8 with the FP32
iteration, counts at most one apart.  That the launch ran, and not the streaming
kernels twice, shows at the end: with a workgroup that stops looking the next step
lasts as long as the others look for it.
"""
import time

import numpy as np
import pytest

from paper_2510_12011_amd import inputs

pytestmark = pytest.mark.gpu

PER_ROW = 256 * 512      # nodes that one row a thread takes


def torus(n):
    """Closed triangle surface, 7 entries a row: a torus of about n nodes."""
    b = 390
    a = n // b
    i, j = np.meshgrid(np.arange(a), np.arange(b), indexing="ij")
    u, v = 2 * np.pi * i.ravel() / a, 2 * np.pi * j.ravel() / b
    r = 0.05 * b / (2 * np.pi)
    R = max(0.05 * a / (2 * np.pi), 1.5 * r)
    xyz = np.stack([(R + r * np.cos(v)) * np.cos(u), (R + r * np.cos(v)) * np.sin(u), r * np.sin(v)], 1)
    at = lambda p, q: (p % a) * b + q % b
    i, j = i.ravel(), j.ravel()
    tri = np.concatenate([np.stack([at(i, j), at(i + 1, j), at(i + 1, j + 1)], 1),
                          np.stack([at(i, j), at(i + 1, j + 1), at(i, j + 1)], 1)]).astype(np.int32)
    return inputs.Mesh(xyz=xyz, tets=tri, grid=xyz.copy(), fibre=None,
                       region=np.zeros(tri.shape[0], np.int32))


def box(n):
    """Kuhn tetrahedra, 15 entries a row: a cube of about n nodes."""
    k = int(round(n ** (1 / 3))) - 1
    return inputs.kuhn_box(k, k, k, 0.1 * k, 0.1 * k, 0.1 * k, jitter=0.05, seed=1, fibre=(0.6, 0.8, 0.0))


def split_box(n):
    """One tetrahedron in six split at its centroid, 19 entries a row (and 5)."""
    m = box(n / 2)
    cut = np.zeros(m.tets.shape[0], bool)
    cut[::6] = True
    t = m.tets[cut]
    c = (m.xyz.shape[0] + np.arange(t.shape[0])).astype(np.int32)
    parts = [m.tets[~cut]]
    for k in range(4):
        q = t.copy()
        q[:, k] = c
        parts.append(q)
    tets = np.concatenate(parts).astype(np.int32)
    xyz = np.concatenate([m.xyz, m.xyz[t].mean(1)])
    return inputs.Mesh(xyz=xyz, tets=tets, grid=xyz.copy(), fibre=None,
                       region=np.zeros(tets.shape[0], np.int32))


def spec_of(mesh, precision):
    x = mesh.xyz[:, 0]
    nodes = np.flatnonzero(x <= x.min() + 0.1 * (x.max() - x.min())).astype(np.int32)
    s = inputs.small_box()
    s.mesh, s.stimuli = mesh, [inputs.Stimulus(nodes, 0.0, 2.0, s.stimuli[0].intensity)]
    s.rtol, s.rel_mode, s.dt = (1e-10, 0, 0.02) if precision == "fp64" else (1e-8, 1, 0.02)
    return s


# (mesh, rows a thread, precision)
SHAPES = ([(torus, r, "fp64") for r in (3, 5)] + [(torus, r, "mixed") for r in (3, 5, 8, 9, 11, 12)] +
          [(box, 3, "fp64")] + [(box, r, "mixed") for r in (5, 8, 9)] +
          [(split_box, r, "fp64") for r in (1, 2)] + [(split_box, r, "mixed") for r in (1, 2, 3, 4)])


def _two_ways(s, steps):
    s.run(3)
    state = s.get_state()
    out = []
    for polls in (20000, 0):
        s.set_tuning(onchip_polls=polls)
        s.set_state(**state)
        v, st = s.run(steps, out_every=steps)
        out.append((np.concatenate([np.ravel(x) for x in v]), st))
        out[-1] += (np.asarray(s.instance_iterations(steps) if getattr(s, "node_ptr", None) is not None
                               else s.iterations(steps)),)
    (v, st, it), (w, su, jt) = out
    print("  rel", np.linalg.norm(v - w) / np.linalg.norm(w), "iterations", it.sum(), jt.sum(), flush=True)
    assert st == su == 0
    assert np.abs(it - jt).max() <= 1
    s.set_tuning(onchip_polls=300_000, onchip_give_up=(1, 0, 1))
    t = time.perf_counter()
    s.run(1)
    assert time.perf_counter() - t > 0.02
    return np.linalg.norm(v - w) / np.linalg.norm(w)


@pytest.mark.parametrize("mesh,rows,precision", SHAPES, ids=lambda p: getattr(p, "__name__", str(p)))
def test_shape_matches_streaming_kernels(mesh, rows, precision):
    from paper_2510_12011_amd import sim
    m = mesh(int((rows - 0.4) * PER_ROW))
    assert (rows - 1) * PER_ROW < m.n_nodes <= rows * PER_ROW, m.n_nodes
    print("[case]", mesh.__name__, rows, precision, m.n_nodes, flush=True)
    err = _two_ways(sim.from_spec(spec_of(m, precision), precision=precision), 8)
    assert err <= (1e-11 if precision == "fp64" else 1e-8)


@pytest.mark.parametrize("mesh,rows", [(torus, 5), (torus, 9), (box, 5)],
                         ids=lambda p: getattr(p, "__name__", str(p)))
def test_batched_shape_matches_streaming_kernels(mesh, rows):
    from paper_2510_12011_amd import sim
    inst = []
    for part in (0.37, 0.6):
        m = mesh(int(part * (rows - 0.2) * PER_ROW))
        inst.append(inputs.Instance(m, 0.17, 0.019, spec_of(m, "mixed").stimuli))
    spec = inputs.BatchSpec(name="two", instances=inst, chi=140.0, cm=0.01, theta=0.5, ionic="ms", dt=0.02,
                            n_steps=40)
    print("[case] batch", mesh.__name__, rows, spec.n_nodes, flush=True)
    assert _two_ways(sim.batch_from_spec(spec), 8) <= 1e-8


def test_batch_against_each_instance_alone():
    """The rows a thread, and with them an instance's blocks, follow from the whole
    batch: 4 here, and alone 1 (the small box) and 2.  Another order of the FP64
    sums may round alpha to the neighbouring FP32 value, which moves a step's
    correction (some 1e-2 of V) by 6e-8 of itself: bar 1e-8 of the norm."""
    from paper_2510_12011_amd import sim
    inst = []
    for k, (nx, ny, nz) in enumerate([(70, 56, 50), (9, 8, 7), (70, 56, 50)]):
        one = inputs.small_box(nx=nx, ny=ny, nz=nz, lx=0.15 * nx, ly=0.15 * ny, lz=0.15 * nz, seed=k)
        inst.append(inputs.Instance(one.mesh, 0.17, 0.019 * (1 + k), one.stimuli))

    def run(instances):
        spec = inputs.BatchSpec(name="boxes", instances=instances, chi=140.0, cm=0.01, theta=0.5, ionic="ms",
                                dt=0.02, n_steps=40)
        print("[case] batch of", len(instances), spec.n_nodes, flush=True)
        s = sim.batch_from_spec(spec)
        v, st = s.run(40, out_every=10)
        assert st == 0
        return np.asarray(v), np.asarray(s.instance_iterations(40)), spec.node_ptr()

    v, it, ptr = run(inst)
    for k, one in enumerate(inst):
        w, jt, _ = run([one])
        part = v[:, ptr[k]:ptr[k + 1]]
        print("  instance", k, "rel", np.linalg.norm(part - w) / np.linalg.norm(w), flush=True)
        assert np.linalg.norm(part - w) <= 1e-8 * np.linalg.norm(w)
        assert np.abs(it[:, k] - jt[:, 0]).max() <= 1
