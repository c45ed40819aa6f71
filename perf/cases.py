"""Performance cases: the work a program has this library do, through its public
entry points.

Whole runs are windows of a time loop that goes on from call to call, as a
program advances a simulation from one saved snapshot of V to the next; every
run is started, and taken past its stimulus, before it is timed.  The meshes
do not depend on the seed; the conductivities' scale, the stimulus site and
all arrays of the other cases do.
"""
import ctypes
import functools
import math
import os

import numpy as np
import torch

from paper_2510_12011_amd import _lib, inputs, learn, sim

DEV = "cuda:0"
RUN_STEPS = {"cube": 0, "slab": 200, "shell": 100, "surface": 200}   # past the 2 ms stimulus


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # a unit-cube test problem, restarted from a checkpoint each time (a
        # parameter study): launches and latency are all there is
        dict(name="tiny_cube", kind="run", geom="cube", size=20, ionic="ms", precision="fp64",
             steps=100, every=50, iters=8),
        # the N-version cuboid at 0.2 mm: a small mesh with a full cell model
        dict(name="slab_58k_fp64", kind="run", geom="slab", size=0.2, ionic="tt", precision="fp64",
             steps=100, every=50, iters=8),
        # the same cuboid at 0.1 mm, the ordinary single-mesh run in FP64
        dict(name="slab_442k_fp64", kind="run", geom="slab", size=0.1, ionic="tt", precision="fp64",
             steps=100, every=50, iters=13),
        # the precision form on a mesh whose matrices leave the caches
        dict(name="slab_871k_mixed", kind="run", geom="slab", size=0.08, ionic="tt",
             precision="mixed", steps=100, every=50, iters=7),
        # the ventricle-like shell with the committed network's warm start: the
        # library's headline workload and the largest case
        dict(name="shell_1255k_learned", kind="run", geom="shell", size=1_200_000, ionic="tt",
             precision="learned", steps=100, every=50, iters=9),
        # the atrial surface, two-variable cells: one iteration a step, so the
        # passes around the solve count
        dict(name="atrium_655k_ms", kind="run", geom="surface", size=8, ionic="ms",
             precision="fp64", steps=200, every=100, iters=1),
        # a coarser atrial surface with the atrial cell model
        dict(name="atrium_164k_crn", kind="run", geom="surface", size=7, ionic="crn",
             precision="fp64", steps=200, every=100, iters=1),
        # a cohort of unstructured shells of uneven sizes in one batched run
        dict(name="cohort_shells", kind="batch", geom="shell", inst=12, size=240_000, steps=100,
             every=50, iters=4),
        # a cohort of atrial surfaces
        dict(name="cohort_surfaces", kind="batch", geom="surface", inst=8, size=7, steps=100,
             every=50, iters=3),
        # single-cell steps of a population of cells on device tensors
        dict(name="cells_tt_300k", kind="cells", ionic="tt", n=300_007),
        # the warm-start network on the nodes of the large shell
        dict(name="network_1255k", kind="network", n=1_255_450),
        # one training step of the network at the training pipeline's batch
        dict(name="train_8192", kind="train", n=8192),
    ]


def draw(rng):
    def log(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    which = rng.choice(["cube", "slab", "slab", "shell", "surface", "batch", "batch", "cells",
                        "cells", "network", "train"])
    if which == "cube":
        return dict(kind="run", geom="cube", size=rng.randint(6, 24), ionic="ms", precision="fp64",
                    steps=rng.randint(40, 120), every=20, iters=8)
    if which == "slab":
        prec = rng.choice(["fp64", "mixed"])
        return dict(kind="run", geom="slab", size=round(log(0.1, 0.5), 4), ionic="tt",
                    precision=prec, steps=rng.randint(40, 100), every=20,
                    iters=13 if prec == "fp64" else 7)
    if which == "shell":
        return dict(kind="run", geom="shell", size=int(log(2e4, 6e5)), ionic="tt",
                    precision=rng.choice(["fp64", "mixed", "learned"]), steps=rng.randint(40, 100),
                    every=20, iters=9)
    if which == "surface":
        return dict(kind="run", geom="surface", size=rng.randint(4, 7),
                    ionic=rng.choice(["ms", "crn"]), precision=rng.choice(["fp64", "mixed"]),
                    steps=rng.randint(80, 200), every=40, iters=1)
    if which == "batch":
        if rng.random() < 0.5:
            return dict(kind="batch", geom="shell", inst=rng.randint(2, 6),
                        size=int(log(2e4, 6e4)), steps=rng.randint(40, 100), every=20, iters=4)
        return dict(kind="batch", geom="surface", inst=rng.randint(2, 16), size=rng.randint(4, 6),
                    steps=rng.randint(40, 100), every=20, iters=3)
    if which == "cells":
        return dict(kind="cells", ionic=rng.choice(["ms", "tt", "crn"]), n=int(log(1e3, 1.2e6)))
    if which == "network":
        return dict(kind="network", n=int(log(2e4, 1.2e6)))
    return dict(kind="train", n=int(log(500, 65536)))


# ---------------------------------------------------------------------------
# problems
# ---------------------------------------------------------------------------
@functools.lru_cache(maxsize=6)
def _mesh(geom, size):
    if geom == "cube":
        return inputs.tiny_cube(n=size).mesh
    if geom == "slab":
        return inputs.slab(h=size).mesh
    if geom == "shell":
        return inputs.shell_run(n_nodes=size).mesh
    return inputs.ellipsoid_surface(size, fibres=False)


@functools.lru_cache(maxsize=3)
def _cohort(geom, inst, size):
    if geom == "shell":
        return inputs.batch_shells(inst, size, n_min=4_000, n_max=60_000)
    return inputs.batch_surfaces(inst, levels=(size, size), axes_mm=(20.0, 40.0), stim_radius=2.0)


def _near(mesh, centre, radius):
    d = np.linalg.norm(mesh.grid - centre, axis=1)
    return np.flatnonzero(d <= radius).astype(np.int32)


def _spec(case, seed):
    """The run's problem statement (inputs.RunSpec)."""
    rng = np.random.default_rng(seed)
    mesh = _mesh(case["geom"], case["size"])
    scale = rng.uniform(0.8, 1.25)
    fp64 = case["precision"] == "fp64"
    if case["geom"] in ("cube", "slab"):   # stimulus: the box at a random corner
        lo, hi = mesh.grid.min(0), mesh.grid.max(0)
        corner = np.where(rng.integers(0, 2, 3) == 1, hi, lo)
        extent = 0.5 if case["geom"] == "cube" else 1.5
        nodes = np.flatnonzero((np.abs(mesh.grid - corner) <= extent + 1e-9).all(1))
        sl, st = (0.1, 0.1) if case["geom"] == "cube" else (0.17, 0.019)
        tol = dict(rtol=1e-10, rel_mode=0) if fp64 else dict(rtol=1e-8, rel_mode=1)
        dt = 0.01
    elif case["geom"] == "shell":
        nodes = inputs.endocardial_site(mesh, int(rng.integers(1 << 30)))
        sl, st, dt = 0.17, 0.019, 0.02
        tol = dict(rtol=3e-9, rel_mode=1)
    else:
        nodes = _near(mesh, mesh.grid[rng.integers(mesh.n_nodes)], 2.0)
        sl, st, dt = 0.4, 0.4, 0.01
        tol = dict(rtol=1e-5, atol=1e-5, rel_mode=1, max_iter=100)
    params = inputs.ATRIUM_MS_PARAMS if case["geom"] == "surface" and case["ionic"] == "ms" else None
    stim = inputs.Stimulus(nodes.astype(np.int32), 0.0, 2.0, 0.5)
    return inputs.RunSpec(name="case", mesh=mesh, sigma_l=sl * scale, sigma_t=st * scale, chi=140.0,
                          cm=0.01, theta=0.5, ionic=case["ionic"], dt=dt, n_steps=case["steps"],
                          stimuli=[stim], warm_start=2 if case["precision"] == "learned" else 1,
                          precision="fp64" if fp64 else "mixed", ionic_params=params, **tol)


def _batch_spec(case, seed):
    rng = np.random.default_rng(seed)
    base = _cohort(case["geom"], case["inst"], case["size"])
    inst = []
    for it in base.instances:
        if case["geom"] == "shell":
            nodes = inputs.endocardial_site(it.mesh, int(rng.integers(1 << 30)))
        else:
            nodes = _near(it.mesh, it.mesh.grid[rng.integers(it.mesh.n_nodes)], 2.0)
        f = rng.uniform(0.8, 1.25)
        inst.append(inputs.Instance(it.mesh, it.sigma_l * f, it.sigma_t * f,
                                    [inputs.Stimulus(nodes, 0.0, 2.0, 0.5)]))
    return inputs.BatchSpec(name="case", instances=inst, chi=base.chi, cm=base.cm, theta=base.theta,
                            ionic=base.ionic, dt=base.dt, n_steps=case["steps"], rtol=base.rtol,
                            precision=base.precision, ionic_params=base.ionic_params)


@functools.lru_cache(maxsize=1)
def _network():
    path = os.path.join(os.path.dirname(_lib.__file__), "weights", "shell_tt_dt0.02.npz")
    params, norm, _ = learn.load(path)
    return params, norm


def _pre(case):
    return RUN_STEPS[case["geom"]]


def _cells(case, seed):
    """V [n] over the range of an action potential and the states of cells
    spread about the model's rest state."""
    rng = np.random.default_rng(seed)
    n = case["n"]
    V = rng.uniform(-90.0, 45.0, n)
    if case["ionic"] == "ms":
        u = rng.uniform(0.0, 1.0, (1, n))
    elif case["ionic"] == "tt":
        u = np.empty((18, n))
        for i, (lo, hi) in enumerate([(130.0, 145.0), (6.0, 12.0), (5e-5, 1.2e-3), (1.0, 5.0),
                                      (1e-4, 1e-2), (0.3, 1.0)]):
            u[i] = rng.uniform(lo, hi, n)
        u[6:] = rng.uniform(0.0, 1.0, (12, n))
    else:
        u = np.empty((20, n))
        for i, (lo, hi) in enumerate([(9.0, 14.0), (130.0, 145.0), (5e-5, 1e-3), (0.5, 2.0),
                                      (0.1, 2.0)]):
            u[i] = rng.uniform(lo, hi, n)
        u[5:] = rng.uniform(0.0, 1.0, (15, n))
    return V, u


def _training(case, seed):
    """Recorded rows (features as a run records them), a batch's indices, and
    the optimiser's state in the middle of a training run."""
    rng = np.random.default_rng(seed)
    params, norm = _network()
    rows = 4 * case["n"]
    X = (norm[:4] + norm[4:8] * rng.standard_normal((rows, 4))).astype(np.float32)
    dV = (X[:, 1] + norm[8] * rng.standard_normal(rows)).astype(np.float32)
    idx = rng.permutation(rows)[:case["n"]].astype(np.int64)
    p = (params + 0.01 * rng.standard_normal(params.size)).astype(np.float32)
    m = (1e-3 * rng.standard_normal(p.size)).astype(np.float32)
    v = rng.uniform(1e-5, 1e-4, p.size).astype(np.float32)
    return X, dV, idx, p, m, v, norm


# ---------------------------------------------------------------------------
# prepare / run
# ---------------------------------------------------------------------------
def prepare(case, seed):
    st = dict(case=case)
    if case["kind"] == "run":
        s = sim.from_spec(_spec(case, seed))
        if case["precision"] == "learned":
            learn.install(s, *_network())
        if case["geom"] == "cube":
            s.run(20)
            st["checkpoint"] = s.get_state()
        else:
            s.run(_pre(case))
        st["sim"] = s
    elif case["kind"] == "batch":
        s = sim.batch_from_spec(_batch_spec(case, seed))
        s.autotune(reps=10)
        s.set_tuning(graph=True)
        s.run(200)
        st["sim"] = s
    elif case["kind"] == "cells":
        s = sim.Simulation(0)
        s.set_ionic(case["ionic"])
        V, u = _cells(case, seed)
        st.update(sim=s, V=torch.from_numpy(V).to(DEV), u=torch.from_numpy(u).to(DEV))
    elif case["kind"] == "network":
        g = torch.Generator(device=DEV)
        g.manual_seed(int(seed))
        st.update(sim=sim.Simulation(0), P=torch.from_numpy(_network()[0]).to(DEV),
                  X=torch.randn((case["n"], 4), generator=g, device=DEV),
                  y=torch.empty(case["n"], device=DEV))
    else:
        X, dV, idx, p, m, v, norm = _training(case, seed)
        n = case["n"]
        nb = _lib.lib().mdx_mlp_grad_scratch(n)
        st.update(sim=sim.Simulation(0), t=100, norm=np.ascontiguousarray(norm), nb=nb,
                  X=torch.from_numpy(X).to(DEV), dV=torch.from_numpy(dV).to(DEV),
                  idx=torch.from_numpy(idx).to(DEV), P=torch.from_numpy(p).to(DEV),
                  m=torch.from_numpy(m).to(DEV), v=torch.from_numpy(v).to(DEV),
                  Xb=torch.empty((n, 4), device=DEV), Tb=torch.empty(n, device=DEV),
                  G=torch.empty(p.size, device=DEV), loss=torch.empty(1, device=DEV),
                  scratch=torch.empty(nb // 4 + 64, device=DEV))
    return st


def _p(t):
    return ctypes.c_void_p(t.data_ptr())


def run(st):
    case, s = st["case"], st["sim"]
    if case["kind"] == "run":
        if "checkpoint" in st:   # resume the checkpoint, advance, checkpoint again
            s.set_state(**st["checkpoint"])
            snaps, _ = s.run(case["steps"], out_every=case["every"])
            end = s.get_state()
            return {"V": snaps, "u": end["u"], "Vprev": end["Vprev"], "lat": end["lat"]}
        return {"V": s.run(case["steps"], out_every=case["every"])[0]}
    if case["kind"] == "batch":
        return {"V": s.run(case["steps"], out_every=case["every"])[0]}
    if case["kind"] == "cells":
        i = s.ionic_step(0.01, st["V"], st["u"])
        return {"iion": i, "u": st["u"]}
    lib = _lib.lib()
    if case["kind"] == "network":
        s._check(lib.mdx_mlp_forward(s._h, _p(st["P"]), case["n"], _p(st["X"]), _p(st["y"])))
        return st["y"]
    n = case["n"]
    nm = st["norm"].ctypes.data_as(ctypes.c_void_p)
    st["t"] += 1
    s._check(lib.mdx_mlp_samples(s._h, n, _p(st["idx"]), 4 * n, _p(st["X"]), _p(st["dV"]), nm,
                                 _p(st["Xb"]), _p(st["Tb"])))
    s._check(lib.mdx_mlp_grad(s._h, _p(st["P"]), n, _p(st["Xb"]), _p(st["Tb"]), _p(st["G"]),
                              _p(st["loss"]), _p(st["scratch"]), st["nb"]))
    s._check(lib.mdx_mlp_adam(s._h, _p(st["P"]), _p(st["m"]), _p(st["v"]), _p(st["G"]), st["t"],
                              2e-3, 0.9, 0.999, 1e-8))
    return {"P": st["P"], "m": st["m"], "v": st["v"], "grad": st["G"], "loss": st["loss"]}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
STATES = {"ms": 1, "tt": 18, "crn": 20}
CELL_FLOPS = {"ms": 40, "tt": 1500, "crn": 1700}


def work(case):
    n_par = 8705
    if case["kind"] == "cells":
        return {"bytes": case["n"] * 8.0 * (2 * STATES[case["ionic"]] + 2),
                "flops": float(case["n"] * CELL_FLOPS[case["ionic"]])}
    if case["kind"] == "network":
        return {"bytes": case["n"] * 20.0 + 4 * n_par, "flops": case["n"] * 17024.0}
    if case["kind"] == "train":
        return {"bytes": case["n"] * 28.0 + 4.0 * 7 * n_par, "flops": case["n"] * 3 * 17024.0}
    if case["kind"] == "run":
        n, ionic = _mesh(case["geom"], case["size"]).n_nodes, case["ionic"]
        fp32 = case["precision"] != "fp64"
    else:
        n, ionic = _cohort(case["geom"], case["inst"], case["size"]).n_nodes, "ms"
        fp32 = True
    row = 7.0 if case["geom"] == "surface" else 15.0   # nonzeros of a row
    cell = 8.0 * (2 * STATES[ionic] + 2)
    # M, K and a 16-bit column; V, its predecessor, the source; x, r and the diagonal
    rhs = 18.0 * row + 48.0
    # one iteration: A and a column; the vectors an iteration reads and writes
    it = (6.0 * row + 52.0) if fp32 else (10.0 * row + 104.0)
    return {"bytes": case["steps"] * n * (cell + rhs + case["iters"] * it)
            + 8.0 * n * (case["steps"] // case["every"]),
            "flops": case["steps"] * n * (CELL_FLOPS[ionic] + row * (8 + 2.0 * case["iters"]))}


# ---------------------------------------------------------------------------
# the same in 64 bits, in torch
# ---------------------------------------------------------------------------
def _ms(V, u, dt, p):
    tau_in, tau_out, tau_open, tau_close, gate, rest, amp = p
    w = (V - rest) / amp
    up = w < gate
    inf = up.double()
    tau = torch.where(up, torch.full_like(w, tau_open), torch.full_like(w, tau_close))
    h = inf - (inf - u[0]) * torch.exp(-dt / tau)
    return -amp * (h * w * w * (1 - w) / tau_in - w / tau_out), h[None]


def _gate(y, inf, tau, dt):
    return inf - (inf - y) * torch.exp(-dt / tau)


def _tt_current(V, c, g):
    """The twelve currents of the ten Tusscher-Panfilov model (pA/pF)."""
    F, RTF = 96485.3415, 8314.472 * 310.0 / 96485.3415
    ki, nai, cai, _, cass, _ = c
    xr1, xr2, xs, m, h, j, d, f, f2, fc, s, r = g
    ek = RTF * torch.log(5.4 / ki)
    ena = RTF * torch.log(140.0 / nai)
    eks = RTF * torch.log((5.4 + 0.03 * 140.0) / (ki + 0.03 * nai))
    eca = 0.5 * RTF * torch.log(2.0 / cai)
    phi = V / RTF
    a = 0.1 / (1 + torch.exp(0.06 * (V - ek - 200)))
    b = (3 * torch.exp(0.0002 * (V - ek + 100)) + torch.exp(0.1 * (V - ek - 10))) / (
        1 + torch.exp(-0.5 * (V - ek)))
    w = 2 * (V - 15) / RTF
    drive = torch.where(w == 0, torch.ones_like(w), w / torch.expm1(w))
    i = {}
    i["K1"] = 5.405 * a / (a + b) * (V - ek)
    i["to"] = 0.073 * r * s * (V - ek)
    i["Kr"] = 0.153 * xr1 * xr2 * (V - ek)
    i["Ks"] = 0.392 * xs ** 2 * (V - eks)
    i["Na"] = 14.838 * m ** 3 * h * j * (V - ena)
    i["bNa"] = 2.9e-4 * (V - ena)
    i["CaL"] = 3.98e-5 * d * f * f2 * fc * 2 * F * drive * (0.25 * cass * torch.exp(w) - 2.0)
    i["bCa"] = 5.92e-4 * (V - eca)
    i["NaK"] = 2.724 * (5.4 / 6.4) * nai / (
        (nai + 40) * (1 + 0.1245 * torch.exp(-0.1 * phi) + 0.0353 * torch.exp(-phi)))
    i["NaCa"] = 1000.0 * (torch.exp(0.35 * phi) * nai ** 3 * 2.0
                          - torch.exp(-0.65 * phi) * 140.0 ** 3 * cai * 2.5) / (
        (87.5 ** 3 + 140.0 ** 3) * (1.38 + 2.0) * (1 + 0.1 * torch.exp(-0.65 * phi)))
    i["pCa"] = 0.1238 * cai / (0.0005 + cai)
    i["pK"] = 0.0146 * (V - ek) / (1 + torch.exp((25 - V) / 5.98))
    return i


def _tt(V, u, dt, _):
    e = torch.exp
    F, cap, vc, vsr, vss = 96485.3415, 0.185, 0.016404, 0.001094, 0.00005468
    c, g = list(u[:6]), list(u[6:])
    ki, nai, cai, casr, cass, rbar = c
    ca2 = (cass / 0.05) ** 2
    low = V < -40.0
    ah = torch.where(low, 0.057 * e(-(V + 80) / 6.8), torch.zeros_like(V))
    bh = torch.where(low, 2.7 * e(0.079 * V) + 3.1e5 * e(0.3485 * V),
                     0.77 / (0.13 * (1 + e(-(V + 10.66) / 11.1))))
    aj = torch.where(low, (-25428.0 * e(0.2444 * V) - 6.948e-6 * e(-0.04391 * V)) * (V + 37.78)
                     / (1 + e(0.311 * (V + 79.23))), torch.zeros_like(V))
    bj = torch.where(low, 0.02424 * e(-0.01052 * V) / (1 + e(-0.1378 * (V + 40.14))),
                     0.6 * e(0.057 * V) / (1 + e(-0.1 * (V + 32))))
    hinf = 1 / (1 + e((V + 71.55) / 7.43)) ** 2
    inf_tau = [
        (1 / (1 + e((-26 - V) / 7)),
         450 / (1 + e((-45 - V) / 10)) * 6 / (1 + e((V + 30) / 11.5))),
        (1 / (1 + e((V + 88) / 24)), 3 / (1 + e((-60 - V) / 20)) * 1.12 / (1 + e((V - 60) / 20))),
        (1 / (1 + e((-5 - V) / 14)),
         1400 / torch.sqrt(1 + e((5 - V) / 6)) / (1 + e((V - 35) / 15)) + 80),
        (1 / (1 + e((-56.86 - V) / 9.03)) ** 2,
         1 / (1 + e((-60 - V) / 5)) * (0.1 / (1 + e((V + 35) / 5)) + 0.1 / (1 + e((V - 50) / 200)))),
        (hinf, 1 / (ah + bh)),
        (hinf, 1 / (aj + bj)),
        (1 / (1 + e((-8 - V) / 7.5)),
         (1.4 / (1 + e((-35 - V) / 13)) + 0.25) * 1.4 / (1 + e((V + 5) / 5))
         + 1 / (1 + e((50 - V) / 20))),
        (1 / (1 + e((V + 20) / 7)), 1102.5 * e(-(V + 27) ** 2 / 225) + 200 / (1 + e((13 - V) / 10))
         + 180 / (1 + e((V + 30) / 10)) + 20),
        (0.67 / (1 + e((V + 35) / 7)) + 0.33,
         562 * e(-(V + 27) ** 2 / 240) + 31 / (1 + e((25 - V) / 10)) + 80 / (1 + e((V + 30) / 10))),
        (0.6 / (1 + ca2) + 0.4, 80 / (1 + ca2) + 2),
        (1 / (1 + e((V + 28) / 5)), 1000 * e(-(V + 67) ** 2 / 1000) + 8),
        (1 / (1 + e((20 - V) / 6)), 9.5 * e(-(V + 40) ** 2 / 1800) + 0.8),
    ]
    i = _tt_current(V, c, g)
    new = [_gate(y, inf, tau, dt) for y, (inf, tau) in zip(g, inf_tau)]
    kcasr = 2.5 - 1.5 / (1 + (1.5 / casr) ** 2)
    k1 = 0.15 / kcasr
    rel = 0.102 * k1 * cass ** 2 * rbar / (0.06 + k1 * cass ** 2) * (casr - cass)
    up = 0.006375 / (1 + 0.00025 ** 2 / cai ** 2)
    leak, xfer = 0.00036 * (casr - cai), 0.0038 * (cass - cai)
    d = [
        -(i["K1"] + i["to"] + i["Kr"] + i["Ks"] - 2 * i["NaK"] + i["pK"]) * cap / (vc * F),
        -(i["Na"] + i["bNa"] + 3 * i["NaK"] + 3 * i["NaCa"]) * cap / (vc * F),
        ((leak - up) * vsr / vc + xfer - (i["bCa"] + i["pCa"] - 2 * i["NaCa"]) * cap / (2 * vc * F))
        / (1 + 0.2 * 0.001 / (cai + 0.001) ** 2),
        (up - rel - leak) / (1 + 10.0 * 0.3 / (casr + 0.3) ** 2),
        (-i["CaL"] * cap / (2 * vss * F) + rel * vsr / vss - xfer * vc / vss)
        / (1 + 0.4 * 0.00025 / (cass + 0.00025) ** 2),
        -0.045 * kcasr * cass * rbar + 0.005 * (1 - rbar),
    ]
    c = [y + dt * dy for y, dy in zip(c, d)]
    return sum(_tt_current(V, c, new).values()), torch.stack(c + new)


def _crn_current(V, y):
    """The twelve currents of the Courtemanche-Ramirez-Nattel model (pA/pF)."""
    e = torch.exp
    RTF = 8.3143 * 310.0 / 96.4867
    na, k, ca = y[0], y[1], y[2]
    m, h, j, oa, oi, ua, ui, xr, xs, d, f, fca = y[5:17]
    ena, ek, eca = (RTF * torch.log(140.0 / na), RTF * torch.log(5.4 / k),
                    0.5 * RTF * torch.log(1.8 / ca))
    w = V / RTF
    i = {}
    i["Na"] = 7.8 * m ** 3 * h * j * (V - ena)
    i["K1"] = 0.09 * (V - ek) / (1 + e(0.07 * (V + 80)))
    i["to"] = 0.1652 * oa ** 3 * oi * (V - ek)
    i["Kur"] = (0.005 + 0.05 / (1 + e((15 - V) / 13))) * ua ** 3 * ui * (V - ek)
    i["Kr"] = 0.029411765 * xr * (V - ek) / (1 + e((V + 15) / 22.4))
    i["Ks"] = 0.12941176 * xs ** 2 * (V - ek)
    i["CaL"] = 0.12375 * d * f * fca * (V - 65)
    sig = (math.exp(140.0 / 67.3) - 1) / 7
    i["NaK"] = (0.59933874 / (1 + 0.1245 * e(-0.1 * w) + 0.0365 * sig * e(-w))
                / (1 + (10.0 / na) ** 1.5) * 5.4 / 6.9)
    i["NaCa"] = 1600.0 * (e(0.35 * w) * na ** 3 * 1.8 - e(-0.65 * w) * 140.0 ** 3 * ca) / (
        (87.5 ** 3 + 140.0 ** 3) * (1.38 + 1.8) * (1 + 0.1 * e(-0.65 * w)))
    i["bNa"] = 6.744375e-4 * (V - ena)
    i["bCa"] = 1.131e-3 * (V - eca)
    i["pCa"] = 0.275 * ca / (0.0005 + ca)
    return i


def _ratio(x, s):
    """x / (1 - exp(-x / s)), s at x = 0."""
    t = x / s
    return torch.where(t == 0, torch.full_like(x, s), x / -torch.expm1(-t))


def _crn(V, u, dt, _):
    e = torch.exp
    F, cap, vi, vup, vrel = 96.4867, 100.0, 13668.0, 1109.52, 96.48
    y = list(u)
    na, k, ca, cu, cr = y[:5]
    i = _crn_current(V, y)
    rel = 30.0 * y[17] ** 2 * y[18] * y[19] * (cr - ca)
    tr, up, leak = (cu - cr) / 180.0, 0.005 / (1 + 0.00092 / ca), 0.005 * cu / 15.0
    kc = cap / (F * vi)
    fn = 1e-12 * vrel * rel - 5e-13 / F * cap * (0.5 * i["CaL"] - 0.2 * i["NaCa"])
    on = 1 / (1 + e(-(fn - 3.4175e-13) / 13.67e-16))
    low = V < -40.0
    zero = torch.zeros_like(V)
    am, bm = 0.32 * _ratio(V + 47.13, 10.0), 0.08 * e(-V / 11)
    ah = torch.where(low, 0.135 * e(-(V + 80) / 6.8), zero)
    bh = torch.where(low, 3.56 * e(0.079 * V) + 3.1e5 * e(0.35 * V),
                     1 / (0.13 * (1 + e(-(V + 10.66) / 11.1))))
    aj = torch.where(low, (-127140 * e(0.2444 * V) - 3.474e-5 * e(-0.04391 * V)) * (V + 37.78)
                     / (1 + e(0.311 * (V + 79.23))), zero)
    bj = torch.where(low, 0.1212 * e(-0.01052 * V) / (1 + e(-0.1378 * (V + 40.14))),
                     0.3 * e(-2.535e-7 * V) / (1 + e(-0.1 * (V + 32))))
    aa = 0.65 / (e(-(V + 10) / 8.5) + e(-(V - 30) / 59))
    ba = 0.65 / (2.5 + e((V + 82) / 17))
    oi = 1 / (18.53 + e((V + 113.7) / 10.95)) + 1 / (35.56 + e(-(V + 1.26) / 7.44))
    ui = 1 / (21 + e(-(V - 185) / 28)) + e((V - 158) / 16)
    ar = 0.0003 * _ratio(V + 14.1, 5.0)
    br = 7.3898e-5 * _ratio(-(V - 3.3328), 5.1237)
    a_s, b_s = 4e-5 * _ratio(V - 19.9, 17.0), 3.5e-5 * _ratio(-(V - 19.9), 9.0)
    rd = 0.035 * _ratio(V + 10, 6.24) * (1 + e(-(V + 10) / 6.24))
    rw = _ratio(V - 7.9, 5.0) * (1 + 0.3 * e(-(V - 7.9) / 5)) / 6.0
    inf_rate = [
        (am / (am + bm), am + bm), (ah / (ah + bh), ah + bh), (aj / (aj + bj), aj + bj),
        (1 / (1 + e(-(V + 20.47) / 17.54)), 3 * (aa + ba)),
        (1 / (1 + e((V + 43.1) / 5.3)), 3 * oi),
        (1 / (1 + e(-(V + 30.3) / 9.6)), 3 * (aa + ba)),
        (1 / (1 + e((V - 99.45) / 27.48)), 3 * ui),
        (1 / (1 + e(-(V + 14.1) / 6.5)), ar + br),
        (1 / torch.sqrt(1 + e(-(V - 19.9) / 12.7)), 2 * (a_s + b_s)),
        (1 / (1 + e(-(V + 10) / 8)), rd),
        (1 / (1 + e((V + 28) / 6.9)), (0.0197 * e(-0.0337 ** 2 * (V + 10) ** 2) + 0.02) / 9),
        (1 / (1 + ca / 0.00035), zero + 0.5),
        (on, zero + 1 / 8.0),
        (1 - 1 / (1 + e(-(fn - 6.835e-14) / 13.67e-16)), 1 / (1.91 + 2.09 * on)),
        (1 - 1 / (1 + e(-(V - 40) / 17)), rw),
    ]
    d = [
        -kc * (3 * (i["NaK"] + i["NaCa"]) + i["bNa"] + i["Na"]),
        kc * (2 * i["NaK"] - (i["K1"] + i["to"] + i["Kur"] + i["Kr"] + i["Ks"])),
        (0.5 * kc * (2 * i["NaCa"] - i["pCa"] - i["CaL"] - i["bCa"])
         + (vup * (leak - up) + vrel * rel) / vi)
        / (1 + 0.07 * 0.0005 / (ca + 0.0005) ** 2 + 0.05 * 0.00238 / (ca + 0.00238) ** 2),
        up - leak - tr * vrel / vup,
        (tr - rel) / (1 + 10.0 * 0.8 / (cr + 0.8) ** 2),
    ]
    new = [a + dt * b for a, b in zip(y[:5], d)]
    new += [inf - (inf - g) * e(-dt * r) for g, (inf, r) in zip(y[5:], inf_rate)]
    return sum(_crn_current(V, new).values()), torch.stack(new)


CELL = {"ms": _ms, "tt": _tt, "crn": _crn}
MS_PARAMS = (0.3, 6.0, 120.0, 150.0, 0.13, -80.0, 100.0)
REST = {"ms": (-80.0, [1.0]),
        "tt": (-85.23, [136.89, 8.604, 0.000126, 3.64, 0.00036, 0.9073, 0.00621, 0.4712, 0.0095,
                        0.00172, 0.7444, 0.7045, 3.373e-5, 0.7888, 0.9755, 0.9953, 0.999998,
                        2.42e-8]),
        "crn": (-81.18, [11.17, 139.0, 1.013e-4, 1.488, 1.488, 2.908e-3, 0.9649, 0.9775, 3.043e-2,
                         0.9992, 4.966e-3, 0.9986, 3.296e-5, 1.869e-2, 1.367e-4, 0.9996, 0.7755,
                         0.0, 1.0, 0.9992])}


def _matrices(mesh, sl, st):
    """P1 mass and stiffness matrices (sparse CSR, FP64); sl, st per element."""
    x = torch.from_numpy(np.ascontiguousarray(mesh.xyz)).to(DEV)
    el = torch.from_numpy(mesh.tets.astype(np.int64)).to(DEV)
    nv = el.shape[1]
    p = x[el]
    E = p[:, 1:] - p[:, :1]                                  # edge vectors [m, nv-1, 3]
    if nv == 4:   # gradients of nodes 1..3: the dual basis of the edges
        dual = torch.stack([torch.linalg.cross(E[:, (a + 1) % 3], E[:, (a + 2) % 3])
                            for a in range(3)], 1)
        det = (E[:, 0] * dual[:, 0]).sum(1)
        grad = dual / det[:, None, None]
        vol = det.abs() / 6.0
    else:         # the same within the triangle's plane, from the edges' metric
        g00, g01, g11 = ((E[:, a] * E[:, b]).sum(1) for a, b in ((0, 0), (0, 1), (1, 1)))
        det = g00 * g11 - g01 * g01
        grad = torch.stack([g11[:, None] * E[:, 0] - g01[:, None] * E[:, 1],
                            g00[:, None] * E[:, 1] - g01[:, None] * E[:, 0]], 1) / det[:, None, None]
        vol = torch.sqrt(det) / 2.0
    grad = torch.cat([-grad.sum(1, keepdim=True), grad], 1)  # [m, nv, 3]
    K = (grad[:, :, None, :] * grad[:, None, :, :]).sum(3) * st[:, None, None]
    if mesh.fibre is not None:   # tetrahedra only: the surfaces here are isotropic
        f = torch.from_numpy(np.ascontiguousarray(mesh.fibre)).to(DEV)
        gf = (grad * f[:, None, :]).sum(2)
        K = K + (sl - st)[:, None, None] * gf[:, :, None] * gf[:, None, :]
    K = K * vol[:, None, None]
    M = (torch.ones((nv, nv), dtype=torch.float64, device=DEV)
         + torch.eye(nv, dtype=torch.float64, device=DEV)) * (vol / (nv * (nv + 1)))[:, None, None]
    i = el[:, :, None].expand(-1, nv, nv).reshape(-1)
    j = el[:, None, :].expand(-1, nv, nv).reshape(-1)
    n = mesh.n_nodes
    return [torch.sparse_coo_tensor(torch.stack([i, j]), A.reshape(-1), (n, n)).coalesce()
            for A in (M, K)]


def _reference(mesh, sl, st, spec, params, pre, steps, every):
    """The time loop with every system solved to rounding: V snapshots of the
    last `steps` steps, and the final V_prev, u and activation times."""
    M, K = _matrices(mesh, sl, st)
    dt, chi, cm, theta = spec.dt, spec.chi, spec.cm, spec.theta
    A = (M * (chi * cm) + K * (theta * dt)).coalesce()
    i, j = A.indices()
    dinv = torch.zeros(mesh.n_nodes, dtype=torch.float64, device=DEV)
    dinv.index_put_((i[i == j],), 1.0 / A.values()[i == j])
    M, K, A = M.to_sparse_csr(), K.to_sparse_csr(), A.to_sparse_csr()
    v0, u0 = REST[spec.ionic]
    V = torch.full((mesh.n_nodes,), v0, dtype=torch.float64, device=DEV)
    Vp = V.clone()
    u = torch.tensor(u0, dtype=torch.float64, device=DEV)[:, None].repeat(1, mesh.n_nodes)
    lat = torch.full_like(V, math.inf)
    snaps = []
    for k in range(pre + steps):
        iion, u = CELL[spec.ionic](V, u, dt, params)
        s = -cm * iion
        for stim in spec.stimuli:
            if round(stim.start / dt) <= k < round((stim.start + stim.duration) / dt):
                s[torch.from_numpy(stim.nodes.astype(np.int64)).to(DEV)] += stim.intensity
        b = chi * (M @ (cm * V + dt * s)) - (1 - theta) * dt * (K @ V)
        x = 2 * V - Vp
        r = b - A @ x
        z = dinv * r
        p, rho = z.clone(), r @ z
        stop = 1e-14 * float(torch.linalg.norm(dinv * b))
        for _ in range(80):
            if float(torch.linalg.norm(z)) <= stop:
                break
            q = A @ p
            a = rho / (p @ q)
            x = x + a * p
            r = r - a * q
            z = dinv * r
            new = r @ z
            p = z + (new / rho) * p
            rho = new
        V, Vp = x, V
        lat = torch.where(torch.isinf(lat) & (V > 0), torch.full_like(lat, (k + 1) * dt), lat)
        if k >= pre and (k + 1 - pre) % every == 0:
            snaps.append(V.cpu().numpy())
    return {"V": np.stack(snaps) if snaps else np.zeros((0, mesh.n_nodes)), "u": u.cpu().numpy(),
            "Vprev": Vp.cpu().numpy(), "lat": lat.cpu().numpy()}


def _per_element(values, counts):
    return torch.from_numpy(np.repeat(np.asarray(values, np.float64), counts)).to(DEV)


def _net(P, X):
    """The network on FP64 activations with its BF16 weights."""
    def bf(a):
        return a + (a.to(torch.bfloat16).double() - a).detach()
    cut = torch.split(P, [256, 64, 4096, 64, 4096, 64, 64, 1])
    h = torch.relu(X @ bf(cut[0]).view(64, 4).t() + cut[1])
    h = torch.relu(h @ bf(cut[2]).view(64, 64).t() + cut[3])
    h = torch.relu(h @ bf(cut[4]).view(64, 64).t() + cut[5])
    return h @ bf(cut[6]) + cut[7]


def exact(case, seed):
    if case["kind"] == "run":
        spec = _spec(case, seed)
        m = spec.mesh.tets.shape[0]
        pre = 20 if case["geom"] == "cube" else _pre(case)
        out = _reference(spec.mesh, _per_element([spec.sigma_l], [m]),
                         _per_element([spec.sigma_t], [m]), spec, spec.ionic_params or MS_PARAMS,
                         pre, case["steps"], case["every"])
        return out if case["geom"] == "cube" else {"V": out["V"]}
    if case["kind"] == "batch":
        b = _batch_spec(case, seed)
        ptr = b.node_ptr()
        one = [it.mesh for it in b.instances]
        fib = None if one[0].fibre is None else np.concatenate([m.fibre for m in one])
        mesh = inputs.Mesh(xyz=np.concatenate([m.xyz for m in one]),
                           tets=np.concatenate([m.tets + ptr[k] for k, m in enumerate(one)]),
                           grid=np.zeros((0, 3)), fibre=fib, region=np.zeros(0, np.int32))
        b.stimuli = [inputs.Stimulus(s.nodes + ptr[k], s.start, s.duration, s.intensity)
                     for k, it in enumerate(b.instances) for s in it.stimuli]
        count = [m.tets.shape[0] for m in one]
        out = _reference(mesh, _per_element([i.sigma_l for i in b.instances], count),
                         _per_element([i.sigma_t for i in b.instances], count), b,
                         b.ionic_params or MS_PARAMS, 200, case["steps"], case["every"])
        return {"V": out["V"]}
    if case["kind"] == "cells":
        V, u = (torch.from_numpy(a).to(DEV) for a in _cells(case, seed))
        iion, u = CELL[case["ionic"]](V, u, 0.01, MS_PARAMS)
        return {"iion": iion, "u": u}
    if case["kind"] == "network":
        X = prepare(case, seed)["X"].double()
        return _net(torch.from_numpy(_network()[0]).double().to(DEV), X)
    X, dV, idx, p, m, v, norm = _training(case, seed)
    X, dV = X[idx].astype(np.float64), dV[idx].astype(np.float64)
    x = torch.from_numpy((X - norm[:4]) / norm[4:8]).to(DEV)
    t = torch.from_numpy((dV - X[:, 1]) / norm[8]).to(DEV)
    P, m, v = (torch.from_numpy(a.astype(np.float64)).to(DEV) for a in (p, m, v))
    P.requires_grad_(True)
    loss = ((_net(P, x) - t) ** 2).mean()
    g, = torch.autograd.grad(loss, P)
    m = 0.9 * m + 0.1 * g
    v = 0.999 * v + 0.001 * g * g
    step = 2e-3 * (m / (1 - 0.9 ** 101)) / (torch.sqrt(v / (1 - 0.999 ** 101)) + 1e-8)
    return {"P": P.detach() - step, "m": m, "v": v, "grad": g, "loss": loss.detach()[None]}
