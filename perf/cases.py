"""Timed cases: what a QED-PIC program has this framework do, step after step.

``listed()`` holds the cases, ``draw(rng)`` gives one more of the same ranges,
``prepare(case, seed)`` what the program holds before the call (particles, fields, the
context with its launch shapes and network), ``run(state)`` one pass through the
public entry points, ``work(case)`` the bytes and operations that a pass cannot do
without, ``exact(case, seed)`` the results in 64 bits where there is a closed form.

A pass of a "step" case starts from the prepared momenta: the leptons' momenta, the
photon records and the live counts are put back from the program's own copy (as a
caller does that repeats a step), then the steps run, each with the next step number.
Positions of the leptons and optical depths run on, as in a simulation.

The order in which a step appends particles is unspecified, so the appended particles
(and the photons, which the compaction moves) are returned sorted by id, as a program
writes them to a file.  The hot spots of 16.8 million electrons return the electrons
and the counts only: sorting their eight million photons takes as long as the step; the
same kernels' photons come back whole in the smaller cases.
"""
import json
import math
import os

import numpy as np
import torch

from paper_2008_10468_amd import qed

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(qed.__file__)))
LAST = torch.iinfo(torch.int64).max

# Per population: dt, and per lepton and step about: emissions, sub-steps of Algorithm 1
# (P_max 0.01) and of the optical-depth path (0.1), flops of a sub-step (field kind).
POPULATION = {
    "ring": {"dt": 8.37e4, "emissions": 0.50, "sub": 54.1, "sub_depth": 6.0, "flops": 139},
    "laser": {"dt": 10358.42, "emissions": 0.0178, "sub": 2.45, "sub_depth": 1.01, "flops": 100},
    "spot": {"dt": 2.0696e5, "emissions": 0.293, "sub": 27.7, "sub_depth": 3.62, "flops": 139},
    "weak": {"dt": 1.0e8, "emissions": 0.83, "sub": 90.0, "sub_depth": 9.5, "flops": 139},
    "shower": {"dt": 3.0e5, "emissions": 1.71, "sub": 177.0, "sub_depth": 18.0, "flops": 139},
}
# slots per lepton that a pass may append as photons, and as pairs
GROWTH = {"ring": (1.0, 0.0), "laser": (0.025, 0.002), "spot": (0.65, 0.0), "weak": (1.2, 0.0), "shower": (4.5, 0.8)}


def listed():
    return [
        # a small population in double precision: the correctness configuration of 16,384
        # electrons in a uniform magnetic field, which cannot fill the chip
        {"name": "ring_f64", "path": "step", "population": "ring", "n": 16384, "precision": "f64",
         "scheduler": "naive", "sampler": "rejection", "steps": 1},
        # the plain generator's full physics (emission, pair creation, compaction) in a
        # rotating laser field: 1,048,576 electrons, 262,144 photons, eight steps
        {"name": "laser_plain", "path": "step", "population": "laser", "n": 1048576, "precision": "mixed",
         "scheduler": "naive", "sampler": "rejection", "steps": 8},
        # the same population on the optical-depth paths of leptons and photons
        {"name": "laser_depth", "path": "step", "population": "laser", "n": 1048576, "precision": "mixed",
         "scheduler": "naive", "sampler": "learned", "steps": 8},
        # the uneven batch: one electron in ten in a hot spot of up to a thousand
        # sub-steps
        {"name": "spot_plain", "path": "step", "population": "spot", "n": 16777216, "precision": "mixed",
         "scheduler": "binned", "sampler": "rejection", "steps": 1},
        # the same on the optical-depth path with the learned energies
        {"name": "spot_learned", "path": "step", "population": "spot", "n": 16777216, "precision": "mixed",
         "scheduler": "binned", "sampler": "learned", "steps": 1},
        # a domain's share of it, ragged, with its photons written out
        {"name": "spot_share", "path": "step", "population": "spot", "n": 300007, "precision": "mixed",
         "scheduler": "binned", "sampler": "learned", "steps": 1},
        # in-step cascades: each pass follows the particles that the previous one made
        {"name": "shower", "path": "step", "population": "shower", "n": 65536, "precision": "mixed",
         "scheduler": "naive", "sampler": "rejection", "steps": 1},
        # a whole small PIC step: gather, generator, deposition, in a field with E and B at
        # general angles; launches and latency count
        {"name": "pic_small", "path": "pic", "n": 24571, "cells": 16, "precision": "mixed", "steps": 3},
        # field interpolation to a million particles in random order, 64^3 cells
        {"name": "gather_random", "path": "gather", "n": 1048576, "nx": 64, "ny": 64, "nz": 64, "precision": "mixed",
         "order": "random"},
        # current deposition of two million particles in random order, uneven axes
        {"name": "deposit_random", "path": "deposit", "n": 2000003, "nx": 96, "ny": 50, "nz": 61,
         "precision": "mixed", "order": "random"},
        # the synchrotron functions over a large array (the paper's own microbenchmark)
        {"name": "synchrotron_f32", "path": "synchrotron", "n": 67108867, "precision": "mixed"},
        # training of the sampler's network: table, 400 optimizer steps, validation
        {"name": "train", "path": "train", "steps": 400, "target": 0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["step", "step", "step", "step", "pic", "gather", "deposit", "deposit", "synchrotron", "train"])
    if path == "step":
        pop = rng.choice(["ring", "laser", "laser", "spot", "spot", "weak", "shower"])
        case = {"path": "step", "population": pop, "precision": "mixed", "scheduler": "naive",
                "sampler": "rejection", "steps": 1}
        if pop == "ring":
            case["precision"] = rng.choice(["f64", "mixed"])
            case["n"] = _log_int(rng, 1000, 262144)
            case["scheduler"] = rng.choice(["naive", "binned", "tiled"])
        elif pop == "laser":
            case["n"] = _log_int(rng, 20000, 1048576)
            case["scheduler"] = rng.choice(["naive", "naive", "tiled"])
            case["sampler"] = rng.choice(["rejection", "learned"])
            case["steps"] = rng.randint(2, 8)
        elif pop == "shower":
            case["n"] = _log_int(rng, 500, 65536)
        else:
            case["n"] = _log_int(rng, 30000, 4194304 if pop == "spot" else 1048576)
            case["scheduler"] = "binned"
            case["sampler"] = rng.choice(["rejection", "learned", "fitted"])
        return case
    if path == "pic":
        return {"path": "pic", "n": _log_int(rng, 2000, 200000), "cells": rng.randint(8, 32),
                "precision": rng.choice(["mixed", "mixed", "f64"]), "steps": rng.randint(1, 4)}
    if path in ("gather", "deposit"):
        return {"path": path, "n": _log_int(rng, 3000, 2000000), "nx": _log_int(rng, 8, 128),
                "ny": _log_int(rng, 8, 128), "nz": _log_int(rng, 8, 128),
                "precision": rng.choice(["mixed", "mixed", "f64"]), "order": rng.choice(["random", "cell"])}
    if path == "synchrotron":
        return {"path": path, "n": _log_int(rng, 2000, 67108867), "precision": rng.choice(["mixed", "f64"])}
    return {"path": "train", "steps": _log_int(rng, 50, 400), "target": rng.randint(0, 1)}


# ---------------------------------------------------------------- inputs

class Buffers(qed.SpeciesBuffers):
    """Device buffers of one species, momenta and weight in one block and the positions in
    another (rows of 64-slot multiples), so that a program copies and sorts them at once."""

    def __init__(self, capacity, real, parent, events, tau, birth):
        cap = (int(capacity) + 63) // 64 * 64
        self.capacity, self.real = cap, real
        self.mom = torch.zeros(4, cap, dtype=real, device="cuda")
        self.pos = torch.zeros(3, cap, dtype=torch.float64, device="cuda")
        self.ux, self.uy, self.uz, self.w = self.mom
        self.x, self.y, self.z = self.pos
        self.n = torch.zeros(1, dtype=torch.int64, device="cuda")
        self.id = torch.zeros(cap, dtype=torch.int64, device="cuda")
        self.parent = torch.zeros(cap, dtype=torch.int64, device="cuda") if parent else None
        self.events = torch.zeros(cap, dtype=torch.int32, device="cuda") if events else None
        self.tau = torch.full((cap,), -1.0, dtype=torch.float64, device="cuda") if tau else None
        self.birth = torch.zeros(cap, dtype=torch.float64, device="cuda") if birth else None

    def fill(self, gen, n, momenta, id0, box=1.0e4):
        self.pos[:, :n] = (_uniform(gen, 3, n) * 2.0 - 1.0) * box
        self.mom[:3, :n] = momenta.to(self.real)
        self.mom[3, :n] = 1.0
        self.id[:n] = torch.arange(id0, id0 + n, device="cuda")
        if self.tau is not None:   # depths left over from the step before
            self.tau[:n] = -torch.log1p(-_uniform(gen, n))
        self.n.fill_(n)


class SlotField:
    """One field value per particle slot."""

    def __init__(self, t):
        self.t = t

    def struct(self):
        f = qed.qed_field()
        for k, v in zip(("ex", "ey", "ez", "bx", "by", "bz"), self.t):
            setattr(f, k, v.data_ptr())
        f.stride = 1
        return f


def _uniform(gen, *shape):
    return torch.rand(*shape, generator=gen, device="cuda", dtype=torch.float64)


def _isotropic(gen, n):
    c, p = _uniform(gen, n) * 2.0 - 1.0, _uniform(gen, n) * (2.0 * math.pi)
    s = torch.sqrt(1.0 - c * c)
    return torch.stack((s * torch.cos(p), s * torch.sin(p), c))


def _momenta(gen, n, lo, hi, photons=False):
    energy = 10.0 ** (lo + (hi - lo) * _uniform(gen, n))
    return _isotropic(gen, n) * (energy if photons else torch.sqrt(energy * energy - 1.0))


def _laser_momenta(gen, n, photons=False, e0=1.0e-3):
    """chi log-uniform in [1e-3, 1e2], energy log-uniform in [max(10, 1e3 chi), 1e5], at the
    angle to the field that gives this chi."""
    chi = 10.0 ** (-3.0 + 5.0 * _uniform(gen, n))
    lo = torch.log10(torch.clamp(1.0e3 * chi, min=10.0))
    energy = 10.0 ** (lo + (5.0 - lo) * _uniform(gen, n))
    s = torch.clamp(chi / (e0 * energy), 0.0, 1.0)
    c = torch.sqrt(1.0 - s * s) * torch.where(_uniform(gen, n) < 0.5, -1.0, 1.0)
    p = 2.0 * math.pi * _uniform(gen, n)
    u = energy if photons else torch.sqrt(torch.clamp(energy * energy - 1.0, min=0.0))
    return torch.stack((c, s * torch.cos(p), s * torch.sin(p))) * u


def _uniform_field(real, ex=0.0, ey=0.0, bz=0.0):
    z = np.zeros(1)
    return qed.FieldBuffers({"ex": np.array([ex]), "ey": np.array([ey]), "ez": z, "bx": z, "by": z,
                             "bz": np.array([bz])}, real)


def _recorded_tuning(g, key):
    """The launch shapes recorded for this card and workload."""
    with open(os.path.join(ROOT, "paper_2008_10468_amd", "tuning_gfx950.json")) as f:
        setting = json.load(f)[key]["tuning"]
    t = qed.qed_get_tuning(g.ctx)
    for k, v in setting.items():
        setattr(t, k, int(v))
    if qed.qed_set_tuning(g.ctx, t) != qed.QED_OK:
        raise RuntimeError("tuning refused")


def _network(g):
    m = np.load(os.path.join(ROOT, "paper_2008_10468_amd", "models", "sampler_gfx950.npz"))
    if qed.qed_sampler_set(g.ctx, m["params"], m["fallback"], float(m["log10_chi_lo"]),
                           float(m["log10_chi_hi"])) != qed.QED_OK:
        raise RuntimeError("network refused")


SCHED = {"naive": qed.QED_SCHED_NAIVE, "binned": qed.QED_SCHED_BINNED, "tiled": qed.QED_SCHED_TILED}
TUNING = {("laser", "rejection"): "c2", ("laser", "learned"): "c2s", ("spot", "rejection"): "c3",
          ("spot", "learned"): "c5", ("spot", "fitted"): "c5r", ("weak", "learned"): "w5", ("weak", "fitted"): "w5r"}


def _prepare_step(case, gen):
    pop, n, steps = case["population"], case["n"], case["steps"]
    pairs = pop in ("laser", "shower")
    depth = case["sampler"] != "rejection"
    prec = qed.QED_PREC_F64 if case["precision"] == "f64" else qed.QED_PREC_MIXED
    kind = qed.QED_SAMPLER_SURROGATE if depth else qed.QED_SAMPLER_REJECTION
    g = qed.Generator(precision=prec, capacity=(1, 1, 1), pairs=pairs, scheduler=SCHED[case["scheduler"]],
                      sampler=kind, pair_sampler=kind if pairs else qed.QED_SAMPLER_REJECTION,
                      cascade_generations=5 if pop == "shower" else 0)
    whole = n <= 1 << 21      # the photons are returned too
    n0 = {"laser": (n, 0, n // 4), "shower": (n, n, n)}.get(pop, (n, 0, 0))
    photons, made = (int(n * q * (steps if k == 0 or pop != "shower" else 1)) for k, q in enumerate(GROWTH[pop]))
    made += 4096 if pairs else 0
    cap = (n0[0] + made, n0[1] + made + 16, n0[2] + photons + 4096)
    g.sp = [Buffers(cap[s], g.real, whole, whole, (depth and s < 2) or (depth and pairs), pop == "shower")
            for s in range(3)]
    if pop == "laser":
        g.sp[0].fill(gen, n, _laser_momenta(gen, n), 0)
        g.sp[2].fill(gen, n0[2], _laser_momenta(gen, n0[2], photons=True), n)
    elif pop == "shower":
        for s in range(3):
            g.sp[s].fill(gen, n, _momenta(gen, n, 4.0, 5.5, photons=s == 2), s * n)
    else:
        g.sp[0].fill(gen, n, _momenta(gen, n, 2.0 if pop == "ring" else 3.0, 4.0), 0)
    if pop == "laser":    # the field turns once in 200 steps; one frozen field per step
        turn = [2.0 * math.pi * s / 200.0 for s in range(steps)]
        held = [[_uniform_field(g.real, ex=1.0e-3 * math.cos(a), ey=1.0e-3 * math.sin(a))] * 3 for a in turn]
    elif pop == "spot":
        hot = _uniform(gen, n) < 0.1
        r2 = torch.zeros(n, dtype=torch.float64, device="cuda")
        for _ in range(3):
            r2 += torch.randn(n, generator=gen, device="cuda", dtype=torch.float64) ** 2
        f = torch.zeros(6, n, dtype=g.real, device="cuda")
        f[5] = torch.where(hot, 1.0e-2 * torch.exp(-0.5 * r2), 5.0e-7).to(g.real)
        none = _uniform_field(g.real)
        held = [[SlotField(f), none, none]] * steps
    else:
        held = [[_uniform_field(g.real, bz={"ring": 1.0e-3, "weak": 1.0e-6, "shower": 2.0e-3}[pop])] * 3] * steps
    key = "%s/%s" % (TUNING.get((pop, case["sampler"])), case["scheduler"])
    if key in ("c2/naive", "c2/tiled", "c2s/naive", "c3/binned", "c5/binned", "c5r/binned", "w5/binned", "w5r/binned"):
        _recorded_tuning(g, key)
    if case["sampler"] == "learned":
        _network(g)
    return _kept(g, n0, whole, held, POPULATION[pop]["dt"], steps)


def _kept(g, n0, whole, held, dt, steps):
    """What the program keeps: its copy of the step's start, the argument structures."""
    full = g.sp[2]
    start = {"u": [g.sp[s].mom[:3, :n0[s]].clone() for s in range(2)],
             "photons": [(t[..., :n0[2]], t[..., :n0[2]].clone())
                         for t in (full.mom, full.pos, full.id, full.parent, full.tau) if t is not None and n0[2]],
             "n": [torch.full_like(g.sp[s].n, n0[s]) for s in range(3)]}
    slots = [torch.arange(n0[s] if s < 2 else 0, g.sp[s].capacity, device="cuda") for s in range(3)] if whole else None
    return {"g": g, "n0": n0, "start": start, "slots": slots, "held": held, "dt": dt, "steps": steps, "step": 0,
            "particles": g.particles(), "fields": [[f.struct() for f in h] for h in held]}


def _prepare_pic(case, gen):
    n, m, prec = case["n"], case["cells"], qed.QED_PREC_F64 if case["precision"] == "f64" else qed.QED_PREC_MIXED
    g = qed.Generator(precision=prec, capacity=(1, 1, 1))
    n0 = (n, n // 3, n // 3)
    cap = (n0[0] + n // 2 + 4096, n0[1] + n // 2 + 4096, n0[2] + int(1.0 * n * case["steps"]) + 4096)
    g.sp = [Buffers(c, g.real, True, True, False, False) for c in cap]
    held = []
    id0 = 0
    for s in range(3):
        g.sp[s].fill(gen, n0[s], _momenta(gen, n0[s], 1.0, 3.5, photons=s == 2), id0)
        id0 += n0[s]
        held.append(SlotField(torch.zeros(6, g.sp[s].capacity, dtype=g.real, device="cuda")))
    # smooth fields of a few modes, about 1e-3 of the Schwinger field
    d = 2.0e4 / m
    at = torch.arange(m, device="cuda", dtype=torch.float64) * (2.0 * math.pi / m)
    z, y, x = torch.meshgrid(at, at, at, indexing="ij")
    f = torch.zeros(6, m, m, m, dtype=torch.float64, device="cuda")
    for c in range(6):
        for k in range(4):
            a, q = _uniform(gen, 4).tolist(), [(k + c) % 3, (k * c + 1) % 3, (k + 2 * c) % 2]
            f[c] += 10.0 ** (a[0] - 3.5) * (2.0 * a[1] - 1.0) * torch.cos(q[0] * x + q[1] * y + q[2] * z + 7.0 * a[2])
    geom = {"nx": m, "ny": m, "nz": m, "x0": -1.0e4, "y0": -1.0e4, "z0": -1.0e4, "dx": d, "dy": d, "dz": d}
    state = _kept(g, n0, True, [held], 3.0e4, case["steps"])
    state.update(f=f.to(g.real), j=torch.zeros(3, m, m, m, dtype=torch.float64, device="cuda"))
    state["x"] = [g.sp[s].pos[:, :n0[s]].clone() for s in range(2)]
    state["grid"] = _grid(geom, state["f"])
    state["sp"] = [g.sp[s].struct() for s in range(3)]
    state["out"] = [[t.data_ptr() for t in h.t] for h in held]
    return state


def _grid(geom, f):
    grid = qed.cell_geometry(geom)
    for k, t in zip(("ex", "ey", "ez", "bx", "by", "bz"), f):
        setattr(grid, k, t.data_ptr())
    return grid


def _geometry(case):
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    return {"nx": nx, "ny": ny, "nz": nz, "x0": -1.0e4, "y0": -9.0e3, "z0": -1.1e4,
            "dx": 2.0e4 / nx, "dy": 1.8e4 / ny, "dz": 2.1e4 / nz}


def _prepare_grid(case, gen):
    n, geom = case["n"], _geometry(case)
    g = qed.Generator(precision=qed.QED_PREC_F64 if case["precision"] == "f64" else qed.QED_PREC_MIXED,
                      capacity=(1, 1, 1))
    g.sp[0] = sp = Buffers(n, g.real, False, False, False, False)
    sp.fill(gen, n, _momenta(gen, n, 0.01, 3.0), 0, box=1.15e4)   # some beyond the box: periodic
    sp.mom[3, :n] = (0.5 + _uniform(gen, n)).to(g.real)
    if case["order"] == "cell":
        axis = [torch.remainder(torch.floor((p[:n] - geom[o]) / geom[d]), geom[m]).long()
                for p, o, d, m in zip(sp.pos, ("x0", "y0", "z0"), ("dx", "dy", "dz"), ("nx", "ny", "nz"))]
        at = torch.argsort((axis[2] * geom["ny"] + axis[1]) * geom["nx"] + axis[0], stable=True)
        sp.pos[:, :n] = sp.pos[:, :n][:, at]
        sp.mom[:, :n] = sp.mom[:, :n][:, at]
    shape = (geom["nz"], geom["ny"], geom["nx"])
    state = {"g": g, "n": n, "sp": sp, "struct": sp.struct()}
    if case["path"] == "gather":
        state["f"] = torch.randn(6, *shape, generator=gen, device="cuda", dtype=torch.float64).mul_(1e-3).to(g.real)
        state["e"] = torch.zeros(6, sp.capacity, dtype=g.real, device="cuda")
        state["out"] = [t.data_ptr() for t in state["e"]]
        state["grid"] = _grid(geom, state["f"])
    else:
        state["j"] = torch.zeros(3, *shape, dtype=torch.float64, device="cuda")
        state["grid"] = qed.cell_geometry(geom)
    return state


def _synchrotron_x(case, gen):
    x = 10.0 ** (-4.0 + (math.log10(50.0) + 4.0) * _uniform(gen, case["n"]))
    return x if case["precision"] == "f64" else x.float()


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    path = case["path"]
    if path == "step":
        state = _prepare_step(case, gen)
    elif path == "pic":
        state = _prepare_pic(case, gen)
    elif path in ("gather", "deposit"):
        state = _prepare_grid(case, gen)
    else:
        state = {"g": qed.Generator(capacity=(1, 1, 1))}
        if path == "synchrotron":
            state["x"] = _synchrotron_x(case, gen)
            state["F"], state["G"] = torch.empty_like(state["x"]), torch.empty_like(state["x"])
        else:
            cfg = state["cfg"] = qed.qed_train_config_default()
            cfg.steps, cfg.target, cfg.seed = case["steps"], case["target"], int(seed)
            if case["target"] == 1:
                cfg.log10_chi_lo, cfg.log10_chi_hi, cfg.tolerance = -1.5, 2.5, 2e-3
    state["path"] = path
    return state


# ---------------------------------------------------------------- one pass

def _ok(status):
    if status != qed.QED_OK:
        raise RuntimeError("status %d" % status)


def _back(state):
    """The step's start from the program's own copy."""
    g, n0, start = state["g"], state["n0"], state["start"]
    for s in range(2):
        if n0[s]:
            g.sp[s].mom[:3, :n0[s]].copy_(start["u"][s])
    for t, kept in start["photons"]:
        t.copy_(kept)
    for s in range(3):
        g.sp[s].n.copy_(start["n"][s])


def _by_id(sp, lo, slots):
    """The live particles from slot lo on, sorted by id; the rest of the table is empty."""
    key, order = torch.sort(torch.where(slots < sp.n, sp.id[lo:], LAST))
    live = key != LAST
    out = {"id": key, "mom": torch.where(live, sp.mom[:, lo:][:, order], 0.0),
           "pos": torch.where(live, sp.pos[:, lo:][:, order], 0.0)}
    if sp.parent is not None:
        out["parent"] = torch.where(live, sp.parent[lo:][order], 0)
    if sp.tau is not None:
        out["tau"] = torch.where(live, sp.tau[lo:][order], 0.0)
    return out


def _population(state):
    g, n0 = state["g"], state["n0"]
    out = {"n": [g.sp[s].n for s in range(3)]}
    for s, name in enumerate(("electrons", "positrons")):
        if n0[s]:
            sp = g.sp[s]
            out[name] = {"u": sp.mom[:3, :n0[s]], "pos": sp.pos[:, :n0[s]],
                         "events": None if sp.events is None else sp.events[:n0[s]],
                         "tau": None if sp.tau is None else sp.tau[:n0[s]]}
    if state["slots"] is not None:
        for s, name in enumerate(("new_electrons", "new_positrons", "photons")):
            if state["slots"][s].numel() > 64 or s == 2:
                out[name] = _by_id(g.sp[s], n0[s] if s < 2 else 0, state["slots"][s])
    return out


def run(state):
    path = state["path"]
    if path == "step":
        _back(state)
        g = state["g"]
        for k in range(state["steps"]):
            _ok(qed.qed_step(g.ctx, state["particles"], state["fields"][k], state["dt"], 1, state["step"]))
            state["step"] += 1
        return _population(state)
    if path == "pic":
        _back(state)
        g, j = state["g"], state["j"]
        for s in range(2):
            g.sp[s].pos[:, :state["n0"][s]].copy_(state["x"][s])
        for _ in range(state["steps"]):
            for s in range(3):
                _ok(qed.qed_gather(g.ctx, state["grid"], state["sp"][s], state["out"][s]))
            _ok(qed.qed_step(g.ctx, state["particles"], state["fields"][0], state["dt"], 1, state["step"]))
            state["step"] += 1
            j.zero_()
            for s in range(2):
                _ok(qed.qed_deposit(g.ctx, state["grid"], state["sp"][s], -1.0 if s == 0 else 1.0,
                                    *[c.data_ptr() for c in j]))
        return {"j": j, **_population(state)}
    if path == "gather":
        _ok(qed.qed_gather(state["g"].ctx, state["grid"], state["struct"], state["out"]))
        return state["e"][:, :state["n"]]
    if path == "deposit":
        state["j"].zero_()
        _ok(qed.qed_deposit(state["g"].ctx, state["grid"], state["struct"], -1.0,
                            *[c.data_ptr() for c in state["j"]]))
        return state["j"]
    if path == "synchrotron":
        return qed.synchrotron(state["g"].ctx, state["x"], state["F"], state["G"])
    params, loss, err, fallback = qed.qed_train_sampler(state["g"].ctx, state["cfg"])
    return {"params": params, "loss": loss, "bin_error": err, "fallback": fallback}


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    path = case["path"]
    real = 8 if case.get("precision") == "f64" else 4
    if path == "step":
        p, n, steps = POPULATION[case["population"]], case["n"], case["steps"]
        depth = case["sampler"] != "rejection"
        leptons = n * (2 if case["population"] == "shower" else 1)
        lep = 6 * real + 48 + 8 + (16 if depth else 0) + (24 if case["population"] == "spot" else 0)
        photon = {"laser": n // 4, "shower": n}.get(case["population"], 0)
        born = p["emissions"] * leptons * (24 + 4 * real + 8)
        flops = leptons * (p["sub_depth" if depth else "sub"] * p["flops"] + p["emissions"] * 168)
        return {"bytes": steps * (leptons * lep + photon * (3 * real + 48 + 1) + born), "flops": steps * flops}
    if path == "pic":
        n, cells = case["n"] * 5 // 3, case["cells"] ** 3
        per = 24 + 6 * real + 6 * real + 48 + 6 * real + 8 + 24 + 4 * real
        return {"bytes": case["steps"] * (n * per + cells * (6 * real + 24)), "flops": case["steps"] * n * 900}
    if path in ("gather", "deposit"):
        n, cells = case["n"], case["nx"] * case["ny"] * case["nz"]
        if path == "gather":
            return {"bytes": n * (24 + 6 * real) + cells * 6 * real, "flops": n * 6 * 8 * 5}
        return {"bytes": n * (24 + 4 * real) + cells * 3 * 16, "flops": n * 3 * 8 * 4}
    if path == "synchrotron":
        return {"bytes": 3 * real * case["n"], "flops": 45 * case["n"]}
    # 65,536 samples a step: forward, both backward products, three split products forward
    return {"bytes": case["steps"] * 65536 * 16 + 1025 * 8193 * 8, "flops": case["steps"] * 65536 * 2.0 * 8576 * 3}


# ---------------------------------------------------------------- in 64 bits

STAGGER = ((0.5, 0.0, 0.0), (0.0, 0.5, 0.0), (0.0, 0.0, 0.5), (0.0, 0.5, 0.5), (0.5, 0.0, 0.5), (0.5, 0.5, 0.0))


def _corners(geom, pos, shift):
    """The eight lattice points around each position and their weights."""
    lower, frac = [], []
    for p, o, d, m, h in zip(pos, ("x0", "y0", "z0"), ("dx", "dy", "dz"), ("nx", "ny", "nz"), shift):
        s = (p - geom[o]) / geom[d] - h
        f = torch.floor(s)
        lower.append(torch.remainder(f, geom[m]).long())
        frac.append(s - f)
    for q in range(8):
        w, at = 1.0, []
        for a, m in enumerate(("nx", "ny", "nz")):
            up = (q >> a) & 1
            w = w * (frac[a] if up else 1.0 - frac[a])
            at.append(torch.remainder(lower[a] + up, geom[m]))
        yield (at[2] * geom["ny"] + at[1]) * geom["nx"] + at[0], w


def _synchrotron_64(x):
    """F and G from K_nu(x) = int_0^inf exp(-x cosh t) cosh(nu t) dt by the trapezoid rule
    (which converges faster than any power here)."""
    F, G = torch.zeros_like(x), torch.zeros_like(x)
    h, k = 0.1, 0
    top = math.acosh(745.0 / float(x.min())) + 1.0
    while k * h < top:
        t, w = k * h, (0.5 if k == 0 else 1.0) * h
        e = torch.exp(-x * math.cosh(t))
        F.add_(e, alpha=w * math.cosh(5.0 * t / 3.0) / math.cosh(t))
        G.add_(e, alpha=w * math.cosh(2.0 * t / 3.0))
        k += 1
    return F * x, G * x


def exact(case, seed):
    path = case["path"]
    if path not in ("gather", "deposit", "synchrotron"):
        return None    # drawn events and trained weights: no closed form
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    if path == "synchrotron":
        x = _synchrotron_x(case, gen).double()
        parts = [_synchrotron_64(c) for c in x.split(1 << 23)]
        return tuple(torch.cat(p) for p in zip(*parts))
    state, geom, n = _prepare_grid(case, gen), _geometry(case), case["n"]
    pos = state["sp"].pos[:, :n]
    if path == "gather":
        f = state["f"].double().reshape(6, -1)
        return torch.stack([sum(w * f[c][at] for at, w in _corners(geom, pos, STAGGER[c])) for c in range(6)])
    u = state["sp"].mom[:3, :n].double()
    cur = -state["sp"].mom[3, :n].double() / torch.sqrt(1.0 + (u * u).sum(0)) / (geom["dx"] * geom["dy"] * geom["dz"])
    j = torch.zeros(3, geom["nx"] * geom["ny"] * geom["nz"], dtype=torch.float64, device="cuda")
    for c in range(3):
        for at, w in _corners(geom, pos, STAGGER[c]):
            j[c].index_add_(0, at, w * cur * u[c])
    return j.reshape(state["j"].shape)
