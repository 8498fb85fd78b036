"""Work that programs give the engine, as cases that can be timed and compared.

A case is a dict of plain values. ``prepare`` builds what a program holds
before the call (the engine with its spheres, launch and initial state, made
from the seed alone), ``run`` is one pass through the public entry points,
``work`` the bytes and operations that pass cannot do without, and ``exact``
the same results from a plain FP64 PyTorch implementation of the method
(eqs. 1-8 and 17-27 of arXiv 2303.11811) that shares no code with the engine.

Kinds of pass:

* ``steps``    advance fixed spheres by ``steps`` steps (HIP graphs on), then read
               the forces and the macroscopic fields (and the PDFs if ``pdfs``)
* ``upload``   every step uploads the sphere table, steps and reads the forces (the
               benchmark's main loop); then the macroscopic fields
* ``coupled``  host-integrated spheres: step, upload positions, read forces, upload
               velocities, ``steps`` times; then the macroscopic fields
* ``device``   the spheres are integrated on the GPU (``psm_run``), ``steps`` steps
               between two outputs of spheres, forces and fields
* ``batched``  many independent boxes in one context
* ``save``     write a checkpoint (canonical PDFs and their totals), load it back
* ``look``     set the initial state, read fractions, totals and fields
"""
import math

import numpy as np
import torch

import paper_2303_11811_amd as psm
from paper_2303_11811_amd import inputs

STORAGE = {"f64": psm.PSM_FP64, "f32": psm.PSM_FP32DEV, "f16": psm.PSM_FP16DEV}
VALUE_BYTES = {"f64": 8, "f32": 4, "f16": 2}
# launches that the benchmark times each storage form at
LAUNCH = {"f64": "128,2,1,0", "f32": "128,2,2,0", "f16": "64,4,8,0"}


def _case(name, kind, dims, storage, steps, spheres, radius, launch="", **more):
    c = dict(name=name, kind=kind, nx=dims[0], ny=dims[1], nz=dims[2], storage=storage, steps=steps,
             spheres=spheres, radius=radius, launch=launch, tau=0.6, g=0.0, nsub=0, bed=False, pdfs=False,
             boxes=0, mix=0)
    c.update(more)
    return c


def listed():
    return [
        # the smallest box anyone runs (validation, parameter studies): launches and latency count
        _case("steps_f64_32", "steps", (32, 32, 32), "f64", 100, 8, 4.0, nsub=4, pdfs=True),
        # the same box with the host in the loop: every step is a round trip
        _case("coupled_f64_32", "coupled", (32, 32, 32), "f64", 10, 8, 4.0),
        # the precision study's box in its FP32 form, engine defaults
        _case("steps_f32_64", "steps", (64, 64, 64), "f32", 50, 6, 10.0, tau=0.55, g=1e-6),
        # an odd, ragged box in the FP16 form, engine defaults
        _case("steps_f16_121x90x75", "steps", (121, 90, 75), "f16", 20, 24, 7.0, tau=0.7, g=1e-5),
        # the quick-start program: autotuned 128^3 with host-integrated spheres
        _case("coupled_f64_128", "coupled", (128, 128, 128), "f64", 10, 50, 10.0, launch="auto", tau=0.55, g=1e-6),
        # a sweep over many small uneven boxes in one context
        _case("batched_f32_24", "batched", (0, 0, 0), "f32", 50, 30, 8.0, launch="64,4,2,0", boxes=24, mix=3),
        # a dense suspension integrated on the GPU
        _case("device_f32_256", "device", (256, 256, 256), "f32", 20, 2347, 8.0, launch="64,4,8,0"),
        # a large box in the cheapest storage
        _case("steps_f16_384", "steps", (384, 384, 384), "f16", 20, 1352, 10.0, launch=LAUNCH["f16"], tau=0.55, g=1e-6),
        # the paper's fluidized bed: side walls, inflow, outflow, spheres moving on the GPU
        _case("bed_f64_500x200x800", "device", (500, 200, 800), "f64", 10, 627, 10.0, launch="128,2,8,0", tau=0.65,
              bed=True),
        # the paper-scale box with the sphere table uploaded every step: the largest
        _case("upload_f64_512", "upload", (512, 512, 512), "f64", 10, 3204, 10.0, launch=LAUNCH["f64"], tau=0.55,
              g=1e-6),
        # checkpoint and restart of a mid-sized run
        _case("save_f64_192", "save", (192, 192, 192), "f64", 0, 169, 10.0),
        # start of a run: initial state in, first picture and totals out
        _case("look_f32_256", "look", (256, 256, 256), "f32", 0, 401, 10.0),
    ]


def draw(rng):
    kind = rng.choice(["steps", "steps", "steps", "coupled", "coupled", "upload", "device", "device", "batched",
                       "save", "look"])
    storage = rng.choice(["f64", "f32", "f16"])
    tau = round(rng.uniform(0.55, 1.0), 4)
    if kind == "batched":
        return _drawn("batched", (0, 0, 0), storage, rng.choice([10, 20, 50]), 30, 8.0,
                      rng.choice(["", "64,4,2,0"]), boxes=rng.randrange(4, 25), mix=rng.randrange(1000))
    bed = kind == "device" and rng.random() < 0.4
    radius = rng.choice([4.0, 5.5, 8.0, 10.0])
    least = int(2 * (radius + 1)) + 6
    edge = math.exp(rng.uniform(math.log(32), math.log(220)))
    dims = tuple(max(least, int(edge * rng.uniform(0.75, 1.3))) for _ in range(3))
    cells = dims[0] * dims[1] * dims[2]
    fraction = rng.choice([0.03, 0.10, 0.10, 0.28])
    spheres = max(1, min(int(fraction * cells / (4.2 * radius ** 3)), _lattice_most(dims, radius)))
    steps = {"steps": rng.choice([10, 20, 50]), "device": rng.choice([10, 20])}.get(kind, rng.choice([5, 10]))
    launches = ["", LAUNCH[storage]]
    if storage == "f64" and cells < 1 << 22:
        launches.append("auto")
    return _drawn(kind, dims, storage, 0 if kind in ("save", "look") else steps, spheres, radius,
                  rng.choice(launches), tau=tau, g=0.0 if bed else rng.choice([0.0, 1e-6, 1e-5]),
                  nsub=rng.choice([0, 0, 0, 4]), bed=bed, pdfs=cells < 1 << 20 and rng.random() < 0.5)


def _drawn(*args, **more):
    c = _case("", *args, **more)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# Inputs

def _lattice_most(dims, radius):
    return int(np.prod([int((d - 2) // (2 * radius)) for d in dims]))


def _spheres(dims, n, radius, rng, amp, bed):
    """Non-overlapping spheres (inside walls with a gap of one cell for a bed)."""
    lo = 1.0 if bed else 0.0
    inner = np.asarray(dims, dtype=np.float64) - 2.0 * lo
    solid = n * 4.0 / 3.0 * math.pi * radius ** 3 / float(np.prod(dims))
    if bed or solid > 0.15:   # random addition jams there
        x, r = inputs.jittered_lattice_spheres(tuple(inner), n, radius, rng)
        x = x + lo
    elif n > 64:
        x, r = inputs.rsa_spheres(dims, np.full(n, radius), rng)
    else:
        x, r = inputs.rsa_spheres(dims, rng.uniform(0.8, 1.0, n) * radius, rng)
    U = inputs.uniform_velocities(rng, len(r), 0.0 if bed else amp)
    return x, r, U, inputs.uniform_velocities(rng, len(r), 0.0 if bed else 0.2 * amp)


def _specs(case, seed):
    rng = np.random.default_rng((seed, 1))
    if case["kind"] != "batched":
        dims = (case["nx"], case["ny"], case["nz"])
        spec = inputs.BoxSpec(dims=dims, tau=case["tau"], fext=(case["g"], 0.0, 0.0), mapping=int(case["nsub"] > 0),
                              nsub=max(case["nsub"], 1))
        spec.x, spec.r, spec.U, spec.Om = _spheres(dims, case["spheres"], case["radius"], rng, 0.005, case["bed"])
        if case["bed"]:
            nu = (spec.tau - 0.5) / 3.0
            spec.walls_x = spec.walls_y = spec.walls_z = True
            spec.wall_u = ((0.0, 0.0, nu / (2.0 * case["radius"])), (0.0, 0.0, 0.0))
            spec.face_type, spec.face_rho = (psm.PSM_FACE_VELOCITY, psm.PSM_FACE_PRESSURE), (1.0, 1.0)
        return [spec]
    shapes = np.random.default_rng(case["mix"])   # edges, tau and sphere counts belong to the case
    specs = []
    for _ in range(case["boxes"]):
        edge = int(shapes.choice([32, 48, 64, 96, 128]))
        spec = inputs.BoxSpec(dims=(edge,) * 3, tau=float(shapes.uniform(0.55, 1.0)))
        # at most 12 % solid, so that every sphere finds a place whatever the seed
        n = min(int(shapes.integers(0, case["spheres"] + 1)), int(0.12 * edge ** 3 / (4.2 * case["radius"] ** 3)))
        spec.x, spec.r = inputs.rsa_spheres(spec.dims, rng.uniform(3.0, case["radius"], n), rng)
        spec.U = inputs.uniform_velocities(rng, len(spec.r), 0.01)
        spec.Om = inputs.uniform_velocities(rng, len(spec.r), 0.002)
        specs.append(spec)
    return specs


def _initial(spec, seed, k, device):
    """Density and velocity of a moving fluid: a mean stream, three vortices and noise."""
    gen = torch.Generator(device="cpu").manual_seed(seed * 131 + k)
    nx, ny, nz = spec.dims
    ph = torch.rand(6, generator=gen, dtype=torch.float64).tolist()
    grid = [2 * math.pi * (torch.arange(n, dtype=torch.float64, device=device) + 0.5) / n for n in (nx, ny, nz)]
    X, Y, Z = grid[0].view(1, 1, -1), grid[1].view(1, -1, 1), grid[2].view(-1, 1, 1)
    s = [2 * math.pi * p for p in ph]
    amp, mean = (1e-4, (0.0, 0.0, spec.wall_u[0][2])) if spec.walls_z else (0.01, (0.004, 0.003, 0.002))
    gen = torch.Generator(device=device).manual_seed(seed * 131 + k)
    u = (torch.rand((3, nz, ny, nx), generator=gen, dtype=torch.float64, device=device) - 0.5) * (0.2 * amp)
    u[0] += mean[0] + amp * torch.sin(X + s[0]) * torch.cos(Y + s[1])
    u[1] += mean[1] + amp * torch.sin(Y + s[2]) * torch.cos(Z + s[3])
    u[2] += mean[2] + amp * torch.sin(Z + s[4]) * torch.cos(X + s[5])
    rho = 1.0 + (torch.rand(spec.N, generator=gen, dtype=torch.float64, device=device) - 0.5) * 1e-3
    return rho, u.reshape(3, -1)


def _dynamics(case):
    """Density ratio and external acceleration of the moving spheres."""
    if not case["bed"]:
        return 2.5, (0.0, 0.0, 0.0)
    nu, d, ratio = (case["tau"] - 0.5) / 3.0, 2.0 * case["radius"], 1.1
    g = (8.9 * nu) ** 2 / ((ratio - 1.0) * d ** 3)
    return ratio, (0.0, 0.0, -g * (1.0 - 1.0 / ratio))


def prepare(case, seed):
    specs = _specs(case, seed)
    batched = case["kind"] == "batched"
    descs = [psm.desc_from_spec(s, max_particles=max(len(s.r), 1), max_radius=case["radius"]) for s in specs]
    eng = psm.Engine(descs, storage=STORAGE[case["storage"]])
    start = [_initial(s, seed, k, eng.device) for k, s in enumerate(specs)]
    for b, s in enumerate(specs):
        eng.set_particles(b, s.x, s.r, s.U, s.Om)
        eng.set_equilibrium(b, start[b][1], start[b][0])
        eng.synchronize()
    if case["launch"] == "auto":
        eng.autotune(trial_steps=3)
        eng.set_equilibrium(0, start[0][1], start[0][0])
    elif case["launch"]:
        eng.set_launch(*(int(v) for v in case["launch"].split(",")))
    eng.synchronize()
    state = {"case": dict(case), "eng": eng, "specs": specs}
    spec = specs[0]
    if case["kind"] in ("steps", "device", "batched"):
        eng.set_graph(True)
    if case["kind"] == "device":
        eng.set_dynamics(0, *_dynamics(case))
    if case["kind"] == "coupled":
        eng.set_force_readback(True)
        m = 2.5 * 4.0 / 3.0 * np.pi * spec.r[:, None] ** 3
        state.update(x=spec.x.copy(), U=spec.U.copy(), Om=spec.Om.copy(), F=np.empty_like(spec.x),
                     T=np.empty_like(spec.x), m=m, inertia=0.4 * m * spec.r[:, None] ** 2,
                     L=np.asarray(spec.dims, dtype=np.float64))
    if case["kind"] == "look":
        state.update(rho0=start[0][0], u0=start[0][1])
    if batched:
        state["with_spheres"] = [b for b, s in enumerate(specs) if len(s.r)]
    return state


def run(state):
    return _RUN[state["case"]["kind"]](state, state["eng"], state["case"])


def _fields(eng, box=0):
    rho, u = eng.get_macroscopic(box)
    return {"rho": rho, "u": u}


def _run_steps(state, eng, case):
    eng.step(case["steps"])
    F, T = eng.get_forces(0)
    out = {"F": F, "T": T, **_fields(eng)}
    if case["pdfs"]:
        out["f"] = eng.get_pdfs(0)
    return out


def _run_upload(state, eng, case):
    s = state["specs"][0]
    for _ in range(case["steps"]):
        eng.set_particles(0, s.x, s.r, s.U, s.Om)
        eng.step(1)
        F, T = eng.get_forces(0)
    return {"F": F, "T": T, **_fields(eng)}


def _run_coupled(state, eng, case):
    x, U, Om, F, T = (state[k] for k in ("x", "U", "Om", "F", "T"))
    for _ in range(case["steps"]):
        eng.step(1)
        np.mod(x + U, state["L"], out=x)
        eng.set_particle_positions(0, x)
        eng.get_forces(0, F, T)
        U += F / state["m"]
        Om += T / state["inertia"]
        eng.set_particle_velocities(0, U, Om)
    return {"x": x, "U": U, "Om": Om, "F": F, "T": T, **_fields(eng)}


def _run_device(state, eng, case):
    eng.run(case["steps"], dt=1.0, scheme=psm.PSM_VERLET if case["bed"] else psm.PSM_EULER)
    x, U, Om = eng.get_particles(0)
    F, T = eng.get_forces(0)
    return {"x": x, "U": U, "Om": Om, "F": F, "T": T, **_fields(eng)}


def _run_batched(state, eng, case):
    eng.step(case["steps"])
    forces = [eng.get_forces(b) for b in state["with_spheres"]]
    fields = [eng.get_macroscopic(b) for b in range(case["boxes"])]
    return {"F": np.concatenate([f for f, _ in forces] or [np.zeros((0, 3))]),
            "T": np.concatenate([t for _, t in forces] or [np.zeros((0, 3))]),
            "rho": [r for r, _ in fields], "u": [u for _, u in fields]}


def _run_save(state, eng, case):
    f = eng.get_pdfs(0)
    totals = torch.empty(4, dtype=torch.float64, device=f.device)
    psm.psm_field_stats_noalloc(f.data_ptr(), f.shape[1], totals.data_ptr(),
                                torch.cuda.current_stream(f.device).cuda_stream)
    eng.set_pdfs(0, f)
    return {"f": f, "totals": totals, **_fields(eng)}


def _run_look(state, eng, case):
    s = state["specs"][0]
    eng.set_particles(0, s.x, s.r, s.U, s.Om)
    eng.set_equilibrium(0, state["u0"], state["rho0"])
    B, pid = eng.get_solid_fraction(0)
    mass, momentum, dropped = eng.get_stats(0)
    return {"B": B, "pid": pid, "mass": mass, "momentum": momentum, "dropped": dropped, **_fields(eng)}


_RUN = {"steps": _run_steps, "upload": _run_upload, "coupled": _run_coupled, "device": _run_device,
        "batched": _run_batched, "save": _run_save, "look": _run_look}


def work(case):
    """Every step reads and writes the 19 stored values of a cell once; a read-out reads them once and writes
    FP64 fields (4 values; the canonical PDFs are 19). Operations: about 300 per cell and step."""
    if case["kind"] == "batched":
        cells = sum(s.N for s in _specs(dict(case, spheres=0), 0))
    else:
        cells = case["nx"] * case["ny"] * case["nz"]
    stored = 19 * VALUE_BYTES[case["storage"]]
    fields = stored + 32
    per_cell = {"save": (stored + 152) + 152 + (152 + stored) + fields,
                "look": (32 + stored) + 24 + stored + fields}.get(case["kind"])
    if per_cell is None:
        per_cell = case["steps"] * 2 * stored + fields + (stored + 152 if case["pdfs"] else 0)
    return {"bytes": cells * per_cell, "flops": cells * (300 * case["steps"] + 40)}


# ---------------------------------------------------------------------------
# The same in plain FP64 PyTorch

_C = np.array([(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0),
               (-1, -1, 0), (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1), (-1, 0, 1), (0, 1, 1),
               (0, -1, -1), (0, 1, -1), (0, -1, 1)])
_W = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12
_BAR = [0] + [q + 1 if q % 2 else q - 1 for q in range(1, 19)]


def _dot(q, v):
    return sum(int(c) * a for c, a in zip(_C[q], v) if c) if q else 0.0 * v[0]


class _Fluid:
    """One box in FP64: canonical PDFs f [19][N] and the step of the method."""

    def __init__(self, spec, rho, u):
        self.s, self.dev = spec, rho.device
        base = rho - 1.5 * (u * u).sum(0)
        self.f = torch.empty((19, spec.N), dtype=torch.float64, device=self.dev)
        for q in range(19):
            cu = _dot(q, u)
            self.f[q] = _W[q] * (base + cu * (3.0 + 4.5 * cu))

    def moments(self):
        j = [sum(int(_C[q, a]) * self.f[q] for q in range(19) if _C[q, a]) for a in range(3)]
        return self.f.sum(0), j

    def fields(self):
        rho, j = self.moments()
        return {"rho": rho, "u": torch.stack([a + 0.5 * g for a, g in zip(j, self.s.fext)])}

    def fractions(self, x, r):
        """Cells with solid, their two slots (sphere ids, ascending; -1 empty) and fractions."""
        s, dev = self.s, self.dev
        x, r = (torch.as_tensor(v, dtype=torch.float64, device=dev) for v in (x, r))
        if len(r) == 0:
            z = torch.zeros((2, 0), dtype=torch.int64, device=dev)
            return z[0], z, z.double()
        m = int(math.ceil(float(r.max()))) + 2
        o = torch.arange(-m, m + 1, device=dev)
        off = torch.stack(torch.meshgrid(o, o, o, indexing="ij"), -1).reshape(-1, 3)
        rr = r * r
        root = torch.sqrt(rr - 0.5)
        Va = (1 / 12 - rr) * torch.atan(0.5 * root / (0.5 - rr)) + root / 3 + (rr - 1 / 12) * torch.atan(0.5 / root) \
            - 4 / 3 * r * rr * torch.atan(0.25 / (r * root))
        fr = Va - r + 0.5
        dims = torch.tensor(s.dims, device=dev)
        got = []
        for p0 in range(0, len(r), 256):
            cell = torch.floor(x[p0:p0 + 256]).long()[:, None, :] + off[None]
            d = cell + 0.5 - x[p0:p0 + 256, None, :]
            R, FR = r[p0:p0 + 256, None], fr[p0:p0 + 256, None]
            if s.mapping == 0:
                B = (FR - (torch.sqrt((d * d).sum(-1)) - R)).clamp(max=1.0)
            else:
                near = (d * d).sum(-1) < (R + 1.0) ** 2
                dn, Rn = d[near], R.expand(near.shape)[near]
                inside = torch.zeros(len(Rn), dtype=torch.float64, device=dev)
                t = [(k + 0.5) / s.nsub - 0.5 for k in range(s.nsub)]
                for a in t:
                    for b in t:
                        for c in t:
                            inside += (dn[:, 0] + a) ** 2 + (dn[:, 1] + b) ** 2 + (dn[:, 2] + c) ** 2 <= Rn * Rn
                B = torch.zeros(near.shape, dtype=torch.float64, device=dev)
                B[near] = inside / s.nsub ** 3
            hit = B > 0
            w = torch.remainder(cell[hit], dims)
            pid = torch.arange(p0, p0 + cell.shape[0], device=dev)[:, None].expand(hit.shape)[hit]
            got.append((w[:, 0] + s.dims[0] * (w[:, 1] + s.dims[1] * w[:, 2]), pid, B[hit]))
        n, pid, B = (torch.cat(v) for v in zip(*got))
        order = torch.argsort(B, descending=True, stable=True)
        n, pid, B = n[order], pid[order], B[order]
        order = torch.argsort(n, stable=True)
        n, pid, B = n[order], pid[order], B[order]
        first = torch.ones_like(n, dtype=torch.bool)
        first[1:] = n[1:] != n[:-1]
        at = torch.arange(len(n), device=dev)
        rank = at - torch.cummax(torch.where(first, at, torch.zeros_like(at)), 0)[0]
        cells = n[first]
        slot = torch.full((2, len(cells)), -1, dtype=torch.int64, device=dev)
        frac = torch.zeros((2, len(cells)), dtype=torch.float64, device=dev)
        which = torch.cumsum(first.long(), 0) - 1
        for k in range(2):
            slot[k, which[rank == k]] = pid[rank == k]
            frac[k, which[rank == k]] = B[rank == k]
        swap = (slot[1] >= 0) & (slot[1] < slot[0])
        slot[:, swap], frac[:, swap] = slot[:, swap].flip(0), frac[:, swap].flip(0)
        return cells, slot, frac / frac.sum(0).clamp(min=1.0)

    def step(self, x, r, U, Om, solid=None):
        """One step; returns the force and torque on every sphere."""
        s, f, dev = self.s, self.f, self.dev
        omega, pref = 1.0 / s.tau, 1.0 - 0.5 / s.tau
        g = s.fext
        rho, j = self.moments()
        V = [a + 0.5 * b for a, b in zip(j, g)]
        base = rho - 1.5 * (V[0] ** 2 + V[1] ** 2 + V[2] ** 2)
        Vg = sum(a * b for a, b in zip(V, g))
        cells, slot, frac = self.fractions(x, r) if solid is None else solid
        x, U, Om = (torch.as_tensor(v, dtype=torch.float64, device=dev) for v in (x, U, Om))
        pos = torch.stack([cells % s.dims[0], cells // s.dims[0] % s.dims[1],
                           cells // (s.dims[0] * s.dims[1])], -1) + 0.5
        L = torch.tensor(s.dims, dtype=torch.float64, device=dev)
        fs, rs, js, Vs = f[:, cells], rho[cells], torch.stack([a[cells] for a in j], -1), \
            torch.stack([a[cells] for a in V], -1)
        F, T = torch.zeros_like(x), torch.zeros_like(x)
        Up = []
        for k in range(2):
            p = slot[k].clamp(min=0)
            d = pos - x[p]
            d = d - L * torch.floor(d / L + 0.5)
            up = U[p] + torch.linalg.cross(Om[p], d)
            gk = frac[k][:, None] * (2.0 * js - Vs - up)
            F.index_add_(0, p, gk)
            T.index_add_(0, p, torch.linalg.cross(d, gk))
            Up.append(up)
        Bt = frac.sum(0)
        post = torch.empty_like(f)
        for q in range(19):
            cg = float(np.dot(_C[q], g))
            cu = _dot(q, V)
            E = _W[q] * (base + cu * (3.0 + 4.5 * cu))
            post[q] = f[q] + omega * (E - f[q]) + pref * _W[q] * (3.0 * cg + 9.0 * cg * cu - 3.0 * Vg)
            if len(cells):
                b = _BAR[q]
                new = fs[q] + (1.0 - Bt) * (post[q, cells] - fs[q])
                cb = -cu[cells]
                Eb = _W[q] * (base[cells] + cb * (3.0 + 4.5 * cb))
                for k in range(2):
                    cv = _dot(q, Up[k].T)
                    Ev = _W[q] * (rs + cv * (3.0 + 4.5 * cv) - 1.5 * (Up[k] ** 2).sum(-1))
                    new += frac[k] * (fs[b] - Eb + Ev - fs[q])
                post[q, cells] = new
        self._stream(post)
        return F, T

    def _stream(self, post):
        s = self.s
        nx, ny, nz = s.dims
        p = post.view(19, nz, ny, nx)
        out = self.f.view(19, nz, ny, nx)
        for q in range(19):
            out[q] = torch.roll(p[q], tuple(int(c) for c in _C[q][::-1]), (0, 1, 2))
        if s.walls_z:
            for w, z, inward in ((0, 0, 1), (1, nz - 1, -1)):
                u = [sum(int(_C[q, a]) * p[q, z] for q in range(19) if _C[q, a]) for a in range(3)]
                uu = u[0] ** 2 + u[1] ** 2 + u[2] ** 2
                for q in range(19):
                    if _C[q, 2] != inward:
                        continue
                    if s.face_type[w] == psm.PSM_FACE_VELOCITY:
                        out[q, z] = p[_BAR[q], z] + 6.0 * _W[q] * float(np.dot(_C[q], s.wall_u[w]))
                    else:
                        cu = _dot(q, u)
                        out[q, z] = 2.0 * _W[q] * (s.face_rho[w] + 4.5 * cu * cu - 1.5 * uu) - p[_BAR[q], z]
        for q in range(19):
            if s.walls_y and _C[q, 1]:
                at = 0 if _C[q, 1] > 0 else ny - 1
                out[q, :, at, :] = p[_BAR[q], :, at, :]
            if s.walls_x and _C[q, 0]:
                at = 0 if _C[q, 0] > 0 else nx - 1
                out[q, :, :, at] = p[_BAR[q], :, :, at]


def exact(case, seed):
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    specs = _specs(case, seed)
    if sum(s.N for s in specs) * max(case["steps"], 1) > 1_400_000_000:
        return None
    F, T, fields, fluid = [], [], [], None
    x = U = Om = None
    for k, s in enumerate(specs):
        rho0, u0 = _initial(s, seed, k, dev)
        fluid = _Fluid(s, rho0, u0)
        x, U, Om = (torch.as_tensor(v, dtype=torch.float64, device=dev).clone() for v in (s.x, s.U, s.Om))
        r = torch.as_tensor(s.r, dtype=torch.float64, device=dev)
        moving = case["kind"] in ("coupled", "device")
        solid = None if moving else fluid.fractions(x, r)
        Fk = Tk = torch.zeros_like(x)
        ratio, accel = _dynamics(case)
        m = (ratio * 4.0 / 3.0 * math.pi * r ** 3)[:, None]
        inertia = 0.4 * m * (r ** 2)[:, None]
        L = torch.tensor(s.dims, dtype=torch.float64, device=dev)
        before = None
        for _ in range(case["steps"]):
            Fk, Tk = fluid.step(x, r, U, Om, solid)
            if not moving:
                continue
            Ft = Fk + m * torch.tensor(accel, dtype=torch.float64, device=dev)
            if case["bed"]:
                if before is not None:
                    U = U + (before[0] + Ft) / (2.0 * m)
                    Om = Om + (before[1] + Tk) / (2.0 * inertia)
                before = (Ft, Tk)
                x = x + U + Ft / (2.0 * m)
                lo, hi = (r + 1.0)[:, None], L - (r + 1.0)[:, None]
                U = torch.where((x < lo) | (x > hi), -U, U)
                x = torch.where(x < lo, 2.0 * lo - x, torch.where(x > hi, 2.0 * hi - x, x))
            else:
                x = torch.remainder(x + U, L)
                U, Om = U + Ft / m, Om + Tk / inertia
        F.append(Fk)
        T.append(Tk)
        if case["kind"] not in ("save", "look"):
            fields.append(fluid.fields())
    out = {"F": torch.cat(F), "T": torch.cat(T)}
    if case["kind"] == "batched":
        return {**out, "rho": [v["rho"] for v in fields], "u": [v["u"] for v in fields]}
    if case["kind"] in ("save", "look"):
        look = fluid.fields()
        f = fluid.f
        totals = torch.stack([f.sum()] + [sum(int(_C[q, a]) * f[q].sum() for q in range(19) if _C[q, a])
                                          for a in range(3)])
        if case["kind"] == "save":
            return {"f": f, "totals": totals, **look}
        cells, _, frac = fluid.fractions(x, r)
        B = torch.zeros((2, specs[0].N), dtype=torch.float64, device=dev)
        B[:, cells] = frac
        return {"B": B, "pid": None, "mass": float(totals[0]), "momentum": totals[1:].cpu().numpy(), "dropped": None,
                **look}
    out.update(fields[0])
    if case["kind"] in ("coupled", "device"):
        out.update(x=x, U=U, Om=Om)
    if case["pdfs"]:
        out["f"] = fluid.f
    return out
