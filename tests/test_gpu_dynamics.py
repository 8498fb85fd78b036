"""Device-side sphere integration (Sec. 2.2.2: velocity Verlet of eqs. 15-16,
and explicit Euler) coupled to the fused step, against the oracle's step and
integrator run in the same order, through the C ABI. FP64 tolerances as in
the parity tests: PDFs 1e-12 relative, forces to the force-scale bound,
positions and velocities 1e-12."""
import numpy as np
import pytest

import oracle
import paper_2303_11811_amd as psm
from paper_2303_11811_amd import inputs
from psm_cases import assert_forces_close, assert_pdfs_close, initial_f, make_engine, oracle_box

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", [psm.PSM_VERLET, psm.PSM_EULER])
def test_coupled_motion_matches_oracle(scheme):
    """Spheres that move across tile boundaries, with body force, rotation,
    a density ratio and an external acceleration; the tile lists are rebuilt
    on the device after every update."""
    spec = inputs.random_small((44, 36, 30), 5, (2.5, 4.0), seed=21, tau=0.65, fext=(1e-5, 0.0, -4e-6),
                               vamp=0.1, omamp=0.004)
    rho_p, accel, dt, steps = 1.7, (0.0, 2e-4, -3e-4), 1.0, 16
    print(f"[case] dynamics scheme={scheme} n={len(spec.r)}", flush=True)
    box = oracle_box(spec)
    f = initial_f(spec)
    dyn = oracle.Dynamics(spec.x, spec.r, spec.U, spec.Om)
    for _ in range(steps):
        ref = oracle.run(box, f, 1, dyn.x, dyn.r, dyn.U, dyn.Om)
        f = ref.f
        oracle.integrate(box, dyn, ref.F, ref.T, dt=dt, scheme=scheme, rho_p=rho_p, accel=accel)

    eng = make_engine([spec])
    eng.set_launch(16, 16, 1, 0)
    eng.set_pdfs(0, initial_f(spec))
    eng.set_particles(0, spec.x, spec.r, spec.U, spec.Om)
    eng.set_dynamics(0, rho_p, accel)
    for _ in range(steps):
        eng.step(1)
        eng.integrate(dt, scheme)
    F, T = eng.get_forces(0)
    x, U, Om = eng.get_particles(0)
    fg = eng.get_pdfs(0).cpu().numpy()
    eng.close()
    assert_pdfs_close(fg, f, 1e-12)
    assert_forces_close(F, ref.F, ref.A)
    assert_forces_close(T, ref.T, ref.A, lever=spec.r.max() + 1)
    # the spheres really moved: their bounding boxes (hence tile lists with
    # one cell per tile along z) changed
    rr = (spec.r + 1.0)[:, None]
    assert np.any(np.floor(dyn.x - rr) != np.floor(spec.x - rr))
    assert np.allclose(x, dyn.x, rtol=1e-12, atol=1e-12)
    assert np.allclose(U, dyn.U, rtol=1e-12, atol=1e-15)
    assert np.allclose(Om, dyn.Om, rtol=1e-12, atol=1e-15)


def test_get_particles_returns_the_set_state():
    spec = inputs.random_small((40, 40, 40), 6, (2.0, 3.0), seed=5)
    eng = make_engine([spec])
    x = spec.x.copy()
    x[0] += 40.0   # wrapped on upload
    eng.set_particles(0, x, spec.r, spec.U, spec.Om)
    xg, Ug, Omg = eng.get_particles(0)
    eng.close()
    assert np.allclose(xg, spec.x, rtol=0, atol=1e-12)
    assert np.array_equal(Ug, spec.U)
    assert np.array_equal(Omg, spec.Om)


def test_tile_overflow_after_integration_is_reported():
    """Seventy unit spheres that one Euler update gathers at one point: the
    device-built list of that tile is capped (the step stays in bounds), the
    next synchronising call reports PSM_ECAPACITY, the context refuses to
    step, and a new particle set makes it usable again."""
    n = 48
    g = np.array([(i, j, k) for i in range(5) for j in range(5) for k in range(3)], dtype=float)[:70]
    x0 = 4.0 + g * np.array([9.0, 9.0, 14.0])
    r = np.full(70, 1.0)
    centre = np.array([24.3, 24.7, 24.1])
    U = centre - x0                     # dt = 1 Euler: every sphere lands on the centre
    spec = inputs.BoxSpec(dims=(n, n, n), tau=0.7, fext=(0.0, 0.0, 0.0), mapping=psm.PSM_MAP_LINEAR, nsub=4,
                          x=x0, r=r, U=np.zeros((70, 3)), Om=np.zeros((70, 3)))
    print("[case] overflow after integration", flush=True)
    eng = make_engine([spec], max_radius=1.0)
    eng.set_launch(32, 8, 4, 0)
    u0 = np.zeros((3, spec.N))
    eng.set_equilibrium(0, u0)
    eng.set_particles(0, x0, r, U)       # velocities only used by the integrator here
    eng.step(1)
    eng.integrate(1.0, psm.PSM_EULER)
    eng.step(1)                          # capped lists: runs, results not valid
    with pytest.raises(psm.PsmError) as ei:
        eng.get_forces(0)
    assert ei.value.code == psm.PSM_ECAPACITY
    with pytest.raises(psm.PsmError) as ei:
        eng.step(1)
    assert ei.value.code == psm.PSM_ESTATE
    eng.set_particles(0, x0, r, np.zeros((70, 3)))
    eng.set_equilibrium(0, u0)
    eng.step(2)
    F, _ = eng.get_forces(0)
    eng.close()
    assert np.all(np.isfinite(F))


def test_force_readback_follows_graph_replays():
    """With the force read-back on, psm_get_forces after psm_step and after
    psm_run (graph replays of step + update pairs, and eager ones) returns
    the forces of the last step, as without it, bit for bit."""
    spec = inputs.random_small((40, 36, 28), 4, (2.5, 4.0), seed=31, tau=0.7, fext=(1e-5, 0.0, -4e-6),
                               vamp=0.05, omamp=0.002)
    print("[case] force read-back after graph replays", flush=True)
    out = []
    for readback in (False, True):
        eng = make_engine([spec])
        eng.set_force_readback(readback)
        eng.set_graph(True)
        eng.set_pdfs(0, initial_f(spec))
        eng.set_particles(0, spec.x, spec.r, spec.U, spec.Om)
        eng.set_dynamics(0, 2.0)
        res = []
        eng.step(1)
        res.append(eng.get_forces(0))
        eng.run(10, 1.0, psm.PSM_EULER)      # one graph replay
        res.append(eng.get_forces(0))
        eng.run(3, 1.0, psm.PSM_EULER)       # eager steps
        res.append(eng.get_forces(0))
        eng.step(10)                         # graph replay of plain steps
        res.append(eng.get_forces(0))
        eng.close()
        out.append(res)
    for (Fa, Ta), (Fb, Tb) in zip(*out):
        assert np.array_equal(Fa, Fb) and np.array_equal(Ta, Tb)
    assert not np.array_equal(out[1][0][0], out[1][1][0])


@pytest.mark.parametrize("how", ["run", "graph", "upload", "readback", "unused"])
def test_tile_overflow_that_passes_is_reported(how):
    """Seventy unit spheres that meet at one point for one step and part again
    before the host looks: the step ran on a cut list, so the next synchronising
    call reports PSM_ECAPACITY although the lists hold every sphere by then.
    Lists that were replaced before any step ran on them are not reported."""
    print(f"[case] passing overflow {how}", flush=True)
    n = 48
    g = np.array([(i, j, k) for i in range(5) for j in range(5) for k in range(3)], dtype=float)[:70]
    x0 = 4.0 + g * np.array([9.0, 9.0, 14.0])
    r = np.full(70, 1.0)
    centre = np.array([24.3, 24.7, 24.1])
    dt = 1000.0
    U = (centre - x0) / dt               # one Euler update to the centre, the next away from it
    eng = psm.Engine([psm.make_desc(n, n, n, 0.7, max_particles=70, max_radius=1.0)])
    eng.set_launch(32, 8, 4, 0)
    eng.set_dynamics(0, 1e12)            # the fluid does not turn the spheres
    eng.set_equilibrium(0, np.zeros((3, n ** 3)))
    eng.set_particles(0, x0, r, U)
    if how in ("run", "graph"):
        eng.set_graph(how == "graph")
        eng.run(2 if how == "run" else 10, dt, psm.PSM_EULER)
    else:
        eng.set_force_readback(how == "readback")
        eng.step(1)
        eng.set_particle_positions(0, np.tile(centre, (70, 1)))
        if how != "unused":
            eng.step(1)
        eng.set_particle_positions(0, x0)
        eng.step(1)
    if how == "unused":
        F, _ = eng.get_forces(0)
        assert np.all(np.isfinite(F))
    else:
        with pytest.raises(psm.PsmError) as ei:
            eng.get_forces(0)
        assert ei.value.code == psm.PSM_ECAPACITY
        with pytest.raises(psm.PsmError) as ei:
            eng.step(1)
        assert ei.value.code == psm.PSM_ESTATE
        eng.set_particles(0, x0, r, U)
        eng.set_equilibrium(0, np.zeros((3, n ** 3)))
        eng.step(1)
        assert np.all(np.isfinite(eng.get_forces(0)[0]))
    eng.close()


@pytest.mark.parametrize("readback", [False, True])
def test_tile_overflow_after_host_upload_is_reported(readback):
    """The same gathering uploaded by the host right after a step: without the
    force read-back the force read of that step reports PSM_ECAPACITY; with
    it, that read returns the step's forces (the copy was taken before the
    re-binning) and the read after the next step, which ran on the cut lists,
    reports it. The context then refuses to step until a new particle set."""
    n = 48
    g = np.array([(i, j, k) for i in range(5) for j in range(5) for k in range(3)], dtype=float)[:70]
    x0 = 4.0 + g * np.array([9.0, 9.0, 14.0])
    r = np.full(70, 1.0)
    xg = np.tile(np.array([24.3, 24.7, 24.1]), (70, 1))
    spec = inputs.BoxSpec(dims=(n, n, n), tau=0.7, fext=(1e-5, 0.0, 0.0), mapping=psm.PSM_MAP_LINEAR, nsub=4,
                          x=x0, r=r, U=np.zeros((70, 3)), Om=np.zeros((70, 3)))
    print(f"[case] overflow after host upload readback={readback}", flush=True)
    u0 = np.zeros((3, spec.N))
    ref = make_engine([spec], max_radius=1.0)
    ref.set_launch(32, 8, 4, 0)
    ref.set_equilibrium(0, u0)
    ref.set_particles(0, x0, r, np.zeros((70, 3)))
    ref.step(1)
    F_ref, T_ref = ref.get_forces(0)
    ref.close()
    eng = make_engine([spec], max_radius=1.0)
    eng.set_force_readback(readback)
    eng.set_launch(32, 8, 4, 0)
    eng.set_equilibrium(0, u0)
    eng.set_particles(0, x0, r, np.zeros((70, 3)))
    eng.step(1)
    eng.set_particle_positions(0, xg)
    if readback:
        F, T = eng.get_forces(0)
        assert np.array_equal(F, F_ref) and np.array_equal(T, T_ref)
        eng.step(1)                      # cut lists: runs, results not valid
    with pytest.raises(psm.PsmError) as ei:
        eng.get_forces(0)
    assert ei.value.code == psm.PSM_ECAPACITY
    with pytest.raises(psm.PsmError) as ei:
        eng.step(1)
    assert ei.value.code == psm.PSM_ESTATE
    eng.set_particles(0, x0, r, np.zeros((70, 3)))
    eng.set_equilibrium(0, u0)
    eng.step(1)
    F, T = eng.get_forces(0)
    eng.close()
    assert np.array_equal(F, F_ref) and np.array_equal(T, T_ref)


def test_spheres_bounce_off_walls_like_the_oracle():
    """Spheres driven into the side walls and the z faces of a closed box
    (velocity inflow, pressure outflow) bounce elastically one cell before
    them, in the same step as in the oracle; the coupled run matches."""
    from test_gpu_walls import _bed

    spec = _bed((30, 26, 28), 4, seed=77)
    # aim every sphere at a wall, close enough to reach it within the run
    spec.x[:, 0] = spec.r + 1.3
    spec.U = np.array([[-0.12, 0.05, 0.0], [-0.1, -0.08, 0.03], [-0.15, 0.0, -0.09], [-0.11, 0.07, 0.1]])
    rho_p, accel, dt, steps = 1.3, (0.0, 0.0, -1e-4), 1.0, 10
    print(f"[case] wall contact n={len(spec.r)}", flush=True)
    box = oracle_box(spec)
    f = initial_f(spec)
    dyn = oracle.Dynamics(spec.x, spec.r, spec.U, spec.Om)
    for _ in range(steps):
        ref = oracle.run(box, f, 1, dyn.x, dyn.r, dyn.U, dyn.Om)
        f = ref.f
        oracle.integrate(box, dyn, ref.F, ref.T, dt=dt, scheme=psm.PSM_VERLET, rho_p=rho_p, accel=accel)
    assert np.any(dyn.U[:, 0] > 0)   # at least one sphere bounced off x = 0
    eng = make_engine([spec])
    eng.set_launch(32, 8, 4, 0)
    eng.set_pdfs(0, initial_f(spec))
    eng.set_particles(0, spec.x, spec.r, spec.U, spec.Om)
    eng.set_dynamics(0, rho_p, accel)
    for _ in range(steps):
        eng.step(1)
        eng.integrate(dt, psm.PSM_VERLET)
    x, U, Om = eng.get_particles(0)
    fg = eng.get_pdfs(0).cpu().numpy()
    eng.close()
    assert_pdfs_close(fg, f, 1e-12)
    assert np.allclose(x, dyn.x, rtol=1e-12, atol=1e-12)
    assert np.allclose(U, dyn.U, rtol=1e-12, atol=1e-15)


def test_run_replays_graphs_bitwise():
    """psm_run with graphs (10 step + update pairs per replay, recaptured for a
    new time step) equals the eager step/integrate loop bit for bit after
    every chunk, with synchronising reads between the replays."""
    spec = inputs.random_small((40, 34, 30), 6, (2.5, 4.0), seed=33, tau=0.7, fext=(1e-5, 0, 0),
                               vamp=0.08, omamp=0.003)
    chunks = [(10, 1.0), (13, 1.0), (10, 0.5), (10, 0.5), (10, 1.0)]
    engines = []
    for graph in (False, True):
        eng = make_engine([spec])
        eng.set_pdfs(0, initial_f(spec))
        eng.set_particles(0, spec.x, spec.r, spec.U, spec.Om)
        eng.set_dynamics(0, 1.4, (0.0, -1e-4, 0.0))
        eng.set_graph(graph)
        engines.append(eng)
    for n, dt in chunks:
        eager, graphed = engines
        for _ in range(n):
            eager.step(1)
            eager.integrate(dt, psm.PSM_VERLET)
        graphed.run(n, dt, psm.PSM_VERLET)
        a = (*eager.get_particles(0), *eager.get_forces(0), eager.get_pdfs(0).cpu().numpy())
        b = (*graphed.get_particles(0), *graphed.get_forces(0), graphed.get_pdfs(0).cpu().numpy())
        for u, v in zip(a, b):
            assert np.array_equal(u, v), (n, dt)
    for eng in engines:
        eng.close()


def test_host_coupling_with_split_updates_matches_oracle():
    """The host-driven explicit Euler loop of the moving suspension with the
    split updates: the next positions are uploaded right after the step is
    enqueued (ordered after it on the stream, so the step and its force
    reduction see the old ones), the new velocities after the force
    read-back. Matches the oracle's step + integrator sequence, and the same
    loop with one full psm_set_particles per step bit for bit; so does the
    split loop with the force read-back at the end of each step (forces read
    while the re-binning of the next positions may still run)."""
    spec = inputs.random_small((44, 36, 30), 5, (2.5, 4.0), seed=23, tau=0.65, fext=(1e-5, 0.0, -4e-6),
                               vamp=0.1, omamp=0.004)
    steps = 8
    box = oracle_box(spec)
    f = initial_f(spec)
    dyn = oracle.Dynamics(spec.x, spec.r, spec.U, spec.Om)
    for _ in range(steps):
        ref = oracle.run(box, f, 1, dyn.x, dyn.r, dyn.U, dyn.Om)
        f = ref.f
        oracle.integrate(box, dyn, ref.F, ref.T, dt=1.0, scheme=oracle.EULER, rho_p=1.0)
    m = 4.0 / 3.0 * np.pi * spec.r ** 3
    inv_m, inv_I = (1.0 / m)[:, None], (1.0 / (0.4 * m * spec.r ** 2))[:, None]
    L = np.asarray(spec.dims, dtype=np.float64)
    results = []
    for split, readback in ((True, False), (False, False), (True, True)):
        eng = make_engine([spec])
        eng.set_force_readback(readback)
        eng.set_pdfs(0, initial_f(spec))
        x, U, Om = spec.x.copy(), spec.U.copy(), spec.Om.copy()
        eng.set_particles(0, x, spec.r, U, Om)
        Fb, Tb = np.empty_like(x), np.empty_like(x)
        for _ in range(steps):
            eng.step(1)
            xn = np.mod(x + U, L)
            if split:
                eng.set_particle_positions(0, xn)
                # the caller's arrays, filled in place
                F, T = eng.get_forces(0, Fb, Tb)
                assert F is Fb and T is Tb
                F, T = F.copy(), T.copy()
            else:
                F, T = eng.get_forces(0)
            U = U + F * inv_m
            Om = Om + T * inv_I
            if split:
                eng.set_particle_velocities(0, U, Om)
            else:
                eng.set_particles(0, xn, spec.r, U, Om)
            x = xn
        results.append((eng.get_pdfs(0).cpu().numpy(), F, T, x, U, Om))
        with pytest.raises(psm.PsmError) as e:
            eng.set_particle_velocities(0, U[:-1], Om[:-1])
        assert e.value.code == psm.PSM_EINVAL
        eng.close()
    (fs, Fs, Ts, xs, Us, Oms), (ff, Ff, Tf, *_), (fr, Fr, Tr, *_) = results
    assert np.array_equal(fs, ff) and np.array_equal(Fs, Ff) and np.array_equal(Ts, Tf)
    assert np.array_equal(fs, fr) and np.array_equal(Fs, Fr) and np.array_equal(Ts, Tr)
    assert_pdfs_close(fs, f, 1e-12)
    assert_forces_close(Fs, ref.F, ref.A)
    assert_forces_close(Ts, ref.T, ref.A, lever=spec.r.max() + 1)
    assert np.allclose(xs, dyn.x, rtol=1e-12, atol=1e-12)
    assert np.allclose(Us, dyn.U, rtol=1e-12, atol=1e-15)


@pytest.mark.parametrize("nspheres", [1, 7, 9])
def test_lists_after_launch_changes_between_updates(nspheres):
    """Launches with few and with many tiles in turn, an odd number of list
    builds between them: every launch starts from clean counts, so the run is
    bit for bit the one of a context that keeps the launch (PDFs in FP64 do
    not depend on the tile shape)."""
    spec = inputs.random_small((40, 34, 30), nspheres, (2.5, 3.0), seed=37, tau=0.7, vamp=0.08, omamp=0.003)
    print(f"[case] launch changes n={len(spec.r)}", flush=True)
    f = []
    for launches in ([(16, 16, 1, 0)] * 4, [(16, 16, 1, 0), (256, 1, 32, 0), (32, 8, 4, 0), (16, 16, 1, 0)]):
        eng = make_engine([spec])
        eng.set_pdfs(0, initial_f(spec))
        eng.set_particles(0, spec.x, spec.r, spec.U, spec.Om)
        for launch in launches:
            eng.set_launch(*launch)
            eng.step(1)
            eng.set_particle_positions(0, spec.x + 0.3 * spec.U)
            eng.set_particle_positions(0, spec.x)
            eng.set_particles(0, spec.x + 2.0 * spec.U, spec.r, spec.U, spec.Om)
            eng.step(2)
        f.append(eng.get_pdfs(0).cpu().numpy())
        eng.close()
    assert np.array_equal(f[0], f[1])


def _motions(eng, x, r, U, cells, rng):
    """Steps, uploads and device updates of spheres far from the edges of the
    box: everything the force reduction and the tile lists give."""
    out = []
    eng.set_particles(0, x, r, U, np.zeros_like(U))
    eng.step(3)
    out += [*eng.get_forces(0), eng.get_pdfs_at(0, cells).cpu().numpy()]
    eng.set_particle_positions(0, x + rng.uniform(-1.0, 1.0, x.shape))
    eng.set_force_readback(True)
    eng.step(2)
    out += [*eng.get_forces(0)]
    eng.set_force_readback(False)
    eng.set_graph(True)
    eng.run(10, 1.0, psm.PSM_VERLET)
    eng.set_graph(False)
    eng.run(1, 1.0, psm.PSM_EULER)
    eng.integrate(1.0, psm.PSM_EULER)
    eng.step(1)
    return out + [*eng.get_forces(0), *eng.get_particles(0), eng.get_pdfs_at(0, cells).cpu().numpy(),
                  np.array(eng.get_stats(0)[2])]


def _cloud(n, lo, hi, r, seed):
    rng = np.random.default_rng(seed)
    x = rng.uniform(lo, hi, (n, 3))
    return x, np.full(n, r), inputs.uniform_velocities(rng, n, 0.01)


@pytest.mark.parametrize("storage", [psm.PSM_FP64, psm.PSM_FP16DEV])
@pytest.mark.parametrize("launch", [(64, 4, 8, 0), (256, 1, 1, 0), (16, 16, 16, psm.PSM_LAUNCH_PERSISTENT)])
def test_one_set_of_partials_keeps_the_results(launch, storage):
    """A context with room for so many spheres that its partials have one set
    (its workspace is too small for two) gives bit for bit what one with room
    for the spheres gives."""
    print(f"[case] one set of partials {launch} storage={storage}", flush=True)
    x, r, U = _cloud(40, 20.0, 44.0, 1.5, 5)
    cells = np.random.default_rng(6).integers(0, 64 ** 3, 500)
    got = []
    for room in (40, 200000):
        eng = psm.Engine([psm.make_desc(64, 64, 64, 0.7, max_particles=room, max_radius=1.5)], storage=storage)
        eng.set_launch(*launch)
        eng.set_equilibrium(0, np.zeros((3, 64 ** 3)))
        got.append(_motions(eng, x, r, U, cells, np.random.default_rng(7)))
        eng.close()
    assert all(np.array_equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("n", [40, 300])
def test_compact_lists_of_a_huge_context_keep_the_results(n):
    """A context beyond 64 GiB lists its spheres back to back (its workspace
    has no room for lists of a fixed capacity): forces, motion, PDFs and the
    count of dropped overlaps are bit for bit those of a 96^3 box, whose edges
    the motion does not reach, and a crowded tile is reported."""
    print(f"[case] compact lists n={n}", flush=True)
    import torch

    x, r, U = _cloud(n, 32.0, 64.0, 1.0, 8)
    at = np.random.default_rng(9).integers(0, 96, (500, 3))
    got = []
    for d in ((96, 96, 96), (1024, 1024, 900)):
        N = int(np.prod(d))
        desc = psm.make_desc(*d, 0.7, max_particles=n, max_radius=1.0)
        if N > 96 ** 3:
            fixed = 76 * N + 8 * (N // 256) * min(64, n)
            assert psm.psm_workspace_size([desc], psm.PSM_FP16DEV) < fixed
        eng = psm.Engine([desc], storage=psm.PSM_FP16DEV)
        eng.set_launch(64, 4, 1, 0)
        u = torch.zeros((3, N), dtype=torch.float64, device=eng.device)
        eng.set_equilibrium(0, u)
        del u
        got.append(_motions(eng, x, r, U, at @ [1, d[0], d[0] * d[1]], np.random.default_rng(10)))
        if n > 64:
            eng.set_particles(0, x * 0.0 + 40.0, r, U)
            with pytest.raises(psm.PsmError) as e:
                eng.get_forces(0)
            assert e.value.code == psm.PSM_ECAPACITY
        eng.close()
    torch.cuda.empty_cache()
    assert all(np.array_equal(a, b) for a, b in zip(*got))
