"""Deviation storage forms against the FP64 oracle.

FP32 stores d = f - w_q, FP16 stores 2^10 d; both collide in FP32 and keep
forces, torques and mass sums in FP64. Their error against the oracle is a
property of the rounding, not a parity bar; the bounds asserted here are the
stated error bounds of these forms (about three times the measured values).

Velocity error: L2 of u over all cells relative to the L2 of the oracle's u.
Force error: max over spheres of |dF_p| / max(|F_p|, 0.01 A_p), A_p the sum
over the sphere's cells of B |g| (the magnitude of the terms of eq. 21): a
sphere whose force nearly cancels is measured against 1 % of its terms.

(a) The precision copy of the 512^3 workload: 64^3 periodic box, tau 0.55,
body force 1e-6 along +x, fluid at rest, 6 spheres of radius 10 (10 % solid,
seed 1) with velocities in [-0.005, 0.005]^3, linear mapping, 1000 steps:
  FP32-dev: L2 velocity error <= 5e-5, force error <= 4e-4
  FP16-dev: L2 velocity error <= 6e-4, force error <= 7e-3
(b) 100 steps of a 32^3 Taylor-Green box with 4 spheres (r = 4, tau 0.6):
  FP32-dev: L2 velocity error <= 2e-5, force error <= 1e-4
  FP16-dev: L2 velocity error <= 3e-3, force error <= 2e-2
"""
import os
import time

import numpy as np
import pytest

import oracle
import paper_2303_11811_amd as psm
from paper_2303_11811_amd import inputs
from psm_cases import CX, CY, CZ, W, initial_f, make_engine, run_oracle

pytestmark = pytest.mark.gpu

BOUNDS = {psm.PSM_FP32DEV: (2e-5, 1e-4), psm.PSM_FP16DEV: (3e-3, 2e-2)}
BOUNDS_COPY = {psm.PSM_FP32DEV: (5e-5, 4e-4), psm.PSM_FP16DEV: (6e-4, 7e-3)}


def force_error(F, F_ref, A):
    """max_p |dF_p| / max(|F_p|, 0.01 A_p)."""
    d = np.linalg.norm(F - F_ref, axis=1)
    return float(np.max(d / np.maximum(np.linalg.norm(F_ref, axis=1), 0.01 * A)))


@pytest.fixture(scope="module")
def copy_reference():
    """The oracle on the 64^3 precision copy, 1000 steps. It runs the OpenMP
    timing build of the oracle (the same arithmetic per cell; only the order
    of the force sums over cells differs, far below these bounds)."""
    spec = inputs.paper_scale(n=64, seed=1)
    box = oracle.Box(*spec.dims, tau=spec.tau, fext=spec.fext)
    f0 = oracle.equilibrium(box, np.zeros((3, spec.N)))
    oracle.threads(min(16, os.cpu_count() or 1))
    print(f"[precision copy] oracle 64^3 x 1000 steps, {len(spec.r)} spheres ...", flush=True)
    t0 = time.perf_counter()
    ref = oracle.run(box, f0, 1000, spec.x, spec.r, spec.U, spec.Om, timing_build=True)
    print(f"[precision copy] oracle done in {time.perf_counter() - t0:.1f} s", flush=True)
    _, u_ref = oracle.macroscopic(box, ref.f)
    return spec, u_ref, ref


@pytest.mark.parametrize("storage", [psm.PSM_FP32DEV, psm.PSM_FP16DEV])
def test_precision_copy_of_the_paper_scale_workload(storage, copy_reference):
    spec, u_ref, ref = copy_reference
    eng = make_engine([spec], storage=storage)
    eng.set_equilibrium(0, np.zeros((3, spec.N)))
    eng.set_particles(0, spec.x, spec.r, spec.U, spec.Om)
    eng.set_graph(True)
    eng.step(1000)
    _, u = eng.get_macroscopic(0)
    F, _ = eng.get_forces(0)
    eng.close()
    u = u.cpu().numpy()
    l2 = float(np.linalg.norm(u - u_ref) / np.linalg.norm(u_ref))
    fe = force_error(F, ref.F, ref.A)
    print(f"[precision copy] storage {storage}: L2 u {l2:.3e}, force {fe:.3e}", flush=True)
    bu, bf = BOUNDS_COPY[storage]
    assert l2 <= bu and fe <= bf


def _spec():
    rng = np.random.default_rng(17)
    dims = (32, 32, 32)
    x, r = inputs.rsa_spheres(dims, np.full(4, 4.0), rng)
    U = inputs.uniform_velocities(rng, len(r), 0.01)
    return inputs.BoxSpec(dims=dims, tau=0.6, mapping=0, x=x, r=r, U=U, Om=np.zeros_like(U),
                          u0=inputs.taylor_green(dims, 0.01))


@pytest.mark.parametrize("storage", [psm.PSM_FP32DEV, psm.PSM_FP16DEV])
def test_deviation_storage_error_bounds(storage):
    spec = _spec()
    steps = 100
    ref = run_oracle(spec, steps)
    box = oracle.Box(*spec.dims, tau=spec.tau)
    _, u_ref = oracle.macroscopic(box, ref.f)
    eng = make_engine([spec], storage=storage)
    eng.set_pdfs(0, initial_f(spec))
    eng.set_particles(0, spec.x, spec.r, spec.U, spec.Om)
    eng.step(steps)
    _, u = eng.get_macroscopic(0)
    F, T = eng.get_forces(0)
    u = u.cpu().numpy()
    l2 = np.linalg.norm(u - u_ref) / np.linalg.norm(u_ref)
    fe = force_error(F, ref.F, ref.A)
    print(f"[precision] storage {storage}: L2 u {l2:.3e}, force {fe:.3e}", flush=True)
    bu, bf = BOUNDS[storage]
    assert l2 <= bu and fe <= bf
    # FP64 mass bookkeeping of the rounded state stays close to the true mass
    mass, _, _ = eng.get_stats(0)
    assert abs(mass - ref.f.sum()) / ref.f.sum() < (1e-7 if storage == psm.PSM_FP32DEV else 1e-4)


@pytest.mark.parametrize("storage", [psm.PSM_FP32DEV, psm.PSM_FP16DEV])
def test_deviation_storage_roundtrip(storage):
    """set_pdfs -> get_pdfs rounds d = f - w_q once: exact for FP32 where d is
    representable, within one FP16 ulp of 2^10 d otherwise."""
    spec = inputs.random_small((20, 16, 12), 0, (2, 3), seed=4, tau=0.7)
    f0 = initial_f(spec)
    eng = make_engine([spec], storage=storage)
    eng.set_pdfs(0, f0)
    f = eng.get_pdfs(0).cpu().numpy()
    w = oracle.lattice()[1][:, None]
    d0 = f0 - w
    if storage == psm.PSM_FP32DEV:
        assert np.array_equal(f, d0.astype(np.float32).astype(np.float64) + w)
    else:
        ulp = np.abs(d0) * 2.0 ** -10 + 2.0 ** -24 / 1024 + 1e-16
        assert np.all(np.abs(f - f0) <= ulp)


@pytest.mark.parametrize("scale", [2.0 ** 8, 2.0 ** 12])
def test_fp16_scale_choice(scale):
    """Other power-of-two FP16 scales (the scale is folded into the collision
    constants) give the same physics within the FP16 bounds, and the state
    round trip keeps one FP16 rounding of scale * d."""
    spec = _spec()
    steps = 100
    ref = run_oracle(spec, steps)
    box = oracle.Box(*spec.dims, tau=spec.tau)
    _, u_ref = oracle.macroscopic(box, ref.f)
    eng = make_engine([spec], storage=psm.PSM_FP16DEV, fp16_scale=scale)
    f0 = initial_f(spec)
    eng.set_pdfs(0, f0)
    w = oracle.lattice()[1][:, None]
    back = eng.get_pdfs(0).cpu().numpy()
    # store: FP64 -> FP32 -> FP16 of scale * d; read: FP32 product with 1/scale, then + w in FP64
    h = ((f0 - w) * scale).astype(np.float32).astype(np.float16)
    expect = (h.astype(np.float32) * np.float32(1.0 / scale)).astype(np.float64) + w
    assert np.array_equal(back, expect)
    eng.set_particles(0, spec.x, spec.r, spec.U, spec.Om)
    eng.step(steps)
    _, u = eng.get_macroscopic(0)
    F, T = eng.get_forces(0)
    u = u.cpu().numpy()
    l2 = np.linalg.norm(u - u_ref) / np.linalg.norm(u_ref)
    fe = force_error(F, ref.F, ref.A)
    print(f"[precision] FP16 scale {scale:g}: L2 u {l2:.3e}, force {fe:.3e}", flush=True)
    bu, bf = BOUNDS[psm.PSM_FP16DEV]
    assert l2 <= bu and fe <= bf
    eng.close()


@pytest.mark.parametrize("dims", [(63, 14, 10), (64, 12, 9), (70, 9, 8)])
def test_fp16_one_step_every_cell_row_layouts(dims):
    """Every value of an FP16-deviation box after one step from the engine's
    own state agrees with the FP64 oracle's step from that state to the
    one-step bound of psm_cases.deviation_bound. The widths cover the three
    row layouts of the PDF grid: rows padded to whole 64-cell blocks with an
    odd and with an even width, and rows packed back to back (a wave's cells
    then straddle blocks); two tile widths each, with spheres and a body
    force."""
    from psm_cases import deviation_bound

    rng = np.random.default_rng(23)
    x, r = inputs.rsa_spheres(dims, np.array([2.0, 1.5, 1.8]), rng)
    U = inputs.uniform_velocities(rng, len(r), 0.01)
    spec = inputs.BoxSpec(dims=dims, tau=0.6, mapping=0, x=x, r=r, U=U, Om=np.zeros_like(U),
                          u0=inputs.taylor_green(dims, 0.02), fext=(1e-5, 0.0, 0.0))
    box = oracle.Box(*dims, tau=spec.tau, fext=spec.fext)
    for launch in ((64, 4, 4, 0), (32, 8, 2, 0)):
        print(f"[case] fp16 one step dims={dims} launch={launch}", flush=True)
        eng = make_engine([spec], storage=psm.PSM_FP16DEV, max_radius=2.0)
        eng.set_launch(*launch)
        eng.set_pdfs(0, initial_f(spec))
        eng.set_particles(0, spec.x, spec.r, spec.U, spec.Om)
        eng.step(3)
        f_t = eng.get_pdfs(0).cpu().numpy()
        eng.step(1)
        got = eng.get_pdfs(0).cpu().numpy()
        eng.close()
        ref = oracle.run(box, f_t, 1, x, r, U, spec.Om).f
        bound = deviation_bound(ref.T, psm.PSM_FP16DEV).T
        ratio = np.max(np.abs(got - ref) / bound)
        print(f"[ratio] max |err|/bound = {ratio:.3g}", flush=True)
        assert np.all(np.abs(got - ref) <= bound), ratio


IO_DIMS = [(4, 4, 4), (16, 17, 5), (17, 16, 19), (32, 9, 33), (33, 31, 6), (63, 5, 17), (64, 4, 16), (65, 6, 18),
           (121, 7, 21), (130, 10, 34)]


def _stored(values, storage, scale=1024.0):
    """Canonical values f [19][N] after one rounding to the storage form."""
    if storage == psm.PSM_FP64:
        return values
    w = W[:, None]
    if storage == psm.PSM_FP32DEV:
        return (values - w).astype(np.float32).astype(np.float64) + w
    return ((values - w) * scale).astype(np.float16).astype(np.float64) / scale + w


@pytest.mark.parametrize("storage", [psm.PSM_FP64, psm.PSM_FP32DEV, psm.PSM_FP16DEV])
@pytest.mark.parametrize("dims", IO_DIMS)
def test_state_io_rounds_once_and_reads_back(storage, dims):
    """psm_set_pdfs stores every value of every cell rounded once (to nearest
    even; for FP16 also where an FP32 value in between would be a tie), in boxes
    whose rows end anywhere in a tile, and psm_get_pdfs returns the stored
    values bit for bit; density, velocity and totals follow from them."""
    import torch

    print(f"[case] state io storage={storage} dims={dims}", flush=True)
    rng = np.random.default_rng(sum(dims) + storage)
    N = int(np.prod(dims))
    f = W[:, None] + (rng.random((19, N)) - 0.5) * 4e-3
    # an FP16 tie missed by 2^-30 of the scaled value: FP32 cannot hold the difference
    half = rng.integers(0x3000, 0x4400, (19, N)).astype(np.uint16).view(np.float16).astype(np.float64)
    step = np.spacing(half.astype(np.float16)).astype(np.float64)
    tie = (half + 0.5 * step + np.where(rng.random((19, N)) < 0.5, 1, -1) * 2.0 ** -30) / 1024.0
    f = np.where(rng.random((19, N)) < 0.3, W[:, None] + tie, f)
    g = (3e-6, -2e-6, 1e-6)
    eng = psm.Engine([psm.make_desc(*dims, 0.7, fext=g)], storage=storage)
    eng.set_pdfs(0, f)
    got = eng.get_pdfs(0).cpu().numpy()
    rho, u = (a.cpu().numpy() for a in eng.get_macroscopic(0))
    mass, mom, _ = eng.get_stats(0)
    totals = torch.empty(4, dtype=torch.float64, device=eng.device)
    field = torch.as_tensor(got).to(eng.device)
    torch.cuda.synchronize()
    psm.psm_field_stats_noalloc(field.data_ptr(), N, totals.data_ptr(), eng.stream.cuda_stream)
    eng.synchronize()
    eng.close()
    assert np.array_equal(got, _stored(f, storage))
    c = np.stack([CX, CY, CZ])
    # sums of 19 and of 19 N terms of at most 1/3 and 1/18 each, rounded once per addition
    assert np.all(np.abs(rho - got.sum(0)) <= 19 * 2.0 ** -52)
    assert np.all(np.abs(u - (c @ got + 0.5 * np.array(g)[:, None])) <= 19 * 2.0 ** -52)
    ref = np.array([got.sum(), *(c @ got).sum(1)])
    bound = 2.0 ** -52 * 19 * N * np.array([1.0, 0.1, 0.1, 0.1])
    assert np.all(np.abs(np.array([mass, *mom]) - ref) <= bound)
    assert np.all(np.abs(totals.cpu().numpy() - ref) <= bound)


@pytest.mark.parametrize("dims", IO_DIMS)
def test_equilibrium_start_reaches_every_cell(dims):
    """psm_set_equilibrium (FP64) gives E_q(rho, u) of eq. (5) in every cell of
    boxes smaller than, as large as and past its tiles in every axis."""
    import torch

    print(f"[case] equilibrium dims={dims}", flush=True)
    rng = np.random.default_rng(sum(dims))
    N = int(np.prod(dims))
    rho, u = 1.0 + (rng.random(N) - 0.5) * 1e-2, (rng.random((3, N)) - 0.5) * 0.1
    for r in (rho, None):
        eng = psm.Engine([psm.make_desc(*dims, 0.7)])
        eng.set_equilibrium(0, torch.as_tensor(u), None if r is None else torch.as_tensor(r))
        got = eng.get_pdfs(0).cpu().numpy()
        eng.close()
        cu = np.stack([CX, CY, CZ]).T @ u
        ref = W[:, None] * ((1.0 if r is None else r) + 3.0 * cu + 4.5 * cu ** 2 - 1.5 * (u ** 2).sum(0))
        assert np.all(np.abs(got - ref) <= 16 * 2.0 ** -53 * W[:, None])


@pytest.mark.parametrize("storage", [psm.PSM_FP64, psm.PSM_FP32DEV, psm.PSM_FP16DEV])
@pytest.mark.parametrize("walls", ["x", "yz", "xyz"])
@pytest.mark.parametrize("dims", [(4, 4, 4), (66, 9, 6)])
def test_state_io_rounds_once_at_walls(dims, walls, storage):
    """Every value of every cell between resting walls is stored rounded once
    and read back bit for bit, with values near FP16 ties as in periodic boxes
    (those cells are set by kernels of their own)."""
    print(f"[case] state io at walls storage={storage} dims={dims} walls={walls}", flush=True)
    rng = np.random.default_rng(sum(dims) + storage)
    N = int(np.prod(dims))
    half = rng.integers(0x3000, 0x4400, (19, N)).astype(np.uint16).view(np.float16).astype(np.float64)
    step = np.spacing(half.astype(np.float16)).astype(np.float64)
    tie = (half + 0.5 * step + np.where(rng.random((19, N)) < 0.5, 1, -1) * 2.0 ** -30) / 1024.0
    f = W[:, None] + np.where(rng.random((19, N)) < 0.5, tie, (rng.random((19, N)) - 0.5) * 4e-3)
    eng = psm.Engine([psm.make_desc(*dims, 0.7, walls_x="x" in walls, walls_y="y" in walls, walls_z="z" in walls)],
                     storage=storage)
    eng.set_pdfs(0, f)
    got = eng.get_pdfs(0).cpu().numpy()
    eng.close()
    assert np.array_equal(got, _stored(f, storage))


@pytest.mark.parametrize("storage", [psm.PSM_FP64, psm.PSM_FP32DEV, psm.PSM_FP16DEV])
@pytest.mark.parametrize("dims", [(16, 9, 5), (17, 16, 6), (13, 7, 5), (300, 4, 4), (4, 64, 7), (257, 5, 16)])
@pytest.mark.parametrize("offset", [0, 1, 16])
def test_pdfs_into_any_field(offset, dims, storage):
    """psm_get_pdfs into a field that starts at a 128-byte line or not, of a
    length that keeps every direction there or not, over plane ends inside a
    block: every value, and nothing beside it."""
    import torch

    print(f"[case] pdfs into any field offset={offset} dims={dims} storage={storage}", flush=True)
    N = int(np.prod(dims))
    f = W[:, None] + (np.random.default_rng(N).random((19, N)) - 0.5) * 4e-3
    eng = psm.Engine([psm.make_desc(*dims, 0.7)], storage=storage)
    eng.set_pdfs(0, f)
    out = torch.full((19 * N + 64,), -7.0, dtype=torch.float64, device=eng.device)
    assert out.data_ptr() % 128 == 0
    torch.cuda.synchronize()
    psm.psm_get_pdfs(eng.ctx, 0, out.data_ptr() + 8 * offset)
    eng.synchronize()
    eng.close()
    got = out.cpu().numpy()
    assert np.array_equal(got[offset:offset + 19 * N].reshape(19, N), _stored(f, storage))
    assert np.all(got[:offset] == -7.0) and np.all(got[offset + 19 * N:] == -7.0)
