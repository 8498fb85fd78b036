"""Host-side checks of the C ABI that need no GPU: the library loads, exports
every entry point declared in include/psm.h, and rejects bad arguments with
PSM_EINVAL before anything is enqueued."""
import ctypes
import os
import re
import threading
import types

import pytest

import paper_2303_11811_amd as psm

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "psm.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(psm_[a-z_0-9]+)\s*\(", text)))


def test_every_declared_symbol_is_exported():
    names = _declared()
    assert len(names) >= 20
    L = psm.lib()
    for n in names:
        assert hasattr(L, n), n
        assert n in psm._SIGS, f"binding lacks {n}"


def test_workspace_size_scales_with_storage():
    d = [psm.make_desc(64, 48, 40, 0.6, max_particles=10, max_radius=5.0)]
    s64 = psm.psm_workspace_size(d, psm.PSM_FP64)
    s32 = psm.psm_workspace_size(d, psm.PSM_FP32DEV)
    s16 = psm.psm_workspace_size(d, psm.PSM_FP16DEV)
    grid = 2 * 19 * 64 * 48 * 40
    assert s64 - s32 == grid * 4 and s32 - s16 == grid * 2
    assert s64 > grid * 8


@pytest.mark.parametrize("desc,msg", [
    (dict(nx=3, ny=8, nz=8, tau=0.6), "dimension"),
    (dict(nx=8, ny=8, nz=8, tau=0.5), "tau"),
    (dict(nx=8, ny=8, nz=8, tau=float("nan")), "tau"),
    (dict(nx=16, ny=16, nz=16, tau=0.6, max_particles=2, max_radius=0.5), "max_radius"),
    (dict(nx=16, ny=16, nz=16, tau=0.6, max_particles=2, max_radius=7.0), "2*(max_radius+1)+2"),
    (dict(nx=16, ny=16, nz=16, tau=0.6, mapping=7), "mapping"),
    (dict(nx=16, ny=16, nz=16, tau=0.6, mapping=1, subsample_n=0), "subsample_n"),
    (dict(nx=16, ny=16, nz=16, tau=0.6, max_particles=-1), "max_particles"),
])
def test_invalid_descriptors(desc, msg):
    with pytest.raises(psm.PsmError) as e:
        psm.psm_workspace_size([psm.make_desc(**desc)], psm.PSM_FP64)
    assert e.value.code == psm.PSM_EINVAL and msg in str(e.value)


def test_invalid_storage_and_empty():
    with pytest.raises(psm.PsmError):
        psm.psm_workspace_size([psm.make_desc(8, 8, 8, 0.6)], 7)
    out = ctypes.c_size_t(0)
    assert psm.lib().psm_workspace_size(None, 0, 0, ctypes.byref(out)) == psm.PSM_EINVAL


def test_create_rejects_before_touching_the_gpu():
    d = [psm.make_desc(8, 8, 8, 0.6)]
    need = psm.psm_workspace_size(d, psm.PSM_FP64)
    for ws, nbytes, msg in [(0, need, "NULL"), (256 + 8, need, "aligned"), (1 << 20, need - 1, "needs")]:
        with pytest.raises(psm.PsmError) as e:
            psm.psm_create(d, psm.PSM_FP64, 0.0, 0, ws, nbytes)
        assert e.value.code == psm.PSM_EINVAL and msg in str(e.value)
    with pytest.raises(psm.PsmError) as e:
        psm.psm_create(d, psm.PSM_FP16DEV, 3.0, 0, 1 << 20, 1 << 40)
    assert "power of two" in str(e.value)


def test_null_context_calls():
    L = psm.lib()
    assert L.psm_step(None, 1) == psm.PSM_EINVAL
    assert L.psm_destroy(None) == psm.PSM_EINVAL
    assert L.psm_set_graph(None, 1) == psm.PSM_EINVAL
    assert L.psm_get_forces(None, 0, None, None) == psm.PSM_EINVAL
    assert L.psm_integrate(None, 1.0, psm.PSM_VERLET) == psm.PSM_EINVAL
    assert L.psm_run(None, 10, 1.0, psm.PSM_VERLET) == psm.PSM_EINVAL
    assert L.psm_set_dynamics(None, 0, 1.0, None) == psm.PSM_EINVAL
    assert L.psm_get_particles(None, 0, None, None, None) == psm.PSM_EINVAL
    assert L.psm_set_launch(None, 64, 4, 1, 0) == psm.PSM_EINVAL
    assert L.psm_set_drift_check(None, 0, 1e-12) == psm.PSM_EINVAL
    assert L.psm_set_strict_slots(None, 1) == psm.PSM_EINVAL
    assert L.psm_set_force_readback(None, 1) == psm.PSM_EINVAL
    assert "NULL" in psm.psm_last_error() or "ctx" in psm.psm_last_error()


def test_stream_copy_argument_checks():
    L = psm.lib()
    assert L.psm_stream_copy(None, None, 16, None) == psm.PSM_EINVAL
    ms = ctypes.c_double(0)
    assert L.psm_pattern_copy(None, 1, 1, ctypes.byref(ms)) == psm.PSM_EINVAL
    assert L.psm_stream_copy(ctypes.c_void_p(256), ctypes.c_void_p(4096), 15, None) == psm.PSM_EINVAL
    assert L.psm_stream_copy(ctypes.c_void_p(256), ctypes.c_void_p(264), 64, None) == psm.PSM_EINVAL


def test_header_is_plain_c_and_links(tmp_path):
    """include/psm.h compiles as C99 on its own, and a C program calling the
    host-only entry points links against libpsm.so and runs without a GPU."""
    import shutil
    import subprocess

    cc = shutil.which("gcc")
    if cc is None:
        pytest.skip("no C compiler")
    src = tmp_path / "abi.c"
    src.write_text(r'''
#include <stdio.h>
#include "psm.h"
int main(void) {
    psm_box_desc d = {0};
    size_t bytes = 0;
    d.nx = 40; d.ny = 36; d.nz = 30; d.tau = 0.7;
    d.max_particles = 4; d.max_radius = 4.0; d.mapping = PSM_MAP_LINEAR; d.subsample_n = 4;
    d.walls_z = 1; d.face_type[0] = PSM_FACE_VELOCITY; d.face_type[1] = PSM_FACE_PRESSURE;
    d.face_rho[1] = 1.0;
    if (psm_workspace_size(&d, 1, PSM_FP32DEV, &bytes) != PSM_OK || bytes == 0) return 1;
    d.tau = 0.4;
    if (psm_workspace_size(&d, 1, PSM_FP32DEV, &bytes) != PSM_EINVAL) return 2;
    if (psm_step(NULL, 1) != PSM_EINVAL) return 3;
    printf("%zu %s\n", bytes, psm_last_error());
    return 0;
}
''')
    exe = tmp_path / "abi"
    libdir = os.path.dirname(psm.LIB_PATH)
    subprocess.run([cc, "-std=c99", "-Wall", "-Werror", "-pedantic", "-I", os.path.join(ROOT, "include"),
                    str(src), "-o", str(exe), "-L", libdir, "-lpsm", f"-Wl,-rpath,{libdir}"], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, (out.returncode, out.stdout, out.stderr)
    assert "ctx" in out.stdout


def test_row_pitch_padding_in_workspace_size():
    """Rows are padded to whole 64-cell blocks when that adds at most 1/8 to
    the row (nx 57-64 take the grid bytes of nx 64), narrower ones are packed
    (nx 56 takes less). Tile counts agree for these widths at every tile
    width, so the grids are the only difference."""
    def ws(nx):
        return psm.psm_workspace_size([psm.make_desc(nx, 16, 8, 0.6, max_particles=2, max_radius=2.0)],
                                      psm.PSM_FP64)
    assert ws(60) == ws(64) and ws(57) == ws(64)
    grid64 = 2 * 8 * (64 * 16 // 64) * 19 * 64 * 8
    grid56 = 2 * 8 * -(-(56 * 16) // 64) * 19 * 64 * 8
    assert ws(64) - ws(56) == grid64 - grid56


def test_last_error_is_per_thread():
    """Two threads failing in different ways each read back their own error
    text (psm_last_error is thread-local)."""
    import threading

    L = psm.lib()
    bad = {"tau": psm.make_desc(8, 8, 8, 0.4), "dimension": psm.make_desc(3, 8, 8, 0.6)}
    seen = {}
    barrier = threading.Barrier(2)

    def worker(key):
        arr = psm._desc_array([bad[key]])
        out = ctypes.c_size_t(0)
        msgs = []
        for _ in range(200):
            barrier.wait()
            assert L.psm_workspace_size(arr, 1, psm.PSM_FP64, ctypes.byref(out)) == psm.PSM_EINVAL
            barrier.wait()
            msgs.append(psm.psm_last_error())
        seen[key] = msgs

    ts = [threading.Thread(target=worker, args=(k,)) for k in bad]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for key, msgs in seen.items():
        assert len(msgs) == 200 and all(key in m for m in msgs), (key, set(msgs))


def test_plane_size_limit():
    """In-plane byte offsets are 32-bit signed: a z-plane (rows padded to whole
    64-cell blocks, 19 FP64 values per cell, plus one block) must stay below
    2^31 bytes. 4096 x 3449 cells fit, 4096 x 3450 do not."""
    ok = psm.make_desc(4096, 3449, 4, 0.6)
    assert 4096 * 3449 * 19 * 8 + 64 * 19 * 8 < 2 ** 31 <= 4096 * 3450 * 19 * 8 + 64 * 19 * 8
    assert psm.psm_workspace_size([ok], psm.PSM_FP16DEV) > 0
    with pytest.raises(psm.PsmError) as e:
        psm.psm_workspace_size([psm.make_desc(4096, 3450, 4, 0.6)], psm.PSM_FP16DEV)
    assert e.value.code == psm.PSM_EINVAL and "2^31" in str(e.value)


@pytest.mark.parametrize("storage,line", [(0, 16), (1, 32), (2, 64)])
def test_rows_of_large_grids_start_at_a_line(storage, line):
    """Grids beyond the last-level cache (256 MiB, both grids) whose rows are
    not padded to whole blocks start each at 128 bytes; smaller ones, and those
    beyond 64 GiB, are packed."""
    size = 8 >> storage

    def ws(nx, ny, nz):
        return psm.psm_workspace_size([psm.make_desc(nx, ny, nz, 0.6)], storage)

    def grids(pitch, ny, nz):
        return 2 * nz * -(-(pitch * ny) // 64) * 19 * 64 * size

    for nx, ny, nz in ((70, 64, 16), (70, 512, 128 << storage), (70, 4096, 2048 << (storage > 0))):
        packed, lined = grids(nx, ny, nz), grids(-(-nx // line) * line, ny, nz)
        extra = ws(nx, ny, nz) - ws(64, ny, nz) - (packed - grids(64, ny, nz))
        large = packed > 256 << 20 and lined <= 64 << 30
        tables = ws(64, ny, nz) - grids(64, ny, nz)   # nx 70 has up to twice the tiles of nx 64
        pad = lined - packed if large else 0
        assert pad <= extra <= pad + tables, (nx, ny, nz, large)


@pytest.mark.parametrize("storage", [0, 1, 2])
def test_row_padding_of_large_grids_is_bounded(storage):
    """Rows of one tile or less stay packed, however large the grids and
    whatever box is beside them, and the padding of a context's rows never
    takes more than 8 GiB."""
    size = 8 >> storage

    def ws(*dims):
        return psm.psm_workspace_size([psm.make_desc(*d, 0.6) for d in dims], storage)

    def grids(pitch, ny, nz):
        return 2 * nz * -(-(pitch * ny) // 64) * 19 * 64 * size

    for nx in (4, 9, 24, 33, 48, 56, 64):
        nz = (512 << 20) // (304 >> storage) // (nx * 512) + 1
        pitch = 64 if nx > 56 else nx
        tables = 8 * 512 * nz + (1 << 20)   # beside the grids: two counts per tile, one tile per row at most
        assert ws((nx, 512, nz)) - grids(pitch, 512, nz) <= tables, nx
        both = ws((nx, 512, nz), (192, 192, 128)) - grids(192, 192, 128)
        assert both - grids(pitch, 512, nz) <= tables + 8 * 192 * 128 * 12, nx
    for nx, ny, nz in ((65, 1024, 4096), (65, 2048, 4096), (65, 1024, 1024), (130, 1024, 1024)):
        assert ws((nx, ny, nz)) - grids(nx, ny, nz) <= (8 << 30) + (1 << 30), (nx, ny, nz)


def _plain_workspace(nx, ny, nz, n, rmax, size):
    """Bytes of the packed grids and of what every tile shape needs at least: 8
    per tile, and per slot (a tile a sphere can touch) a list entry and six
    sums; with 256 per sphere for the tables and 1 MiB for the rest."""
    tiles = slots = 0
    for tx in (16, 32, 64, 128, 256):
        for tz in (1, 2, 4, 8, 16, 32):
            T, reach = 1, n
            for L, t in ((nx, tx), (ny, 256 // tx), (nz, tz)):
                nt = -(-L // t)
                T *= nt
                reach *= min(nt, 2 + -(-max(int(2 * (rmax + 1)) + 2 - (L - (nt - 1) * t), 0) // t))
            tiles, slots = max(tiles, T), max(slots, reach)
    return 2 * nz * -(-(nx * ny) // 64) * 19 * 64 * size + 8 * tiles + 56 * slots + 256 * n + (1 << 20)


@pytest.mark.parametrize("storage,dims,n,rmax", [
    (0, (960, 960, 960), 885000, 4.0), (0, (960, 960, 960), 100, 4.0), (2, (1024, 1000, 1000), 1000000, 4.0),
    (2, (1024, 1024, 900), 40, 4.0), (2, (256, 256, 256), 1000000, 1.0), (1, (512, 512, 512), 2347, 10.0),
    (0, (64, 64, 64), 200000, 1.0), (1, (32, 32, 32), 8, 4.0), (2, (64, 64, 64), 0, 1.0)])
def test_lists_and_partials_leave_the_memory_to_the_grids(storage, dims, n, rmax):
    """Room for lists of a fixed capacity, a second set of force partials and
    shared tiles is at most a quarter of the plain workspace or 64 MiB, and
    nothing beyond 64 GiB (boxes of whole 64-cell blocks, so rows are packed)."""
    plain = _plain_workspace(*dims, n, rmax, 8 >> storage)
    got = psm.psm_workspace_size([psm.make_desc(*dims, 0.6, max_particles=n, max_radius=rmax)], storage)
    assert got <= max(plain, min(max(plain + plain // 4, plain + (64 << 20)), 64 << 30))


class _FakeTorch:
    """Streams, events and the current device of torch, as a log of what each
    thread did; the caller's stream of a thread is its name."""
    float64 = "float64"

    def __init__(self):
        fake = self
        self.now, self.log = threading.local(), []

        class Event:
            def record(self, stream):
                fake.log.append((threading.current_thread().name, "record", stream))

        class device:
            def __init__(self, index):
                self.index = index

            def __enter__(self):
                self.before, fake.now.device = getattr(fake.now, "device", 0), self.index

            def __exit__(self, *exc):
                fake.now.device = self.before

        class cuda:
            pass
        cuda.Event, cuda.device = Event, device
        cuda.current_stream = staticmethod(lambda dev: fake.Stream(threading.current_thread().name))
        self.cuda = cuda

    def Stream(self, name, device=0):
        stream = types.SimpleNamespace(name=name, device=device)
        stream.wait_event = lambda ev: self.log.append((threading.current_thread().name, "wait", name))
        return stream

    def empty(self, shape, dtype, device):
        return types.SimpleNamespace(data_ptr=lambda: 0)


def _fake_engine():
    eng = psm.Engine.__new__(psm.Engine)
    eng.torch = _FakeTorch()
    eng.ctx, eng.device, eng.stream = None, "cuda:1", eng.torch.Stream("engine", device=1)
    eng._caller_done, eng._engine_done = eng.torch.cuda.Event(), eng.torch.cuda.Event()
    eng._events = threading.Lock()
    return eng


def test_read_outs_launch_with_the_engines_device_current():
    """An engine on GPU 1 called while GPU 0 is current: the library launches
    with GPU 1 current, and GPU 0 is current again afterwards."""
    eng = _fake_engine()
    eng.torch.now.device = 0
    seen = []
    eng._read_out([((4,), "float64")], lambda p: seen.append(eng.torch.now.device))
    assert seen == [1] and eng.torch.now.device == 0


def test_read_outs_of_two_threads_do_not_mix_their_events():
    """A second thread's read-out does not record the engine's events between a
    first one's record and wait (its own thread-local stream would be waited
    for in place of the first's)."""
    eng = _fake_engine()
    inside, second = threading.Event(), threading.Event()

    def first_launch(p):
        inside.set()
        second.wait(0.5)   # time for the second thread to get in, if it can

    def other():
        inside.wait()
        eng._read_out([((4,), "float64")], lambda p: None)
        second.set()

    a = threading.Thread(target=lambda: eng._read_out([((4,), "float64")], first_launch), name="a")
    b = threading.Thread(target=other, name="b")
    for t in (a, b):
        t.start()
    for t in (a, b):
        t.join()
    assert [who for who, _, _ in eng.torch.log] == ["a"] * 4 + ["b"] * 4
