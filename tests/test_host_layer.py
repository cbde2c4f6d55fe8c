"""The library's host layer (lbm_api, host_copy) on a fake device that runs on the CPU
(host_fake.cpp): order of copies and launches, streams, devices, memory and failing launches."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2609_28679_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_28679_amd", "csrc")
PER_THREAD = 2  # hipStreamPerThread
STREAM = 0x1000  # any other handle
ROCM = "/opt/rocm/include"

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(ROCM),
                                reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def fake_lib(tmp_path_factory):
    out = tmp_path_factory.mktemp("host") / "libhost.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-pthread", "-Wl,-Bsymbolic",
                    "-D__HIP_PLATFORM_AMD__", "-isystem", ROCM, "-I", os.path.join(ROOT, "include"),
                    "-I", CSRC, "-o", str(out), "-x", "c++", os.path.join(CSRC, "lbm_api.hip"),
                    os.path.join(CSRC, "host_copy.hip"),
                    os.path.join(ROOT, "tests", "host_fake.cpp")], check=True)
    lib = ctypes.CDLL(str(out))
    for name, (res, args) in binding.SIGNATURES.items():
        if hasattr(lib, name):
            getattr(lib, name).restype, getattr(lib, name).argtypes = res, args
    lib.fake_uploaded.restype = ctypes.POINTER(ctypes.c_double)
    lib.fake_foreign.restype = lib.fake_pins.restype = lib.fake_pinned_bytes.restype = ctypes.c_long
    lib.fake_capture.argtypes = [ctypes.c_void_p, ctypes.c_int]
    lib.fake_replay.argtypes = [ctypes.c_void_p]
    lib.fake_malloc_limit.argtypes = [ctypes.c_size_t]
    return lib


@pytest.fixture
def fake(fake_lib):
    fake_lib.fake_reset()
    return fake_lib


class Context:
    """One context of the library on the fake device; read-outs hold the steps of the state."""

    def __init__(self, lib, shape=(64, 64), stream=STREAM, expect=binding.LBM_OK, **kw):
        self.lib, self.shape = lib, shape
        p = binding.LbmParams()
        lib.lbm_default_params(ctypes.byref(p))
        p.ny, p.nx = shape[-2:]
        if len(shape) == 3:
            p.lattice, p.nz = 1, shape[0]
        p.stream = stream
        for k, v in kw.items():
            setattr(p, k, v)
        self.D = len(shape)
        self.rho = 1.0 + np.arange(np.prod(shape), dtype=np.float64).reshape(shape) * 1e-9
        u = np.zeros((self.D,) + shape)
        T = np.ones(shape)
        self.ctx = ctypes.c_void_p()
        rc = lib.lbm_create(ctypes.byref(p), binding._dptr(self.rho), binding._dptr(u),
                            binding._dptr(T), ctypes.byref(self.ctx))
        assert rc == expect, lib.lbm_last_error(None)

    def step(self, n, expect=binding.LBM_OK):
        assert self.lib.lbm_step(self.ctx, n) == expect

    def moments(self, totals=False):
        rho = np.full(self.shape, np.nan)
        u = np.full((self.D,) + self.shape, np.nan)
        t = np.empty(5)
        rc = self.lib.lbm_moments(self.ctx, binding._dptr(rho), binding._dptr(u), None,
                                  binding._dptr(t) if totals else None)
        assert rc == binding.LBM_OK, self.lib.lbm_last_error(self.ctx)
        out = np.concatenate([rho.ravel(), u.ravel()])
        tag = (np.arange(out.size) % 4099) / 8192.0
        steps = out - tag
        assert np.all(steps == steps[0]), "values of several states, or out of place"
        return int(steps[0])

    def moments_into(self, rho, u):
        return self.lib.lbm_moments(self.ctx, binding._dptr(rho), binding._dptr(u), None, None)

    def populations(self):
        f = np.full((3 ** self.D,) + self.shape, np.nan)
        assert self.lib.lbm_populations(self.ctx, binding._dptr(f), None) == binding.LBM_OK
        n = f[0].size
        steps = f.reshape(-1, n) - (np.arange(n) % 4099) / 8192.0 - 1000.0 * np.arange(len(f))[:, None]
        assert np.all(steps == steps[0, 0])
        return int(steps[0, 0])

    def close(self):
        self.lib.lbm_destroy(self.ctx)


# 0.3, 5, 20 and 270 MB of fields (uploads are staged from 64 MiB on)
@pytest.mark.parametrize("shape", [(100, 128), (401, 509), (1000, 833), (3307, 3400)])
@pytest.mark.parametrize("stream", [STREAM, PER_THREAD, None])
def test_copies_keep_the_order_of_the_callers_stream(fake, shape, stream):
    """Everything that a copy puts on the caller's stream is put there by the calling thread: a
    handle may mean another queue in another thread."""
    c = Context(fake, shape, stream)
    up = np.ctypeslib.as_array(fake.fake_uploaded(), (c.rho.size,))
    assert np.array_equal(up, c.rho.ravel())
    c.step(3)
    assert c.moments() == 3
    assert c.moments(totals=True) == 3
    if shape[0] <= 1000:
        assert c.populations() == 3
    assert fake.fake_foreign() == 0
    c.close()


def test_copies_leave_the_callers_device(fake):
    """A program with several GPUs reads out a context of device 0 while device 1 is current."""
    c = Context(fake, (401, 509))
    fake.fake_set_device(1)
    c.step(2)
    assert c.moments() == 2 and c.populations() == 2
    assert fake.fake_current_device() == 1
    fresh = Context(fake, (1000, 833))  # its first copy, and so its events, with device 1 current
    assert fresh.moments() == 0
    assert fake.fake_current_device() == 1
    c.close()
    fresh.close()


def test_pinned_memory_of_the_caller_is_copied_directly(fake):
    c = Context(fake, (1000, 833))
    n = c.rho.size
    p = ctypes.c_void_p()
    fake.hipHostMalloc(ctypes.byref(p), ctypes.c_size_t(3 * n * 8), 0)
    out = np.ctypeslib.as_array(ctypes.cast(p, binding._D), (3, n))
    pins = fake.fake_pins()
    copies = fake.fake_copies()
    assert c.moments_into(out[0], out[1:]) == binding.LBM_OK
    assert fake.fake_pins() == pins and fake.fake_copies() == copies + 2
    assert np.array_equal(out[0], np.arange(n) % 4099 / 8192.0)
    c.close()
    fake.hipHostFree(p)


def test_contexts_made_one_at_a_time_pin_nothing_to_start(fake):
    """Initial fields of 15 MB need no staging memory. A read-out pins one slab, which later ones
    of any context use too, and the last context to go gives it back."""
    shape = (700, 900)
    for _ in range(3):
        Context(fake, shape).close()
    assert fake.fake_pins() == 0
    a = Context(fake, shape)
    assert a.moments() == 0 and fake.fake_pins() == 1
    b = Context(fake, shape)
    assert b.moments() == 0 and a.moments() == 0 and fake.fake_pins() == 1
    a.close()
    assert fake.fake_pinned_bytes() > 0
    b.close()
    assert fake.fake_pinned_bytes() == 0


def _workspace_size(lib, shape, **kw):
    p = binding.LbmParams()
    lib.lbm_default_params(ctypes.byref(p))
    p.ny, p.nx = shape
    for k, v in kw.items():
        setattr(p, k, v)
    n = ctypes.c_size_t(0)
    assert lib.lbm_workspace_size(ctypes.byref(p), ctypes.byref(n)) == 0
    return n.value


def _up(n):
    return (n + 255) // 256 * 256


@pytest.mark.parametrize("storage,elem", [("fp32", 4), ("fp64", 8)])
def test_workspace_without_room_for_several_steps_per_launch(fake, storage, elem):
    """A caller's workspace that holds one state and the read-out area is accepted, as is device
    memory of that size; the run takes one step per launch."""
    shape = (40, 65)
    kw = dict(storage=binding.STORAGES[storage])
    full = _workspace_size(fake, shape, **kw)
    least = full - (_up(9 * 128 * 40 * elem) - _up(5 * 65 * 40 * 8))
    buf = ctypes.create_string_buffer(full + 256)
    base = (ctypes.addressof(buf) + 255) // 256 * 256
    for size, launches in ((full, 3), (full - 1, 13), (least, 13)):
        c = Context(fake, shape, workspace=base, workspace_bytes=size, **kw)
        before = fake.fake_step_launches()
        c.step(13)
        assert fake.fake_step_launches() - before == launches
        assert c.moments() == 13 and c.populations() == 13
        c.close()
    Context(fake, shape, expect=binding.LBM_ENOMEM, workspace=base, workspace_bytes=least - 1, **kw)
    fake.fake_malloc_limit(full - 1)
    c = Context(fake, shape, **kw)
    c.step(13)
    assert c.moments() == 13
    c.close()
    fake.fake_malloc_limit(least - 1)
    Context(fake, shape, expect=binding.LBM_ENOMEM, **kw)


def test_workspace_with_records_of_the_plans_windows(fake):
    """Lower windows than the plan's own may write more records."""
    shape = (3200, 16)
    records = fake.fake_ddf_records(shape[1], shape[0], 1, 0)
    assert records > 1024
    full = _workspace_size(fake, shape, model=1)
    least = full - (_up(records * 40) - _up(1024 * 40))
    buf = ctypes.create_string_buffer(full + 256)
    base = (ctypes.addressof(buf) + 255) // 256 * 256
    for size, room in ((full, records), (least, 1024)):
        c = Context(fake, shape, model=1, diag_every=1, workspace=base, workspace_bytes=size)
        c.step(5)
        assert fake.fake_record_room() == room and c.moments() == 5
        c.close()


MODELS = {"d2q9": ((40, 65), {}), "d2q9_two": ((40, 65), dict(streaming=1)),
          "d3q27_two": ((20, 100, 100), dict(streaming=1)), "ddf": ((840, 840), dict(model=1)),
          "bf16": ((40, 65), dict(storage=1))}


@pytest.mark.parametrize("model", sorted(MODELS))
@pytest.mark.parametrize("n", [2, 4, 6, 8, 10, 12, 14, 18, 20, 26])
def test_replays_of_a_captured_call_advance_the_state(fake, model, n):
    shape, kw = MODELS[model]
    for before in (0, 2, 6, 7):
        fake.fake_reset()
        c = Context(fake, shape, **kw)
        c.step(before)
        fake.fake_capture(STREAM, 1)
        c.step(n)
        fake.fake_capture(STREAM, 0)
        assert c.moments() == before  # captured, not run
        for k in range(1, 4):
            fake.fake_replay(STREAM)
            assert c.moments() == before + k * n, (before, k)
        c.close()


@pytest.mark.parametrize("model", sorted(MODELS))
def test_calls_take_their_steps(fake, model):
    """Any cutting of a run into calls, with and without diagnostics entries."""
    shape, kw = MODELS[model]
    for every in (0, 1, 2, 3, 4, 7):
        c = Context(fake, shape, diag_every=every, **kw)
        t = 0
        for n in (1, 2, 3, 5, 6, 7, 0, 12, 13, 25, 4, 40):
            c.step(n)
            t += n
            assert c.moments() == t, (every, n)
        c.close()


@pytest.mark.parametrize("model", sorted(MODELS))
@pytest.mark.parametrize("k", [1, 2, 3])
def test_failing_launch_leaves_a_state_that_can_be_read(fake, model, k):
    """The k-th launch of a call fails: the context stands at the steps taken until then."""
    shape, kw = MODELS[model]
    c = Context(fake, shape, **kw)
    fake.fake_fail_step_launch(k)
    c.step(24, expect=binding.LBM_EDEVICE)
    t = ctypes.c_int64(0)
    assert fake.lbm_time(c.ctx, ctypes.byref(t)) == 0
    for _ in range(2):
        assert c.moments() == t.value
    assert c.populations() == t.value
    c.step(7)
    assert c.moments() == t.value + 7
    c.close()


# (nx, ny): us per step of one step per launch / of two, measured on MI355X
PLAIN, SOURCES, TRANSPORT, VDW = (0, 0, 0, 0), (1, 0, 0, 0), (0, 1, 0, 0), (0, 0, 1, 0)
NEQ, NEQ_TRANSPORT, NEQ_VDW = (0, 0, 0, 1), (0, 1, 0, 1), (0, 0, 1, 1)
FASTER = {
    PLAIN: [(2048, 2048), (1024, 1024), (120000, 6), (250, 3000), (3, 240000), (60, 12000)],
    SOURCES: [(2048, 2048), (1100, 1001), (900, 900), (30000, 48), (200, 6000)],
    TRANSPORT: [(2048, 2048), (1024, 1024), (900, 900), (30000, 48), (1100, 1001)],
    VDW: [(2048, 2048), (1024, 1024), (1100, 1001), (30000, 48)],
    NEQ: [(2048, 2048), (1021, 509), (700, 600), (120000, 6), (270, 2000), (3, 240000)],
    NEQ_TRANSPORT: [(2048, 2048), (1021, 509), (700, 640), (304, 10605), (60000, 12), (499, 2003)],
    NEQ_VDW: [(2048, 2048), (1021, 509), (1000, 768), (60000, 12)],
}
SLOWER = {
    PLAIN: [(512, 512), (240000, 3), (130, 6000)],                           # 1.17, 1.04 x
    SOURCES: [(240000, 3), (120000, 6), (30, 25000), (130, 6000), (256, 3000), (200000, 12),
              (768, 1000)],                                                  # 1.87 ... 1.05 x
    TRANSPORT: [(240000, 3), (120000, 6), (3, 240000), (60, 12000), (130, 6000), (200000, 12)],
    VDW: [(240000, 3), (3, 240000), (30, 25000), (1024, 700), (1000, 768), (768, 1000), (260, 2900)],
    NEQ: [(512, 512), (240000, 3), (130, 6000)],                             # 1.20, 1.38 x
    NEQ_TRANSPORT: [(240000, 3), (3, 240000), (130, 6000), (270, 2000), (311, 1992)],  # 1.33 ... 1.09 x
    NEQ_VDW: [(240000, 3), (120000, 6), (30, 25000), (200000, 12), (270, 2000)],
}


@pytest.mark.parametrize("options", sorted(FASTER))
def test_two_ddf_steps_per_launch_where_they_are_faster(fake, options):
    for nx, ny in FASTER[options]:
        assert fake.fake_ddf_pair(nx, ny, *options) == 1, (nx, ny)
    for nx, ny in SLOWER[options]:
        assert fake.fake_ddf_pair(nx, ny, *options) == 0, (nx, ny)


# collisions: 0 plain, 1 sources or transport control, 2 van der Waals; us a step
@pytest.mark.parametrize("nx,ny,phi,fmt,collision,rows", [
    (700, 640, 1, 0, 0, 4),   # 19.3; 3 rows 21.8
    (512, 512, 1, 0, 0, 2),   # 14.0; 4 rows 16.0
    (640, 500, 1, 0, 0, 2),   # 15.4; 4 rows 18.0
    (2048, 2048, 1, 0, 0, 4),
    (4096, 4096, 1, 2, 0, 16),  # bfloat16: 514; 14 rows 527
    (2048, 2048, 1, 3, 0, 16),  # float16: 137; 13 rows 146
    (3000, 3000, 1, 2, 0, 16),  # 282; 15 rows 305
    (512, 512, 1, 3, 0, 4),     # 22.2; 16 rows 40.2
    (512, 512, 1, 0, 1, 4),   # 17.9; 8 rows 22.7
    (1021, 509, 1, 0, 1, 5),  # 24.8; 8 rows 32.1
    (64, 64, 2, 0, 0, 1),
    (270, 2000, 2, 0, 2, 16),  # 52.3; 8 rows 55.9
    (270, 2000, 2, 1, 1, 16),  # 56.9; 8 rows 62.5
    (768, 768, 2, 1, 1, 12),   # 54.4; 6 rows 68.7
    (768, 768, 2, 0, 2, 12),   # 43.7; 6 rows 50.2
    (1024, 1024, 2, 0, 1, 11),
])
def test_window_rows_of_one_ddf_step(fake, nx, ny, phi, fmt, collision, rows):
    assert fake.fake_ddf_rows(nx, ny, phi, fmt, collision, 0) == rows


def test_two_d3q27_steps_per_launch_where_they_are_faster(fake):
    for shape in ((64, 64, 64), (100, 100, 20), (129, 500, 20), (1000, 1000, 3), (700, 9, 64),
                  (66, 20, 1000), (30, 300, 64), (256, 256, 256)):
        assert fake.fake_bgk3_pair(*shape) == 1, shape
    # 1.4 to 2 times slower, and six times on 3 x 3 columns
    for shape in ((10, 10, 10), (32, 32, 32), (48, 48, 48), (3000, 1, 1), (65, 300, 4),
                  (2000, 2000, 1), (1000, 500, 2), (64, 9, 200), (128, 9, 300), (3, 3, 100000)):
        assert fake.fake_bgk3_pair(*shape) == 0, shape
