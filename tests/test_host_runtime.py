"""The host side of the C ABI against a stand-in for the HIP runtime
(tests/fake_hip.cpp, linked with the library's own objects): on which device
streams and graphs are made, what is launched, what happens when the runtime
refuses a call. No GPU is needed; kernels are recorded, not run."""
import ctypes
import glob
import importlib.util
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2311_10314_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def fake_module(tmp_path_factory):
    """The binding over the library's objects linked with the stand-in."""
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ not available")
    objs = [os.path.join(B.BUILD, os.path.splitext(s)[0] + ".o")
            for s in B.SOURCES]
    newest = max(os.path.getmtime(f)
                 for f in glob.glob(os.path.join(B.CSRC, "*")))
    if not all(os.path.exists(o) and os.path.getmtime(o) >= newest
               for o in objs):
        B.build()
    d = tmp_path_factory.mktemp("fake")
    obj = str(d / "fake_hip.o")
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-fPIC",
                    "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-c",
                    os.path.join(HERE, "fake_hip.cpp"), "-o", obj], check=True)
    # the stand-in's names are bound inside the library, whatever runtime
    # this process has loaded
    subprocess.run([gxx, "-shared", "-Wl,-Bsymbolic", "-Wl,-z,defs", "-o",
                    str(d / "libddcc.so"), obj] + objs, check=True)
    shutil.copy(os.path.join(os.path.dirname(B.LIB), "ddcc.py"),
                str(d / "ddcc.py"))
    spec = importlib.util.spec_from_file_location("ddcc_on_fake",
                                                  str(d / "ddcc.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    mod.LIB.fake_get.restype = ctypes.c_longlong
    mod.LIB.fake_set.argtypes = [ctypes.c_char_p, ctypes.c_longlong]
    return mod


class Fake:
    def __init__(self, mod):
        self.d, self.lib = mod, mod.LIB

    def set(self, key, value):
        self.lib.fake_set(key.encode(), value)

    def get(self, key):
        return self.lib.fake_get(key.encode())

    def launches(self, start=0):
        """(kernel, grid, block, device of the stream, current device,
        captured) of the launches from `start` on."""
        out, name = [], ctypes.create_string_buffer(1024)
        v = (ctypes.c_longlong * 9)()
        for i in range(start, self.get("launches")):
            self.lib.fake_launch(i, name, 1024, v)
            out.append((name.value.decode(), tuple(v[:3]), tuple(v[3:6]),
                        v[6], v[7], bool(v[8])))
        return out

    def sim(self, shape, N=2, precision="fp32", lattice="D3Q15"):
        dim = len(shape)
        prm = dict(d0=0.3) if lattice == "D3Q7" else {}
        p = self.d.make_params(dim, shape, N,
                               "D2Q9" if dim == 2 else lattice,
                               "D2Q9" if dim == 2 else "D3Q19", precision,
                               **prm)
        s = self.d.Sim(p)
        s.init_geometry(np.ones(shape))
        C = np.zeros((N,) + tuple(shape))
        C[0] = 1.0
        s.init_fields(C)
        return s


@pytest.fixture
def fake(fake_module):
    fake_module.LIB.fake_reset()
    f = Fake(fake_module)
    yield f
    fake_module.LIB.fake_reset()


# ---- devices -----------------------------------------------------------------
def test_captured_groups_are_made_on_the_contexts_device(fake):
    """A context of device 1 stepped while device 0 is current: its captured
    groups are recorded on a stream of device 1, with device 1 current, and
    device 0 is current again afterwards."""
    fake.lib.hipSetDevice(1)
    s = fake.sim((40, 70))
    fake.lib.hipSetDevice(0)
    s.step(128)
    s.step(200)
    assert fake.get("graph_calls") > 0
    captured = [x for x in fake.launches() if x[5]]
    assert captured and all(x[3] == 1 and x[4] == 1 for x in captured)
    assert fake.get("streams_on_0") == 0
    assert fake.get("current") == 0
    s.close()


def test_adjoint_stream_is_made_on_the_contexts_device(fake):
    fake.set("fill", 0x3f)      # the phase mass is not zero
    fake.lib.hipSetDevice(1)
    s = fake.sim((24, 70), precision="fp64")
    fake.lib.hipSetDevice(0)
    s.adjoint(6, 2, 0, np.ones((24, 70)))
    assert fake.get("streams_on_1") == 2      # the context's own and this one
    assert fake.get("streams_on_0") == 0 and fake.get("events_on_0") == 0
    assert all(x[3] == 1 for x in fake.launches())
    assert fake.get("current") == 0
    s.close()


# ---- captured groups of steps ------------------------------------------------
def test_a_new_tile_does_not_make_step_wait(fake):
    """ddcc_step enqueues and returns, also after a change of the tile: groups
    in flight are neither waited for nor dropped, and the first tile's serve
    again when it comes back."""
    s = fake.sim((40, 70))
    s.step(128)
    s.step(200)
    made, waits = fake.get("graphs"), fake.get("syncs")
    s.set_tile(0, 8)
    s.step(200)
    other = fake.get("graphs")
    assert other > made
    s.set_tile(0, 2)
    s.step(200)
    assert fake.get("graphs") == other
    assert fake.get("syncs") == waits
    assert s.time == 728
    s.close()
    assert fake.get("graphs") == 0


def test_a_new_tile_while_the_thread_captures_elsewhere(fake):
    """The caller's thread records on a stream of its own meanwhile: ddcc_step
    calls nothing that would break that recording."""
    s = fake.sim((40, 70))
    s.step(128)
    s.step(200)
    s.set_tile(0, 8)
    fake.set("thread_captures", 1)
    s.step(200)
    assert fake.get("captures_broken") == 0
    assert s.time == 528
    fake.set("thread_captures", 0)
    s.close()


@pytest.mark.parametrize("key,value", [("fail_is_capturing", 1),
                                       ("fail_instantiate", 1),
                                       ("fail_graph", 1), ("fail_graph", 2)])
def test_steps_go_on_one_by_one_where_groups_are_refused(fake, key, value):
    """Groups are a way of launching only: where the runtime refuses the query,
    the group or its launch, the same steps are launched one by one, and the
    refusal is not taken for an error of theirs."""
    s = fake.sim((40, 70))
    s.step(128)
    before = fake.get("launches")
    fake.set(key, value)
    s.step(200)
    assert s.time == 328
    single = [x for x in fake.launches(before) if not x[5]]
    assert len(single) + fake.get("graph_kernels") == 200
    s.close()


def test_occupancy_query_leaves_no_error_behind(fake):
    fake.set("fail_occupancy", 1)
    s = fake.sim((6, 8, 20), precision="fp16", lattice="D3Q7")
    s.step(1)
    s.close()


# ---- adjoint -------------------------------------------------------------------
def test_a_failed_adjoint_leaves_time_with_the_state(fake):
    """The last segment's forward steps are written to the sweep's own memory:
    if one of them fails, or the first copy of the final state, the context
    holds the level of that segment's checkpoint, and says so."""
    fake.set("fill", 0x3f)
    for failing, want in (("kernel", 4), ("copy", 4), ("none", 6)):
        s = fake.sim((24, 70), precision="fp64")
        if failing == "kernel":       # the sixth step from here
            fake.set("fail_kernel", fake.get("kernel_calls") + 6)
        elif failing == "copy":
            # weights; populations, rest, g, history, T of the checkpoints of
            # levels 0, 2 and 4; then the final state's
            fake.set("fail_copy", fake.get("copies") + 1 + 3 * 5 + 1)
        w = np.ones((24, 70))
        if failing == "none":
            s.adjoint(6, 2, 0, w)
        else:
            with pytest.raises(fake.d.DDCCError, match=(
                    "step kernel" if failing == "kernel" else "final state")):
                s.adjoint(6, 2, 0, w)
        assert s.time == want, failing
        s.close()


# ---- errors ----------------------------------------------------------------------
def test_an_error_is_reported_once(fake):
    """A refused allocation or copy fails its call; the next calls, on this
    context or another, launch their kernels as if it had not been."""
    s = fake.sim((40, 70))
    fake.set("fail_copy", fake.get("copies") + 1)
    with pytest.raises(fake.d.DDCCError, match="copy"):
        s.read_moments()
    s.step(1)
    fake.set("memory", fake.get("allocated") + 1000)
    with pytest.raises(fake.d.DDCCError) as e:
        fake.sim((40, 70))
    assert e.value.code == fake.d.DDCC_E_NOMEM
    s.step(1)
    p = fake.d.make_params(2, (40, 70), 2, "D2Q9", "D2Q9", "fp32")
    with pytest.raises(fake.d.DDCCError):
        fake.d.Batch(p, [(40, 70), (30, 20)])
    s.step(1)
    fake.set("memory", 0)
    s.close()


# ---- batches -----------------------------------------------------------------------
def test_a_batch_of_more_tiles_than_one_launch_takes(fake):
    """One instance of 1 x 2^26 nodes has 2^23 tiles of 64 x 8, 2^32 threads,
    which is more than a launch takes: every tile is launched once all the
    same."""
    ny = 1 << 26
    p = fake.d.make_params(2, (ny, 1), 2, "D2Q9", "D2Q9", "fp32")
    b = fake.d.Batch(p, [(ny, 1)])
    b.init_geometry(0, np.zeros((ny, 1)))
    b.init_fields(0, np.zeros((2, ny, 1)))
    start = fake.get("launches")
    b.step(1)
    steps = fake.launches(start)
    assert len(steps) > 1
    assert sum(x[1][0] for x in steps) == ny // 8
    b.close()


# ---- memory ------------------------------------------------------------------------
def test_a_box_whose_padded_rows_do_not_fit_keeps_its_rows(fake):
    """Rows of 100 FP32 nodes are padded to 128 on the device. With memory for
    the dense box only, the context is made with dense rows; with less, it is
    refused, and nothing is left behind."""
    shape = (300, 200, 100)       # above the cache's size either way
    s = fake.sim(shape)
    padded = fake.get("allocated")
    s.close()
    assert fake.get("allocated") == 0
    p = fake.d.make_params(3, shape, 2, "D3Q15", "D3Q19", "fp32")
    dense = 100 * padded // 128   # and some small buffers
    fake.set("memory", dense + (1 << 20))
    s = fake.d.Sim(p)
    assert 0 < fake.get("allocated") <= dense + (1 << 20)
    s.close()
    fake.set("memory", dense // 2)
    with pytest.raises(fake.d.DDCCError) as e:
        fake.d.Sim(p)
    assert e.value.code == fake.d.DDCC_E_NOMEM
    assert fake.get("allocated") == 0 and fake.get("streams") == 0


@pytest.mark.parametrize("nsteps,interval,states", [
    (1, 1, 2), (2, 1, 4), (6, 2, 7), (5, 2, 7), (6, 6, 7), (6, 100, 7)])
def test_adjoint_holds_no_state_it_does_not_use(fake, nsteps, interval, states):
    """Stored states: a checkpoint for each segment but the last, two segment
    buffers (one where there is one segment), the final state."""
    fake.set("fill", 0x3f)
    s = fake.sim((24, 70), precision="fp64")
    def peak(n, k):
        fake.set("peak", 0)
        s.adjoint(n, k, 0, np.ones((24, 70)))
        return fake.get("peak")
    none = peak(0, 1)             # the final state alone
    s.close()
    # populations and rest populations, flow set, history and T of the sweep's
    # slots: each a whole number of 256 bytes
    n = 24 * 70 * 8
    state = sum((x * n + 255) // 256 * 256 for x in (2 * 8, 2, 9, 8, 1))
    s = fake.sim((24, 70), precision="fp64")
    assert peak(nsteps, interval) - none == (states - 1) * state
    s.close()


# ---- launch shapes -------------------------------------------------------------------
def _step_kernel(fake, shape, N, precision, lattice="D3Q15", tile=0):
    """Name and workgroup size of the last kernel of a step."""
    s = fake.sim(shape, N, precision, lattice)
    s.set_tile(0, tile)
    s.step(1)
    name, _, block = fake.launches(fake.get("launches") - 1)[0][:3]
    s.close()
    return name, block[0]


@pytest.mark.parametrize("N,precision,ny,wide", [
    (4, "fp16", 160, True), (4, "fp16", 180, False), (4, "bf16", 256, False),
    (4, "fp32", 256, True), (3, "fp16", 256, True), (2, "bf16", 257, False)])
def test_wide_workgroups_of_four_phases_leave_room(fake, N, precision, ny,
                                                   wide):
    """256 nodes wide, 256 compute units: 64 x 4 tiles in wide workgroups while
    they are at most 256, and 170 for four phases in 16-bit storage."""
    name, block = _step_kernel(fake, (ny, 256), N, precision)
    assert ("k_step2d_wide" in name) == wide
    assert block == (576 if wide else 512)


@pytest.mark.parametrize("N,precision,shape,pitch", [
    (2, "fp32", (42, 90, 130), 130),    # 0.98 of the cache dense, 1.21 padded
    (3, "fp32", (36, 110, 80), 80),     # 0.81, 0.97
    (2, "fp16", (79, 110, 80), 80),     # 0.90, 1.08
    (2, "fp32", (25, 100, 150), 160),   # 0.75, 0.80
    (2, "fp32", (63, 110, 100), 128),   # 1.38, 1.77
    (2, "fp64", (48, 110, 130), 144)])  # 2.8, 3.1
def test_rows_are_padded_where_the_cache_holds_them_or_neither(
        fake, N, precision, shape, pitch):
    """Device memory of the context: the planes are pitch nodes wide."""
    def allocated(width):
        p = fake.d.make_params(3, shape[:2] + (width,), N, "D3Q15", "D3Q19",
                               precision)
        s = fake.d.Sim(p)
        n = fake.get("allocated")
        s.close()
        return n
    # 64 nodes a row are never padded
    per_row_node = allocated(64) / 64.0
    assert abs(allocated(shape[2]) / per_row_node - pitch) < 0.5


@pytest.mark.parametrize("precision,shape,tile,narrow", [
    ("fp64", (90, 60, 65), 0, True), ("fp64", (64, 90, 72), 0, True),
    ("fp64", (64, 90, 96), 0, False), ("fp64", (80, 100, 88), 0, False),
    ("fp64", (40, 40, 96), 0, False), ("fp64", (60, 90, 96), 0, True),
    ("fp64", (79, 110, 96), 0, True), ("fp64", (100, 160, 80), 4, True),
    ("fp64", (90, 60, 97), 0, False), ("fp64", (90, 60, 129), 0, True),
    ("fp64", (90, 60, 160), 0, True), ("fp64", (90, 60, 161), 0, False),
    ("fp32", (90, 60, 65), 0, False), ("fp32", (20, 20, 32), 0, True),
    ("fp64", (90, 60, 65), 2, False)])
def test_shape_of_3d_tiles(fake, precision, shape, tile, narrow):
    """32 x 8 instead of 64 x 4 tiles (256 compute units); 64 x 2 as asked."""
    name, block = _step_kernel(fake, shape, 2, precision, tile=tile)
    want = "32, 8>" if narrow else "64, %d>" % (tile or 4)
    assert "k_step3d" in name and want in name.split("(ddcc::Coef")[0]
    assert block == (128 if tile == 2 else 256)


def test_no_wide_kernel_is_built_that_nothing_launches(fake):
    name, wide = ctypes.create_string_buffer(1024), []
    for i in range(fake.lib.fake_kernel_count()):
        fake.lib.fake_kernel_name(i, name, 1024)
        if b"k_step2d_wide<" in name.value:
            wide.append(name.value.decode().split(">(")[0].split("<")[1])
    assert len(wide) > 0
    assert not [w for w in wide if "double, double, double" in w
                and w.endswith(", 4")]


def test_geometry_needs_memory_for_its_walls_only(fake):
    """The planes that host-array calls share do not fit, the walls do."""
    shape = (64, 128)
    p = fake.d.make_params(2, shape, 3, "D2Q9", "D2Q9", "fp64")
    s = fake.d.Sim(p)
    plane = 8 * 64 * 128
    # psi and two angles; float64 psi and angles that stay for the adjoint
    fake.set("memory", fake.get("allocated") + 6 * plane + 1000)
    s.init_geometry(np.ones(shape), np.zeros((2,) + shape))
    fake.set("memory", 0)
    s.close()
