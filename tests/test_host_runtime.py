"""The library's host side on the CPU: mvf_runtime.cpp against a HIP runtime
and kernel launchers over host memory (native/host_hip.cpp), which note the
device that is current at each call, work that nothing orders after the
earlier work on other streams, and allocations."""
import ctypes as C
import os
import subprocess
import tempfile

import numpy as np
import pytest

from paper_1511_07106_amd import _lib as L

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1511_07106_amd", "csrc")


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("needs the HIP headers")
    so = os.path.join(tempfile.mkdtemp(prefix="mvf_host_"), "libmvf_host.so")
    # bound to each other: a HIP runtime in the process (torch's) has the same names
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-w", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", f"-I{ROOT}/include", f"-I{CSRC}", os.path.join(CSRC, "mvf_runtime.cpp"),
                    os.path.join(ROOT, "tests", "native", "host_hip.cpp"), "-o", so, "-lpthread"], check=True)
    lib = C.CDLL(so)
    for name, args in L.SIGNATURES.items():
        getattr(lib, name).argtypes = args
        getattr(lib, name).restype = C.c_int32
    lib.mvf_last_error.restype = C.c_char_p
    lib.t_elsewhere.restype = lib.t_unordered.restype = lib.t_stale.restype = C.c_char_p
    lib.t_fail.argtypes = [C.c_char_p]
    lib.t_stream.restype = C.c_void_p
    return lib


class Map:
    """A context on a device, with volumes of 16^3 of one stream in front of the camera and a frame on the host."""

    def __init__(self, lib, device=0, volumes=1, width=32, height=24):
        self.lib, self.h = lib, C.c_void_p()
        self.ok("mvf_create", C.byref(self.h), C.byref(L.mvf_config(0, 0.5, 10.0, device, 0)), ctx=False)
        gid = C.c_int32()
        self.ok("mvf_grid_create", C.byref(L.mvf_grid_desc((C.c_float * 3)(-0.8, -0.8, 1.0), 0.1, 4.0, 128, 0)), C.byref(gid))
        self.stream, self.ids = None, []
        for i in range(volumes):
            vid = C.c_int32()
            d = L.mvf_volume_desc(gid.value, (C.c_int32 * 3)(0, 0, 16 * i), (C.c_int32 * 3)(16, 16, 16), 0)
            self.ok("mvf_volume_create", C.byref(d), C.byref(vid))
            self.ok("mvf_volume_place", vid)
            self.ids.append(vid.value)
        self.pose = (C.c_float * 12)(1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 1, 0)
        self.K = L.mvf_intrinsics(30.0, 30.0, (width - 1) / 2, (height - 1) / 2)
        self.size(width, height)

    def size(self, width, height, out=None):
        ow, oh = out or (width, height)
        self.depth = np.ones((height, width), np.float32)
        self.maps = [np.zeros((oh, ow), np.float32), np.zeros((oh, ow, 3), np.float32), np.zeros((oh, ow, 3), np.float32),
                     np.zeros((oh, ow), np.int32)]
        self.frame = L.mvf_frame(self.depth.ctypes.data, None, width, height, 0, 0)
        self.out = L.mvf_raycast_out(*[m.ctypes.data for m in self.maps], ow, oh)

    def ok(self, name, *args, ctx=True):
        st = getattr(self.lib, name)(*([self.h] if ctx else []), *args)
        assert st == 0, (name, st, self.lib.mvf_last_error())

    def step(self):
        fr = L.mvf_stream_frame(0, self.frame, self.pose, self.K)
        self.ok("mvf_step", 1, C.byref(fr), C.byref(self.out), self.stream)

    def close(self):
        self.ok("mvf_destroy")


CALLS = {
    "integrate": lambda m: m.ok("mvf_integrate", 0, C.byref(m.frame), m.pose, C.byref(m.K), m.stream),
    "raycast": lambda m: m.ok("mvf_raycast", 0, m.pose, C.byref(m.K), C.byref(m.out), m.stream),
    "step": lambda m: m.step(),
    "evict": lambda m: m.ok("mvf_volume_evict", m.ids[0], L.MVF_EVICT_SWAP_OUT),
    "swap_out": lambda m: m.ok("mvf_volume_swap_out", m.ids[0], m.stream),
    "swap_in": lambda m: (m.ok("mvf_volume_swap_out", m.ids[0], m.stream), m.lib.t_set_device(0),
                          m.ok("mvf_volume_swap_in", m.ids[0], m.stream)),
    "extract": lambda m: m.ok("mvf_volume_extract", m.ids[0], None, None, None, 0, C.byref(C.c_int64()), m.stream),
    "read": lambda m: m.ok("mvf_volume_read", m.ids[0], m.maps[0].ctypes.data, None, None),
    "write": lambda m: m.ok("mvf_volume_write", m.ids[0], None, None, None),
}


@pytest.mark.parametrize("call", CALLS)
def test_calls_select_their_device(lib, call):
    """A context on the second device, called by a thread whose current device
    is the first: everything that the call allocates or launches is on the
    context's device."""
    m = Map(lib, device=1)
    m.size(128, 96)   # the read's plane of 16^3 fits a map
    CALLS["integrate"](m)
    lib.t_expect(1)
    lib.t_set_device(0)
    CALLS[call](m)
    elsewhere = lib.t_elsewhere().decode()
    lib.t_expect(-1)
    m.close()
    assert elsewhere == "", elsewhere


@pytest.mark.parametrize("call", ["integrate", "raycast", "step", "extract"])
def test_first_call_on_a_stream(lib, call):
    """A new context's first call of each kind on a non-blocking stream: nothing
    that it launches is left unordered with the clearing of new memory, in
    the call or in a next one on another stream."""
    m = Map(lib, volumes=3)
    streams = [lib.t_stream() for _ in range(2)]
    lib.t_watch()
    for m.stream in streams:
        CALLS[call](m)
    unordered = lib.t_unordered().decode()
    m.close()
    assert unordered == "", unordered


def test_clears_of_a_call_that_fails(lib):
    """A call that clears new memory and then fails (a budget below its volume):
    the next call, on another stream, runs after the clear."""
    m = Map(lib)
    a, b = lib.t_stream(), lib.t_stream()
    for call in ("integrate", "step"):
        m.ok("mvf_set_budget", 1000)
        lib.t_watch()
        m.stream = a
        with pytest.raises(AssertionError):
            CALLS[call](m)
        m.ok("mvf_set_budget", 0)
        m.stream = b
        CALLS[call](m)
        assert lib.t_unordered().decode() == ""
    m.close()


def test_step_buffers_are_kept(lib):
    """A batched step's buffers depend on its outputs' sizes and its volumes:
    another schedule allocates nothing, and other input frames only what a plain
    integration does."""
    m, plain = Map(lib, volumes=3), Map(lib, volumes=3)
    m.step()
    before = lib.t_allocs()
    for z, persistent, lanes in ((2, 0, 4), (8, 1, 2), (4, 1, 8), (4, 0, 4)):
        m.ok("mvf_set_schedule", C.byref(L.mvf_schedule(z, persistent, lanes, 0)))
        m.step()
        assert lib.t_allocs() == before, (z, persistent, lanes)
    CALLS["integrate"](plain)
    for width, height in ((48, 40), (40, 48), (16, 8)):
        counts = []
        for x, call in ((plain, CALLS["integrate"]), (m, CALLS["step"])):
            x.size(width, height, out=(32, 24))
            before = lib.t_allocs()
            call(x)
            counts.append(lib.t_allocs() - before)
        assert counts[0] == counts[1], (width, height)
    for x in (m, plain):
        x.close()


@pytest.mark.parametrize("steps", [1, 2, 3, 4, 5])
def test_calls_run_in_order_on_any_stream(lib, steps):
    """Batched steps, whose table slots are released in fours, between the other
    calls, dealt over three streams and the null stream, over more calls than
    there are slots: everything launched runs after everything before it."""
    m = Map(lib, volumes=3)
    streams = [lib.t_stream() for _ in range(3)] + [None]
    lib.t_watch()
    for i in range(16):
        m.stream = streams[i % 3]
        for _ in range(steps):
            m.step()
        for j, call in enumerate(("integrate", "raycast", "extract", "raycast", "step", "integrate")):
            m.stream = streams[(2 * i + j) % 4]
            CALLS[call](m)
    assert lib.t_unordered().decode() == ""
    m.close()


LAUNCHES = {"integrate": ["frame_prep", "ztable", "integrate", "brick_distance", "volume_init", "fill"],
            "raycast": ["hipMemcpyAsync", "ray_bounds_collect", "ray_bounds_merge", "raycast"],
            "step": ["frame_prep", "ztable", "integrate", "brick_distance", "ray_bounds_merge", "raycast"]}


@pytest.mark.parametrize("call,launch", [(c, n) for c, ns in LAUNCHES.items() for n in ns])
def test_after_a_call_that_fails(lib, call, launch):
    """A call of which one launch fails, in a new context and in one in use: the
    next ones, on another stream, run after what it launched, append to counts
    that are zero, and raycast in an order that has been made."""
    a, b = lib.t_stream(), lib.t_stream()
    for before in ((), ("integrate", "raycast", "step"), ("raycast", "integrate")):
        m = Map(lib, volumes=3)
        for m.stream in (a, b):
            for c in before:
                CALLS[c](m)
        m.stream = a
        lib.t_watch()
        lib.t_fail(launch.encode())
        try:
            CALLS[call](m)
            assert not lib.t_failed()   # nothing of that name was launched (an initialised volume, no new memory)
            lib.t_fail(b"")
        except AssertionError:
            assert lib.t_failed()
        m.stream = b
        for c in ("raycast", "integrate", "step", "integrate", "raycast", "raycast", "step"):
            CALLS[c](m)
        assert (lib.t_stale().decode(), lib.t_unordered().decode()) == ("", ""), before
        m.close()


def test_after_launch_tables_overflow(lib):
    """An integration into more volumes than a table slot holds is refused; the
    next one, with fewer, appends to lists whose counts are zero."""
    m = Map(lib, volumes=0)
    gid = C.c_int32()
    m.ok("mvf_grid_create", C.byref(L.mvf_grid_desc((C.c_float * 3)(-2.048, -2.048, 1.0), 0.002, 4.0, 128, 0)), C.byref(gid))

    def volume(offset, dims):
        vid = C.c_int32()
        d = L.mvf_volume_desc(gid.value, (C.c_int32 * 3)(*offset), (C.c_int32 * 3)(*dims), 0)
        m.ok("mvf_volume_create", C.byref(d), C.byref(vid))
        m.ok("mvf_volume_place", vid)
        return vid.value

    volume((0, 0, 0), (2048, 2048, 100))   # a launch's work items alone
    small = [volume((1000 + i % 64, 1000 + i // 64, 120), (2, 2, 2)) for i in range(6000)]
    for _ in range(2):
        lib.t_watch()
        with pytest.raises(AssertionError):
            CALLS["integrate"](m)
        for v in small:
            m.ok("mvf_volume_evict", v, 0)
        for _ in range(3):
            CALLS["integrate"](m)
        assert lib.t_stale().decode() == ""
        for v in small:
            m.ok("mvf_volume_place", v)
    m.close()
