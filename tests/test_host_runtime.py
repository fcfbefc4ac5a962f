"""What the host library asks of the HIP runtime, on the CPU.

The built library runs in a child process against a stand-in for the runtime
(tests/native/hip_stand_in.cpp) that logs launches, allocations and waits instead of doing
them and can refuse a call.  So the order of launches and waits, the launches of a step
request and the answers to a full device are checked without a GPU.
"""

import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes, os, sys
import numpy as np
sys.modules["torch"] = None  # the library must bind to the stand-in, not to torch's runtime
hip = ctypes.CDLL({stand_in!r}, mode=ctypes.RTLD_GLOBAL)
hip.stand_in_log.restype = ctypes.c_char_p
hip.stand_in_live.restype = ctypes.c_int64
hip.stand_in_limit.argtypes = [ctypes.c_int64]
THEN = ctypes.CFUNCTYPE(None)
hip.stand_in_at_launch.argtypes = [ctypes.c_char_p, ctypes.c_int, THEN]
import workloads as wl
from paper_1906_11925_amd import lib as L
from paper_1906_11925_amd.lb import _desc, links
lib = L.load(build_if_missing=False)

def create(nbr, tau, stream=None, **kw):
    d, keep = _desc(nbr, tau, stream_ptr=stream, **kw)
    h = ctypes.c_void_p()
    L.check(lib.hemelb_lb_create(ctypes.byref(h), ctypes.byref(d)))
    return h

def vessel(g, stream=None, lattice=15, **kw):
    coords, nbr = links(g.labels, g.shape, g.periodic, lattice)
    return create(nbr, g.tau, stream, lattice=lattice, coords=coords, iolets=list(g.iolets),
                  site_weight=g.site_weight(), **kw)

def events():
    return hip.stand_in_log().decode().splitlines()

def launches(name):
    return [k for k, e in enumerate(events()) if e.startswith("launch") and name in e]

def info(h):
    i = L.InfoT()
    L.check(lib.hemelb_lb_info(h, ctypes.byref(i)))
    return i
"""


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory, lib):
    out = str(tmp_path_factory.mktemp("hip") / "libhip_stand_in.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-std=c++17", "-Wall", "-o", out,
                    os.path.join(ROOT, "tests", "native", "hip_stand_in.cpp")], check=True)
    return out


def _run(stand_in, code, **env):
    e = {k: v for k, v in os.environ.items() if not k.startswith("HEMELB_")}
    e.update(env)
    res = subprocess.run([sys.executable, "-c", PRELUDE.format(stand_in=stand_in) + textwrap.dedent(code)],
                         cwd=ROOT, env=e, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]
    return res.stdout


def test_set_objective_returns_with_its_tables_laid_out(stand_in):
    """Later work may go to another stream, so nothing of the call may still be queued."""
    _run(stand_in, """
        g = wl.pipe()
        h = vessel(g, stream=0x10)
        hip.stand_in_clear()
        dome = np.ones(g.n_sites, dtype=np.uint8)
        o = L.ObjectiveT(outlet=1, q_target=0.1, dome=dome.ctypes.data_as(L.P(ctypes.c_uint8)),
                         lam=1.0, t0=0, t1=4)
        L.check(lib.hemelb_lb_set_objective(h, ctypes.byref(o)))
        last = launches("k_objective_tables")[-1]
        assert events()[last].endswith(" 16")
        assert "sync 16" in events()[last + 1:], events()
    """)


def test_a_later_handle_leaves_the_lds_limit_of_an_earlier_one(stand_in):
    """The limit on dynamic LDS is the kernel's, for every handle that uses it."""
    _run(stand_in, """
        limits = []
        for g in (wl.pipe(X=23, Y=21, Z=37, r2=97.0), wl.closed_box(X=3, Y=5, Z=2)):
            hip.stand_in_clear()
            vessel(g)
            limits.append([int(e.split()[-2]) for e in events() if e.startswith("attribute")])
        first, second = limits
        assert first and second and min(second) >= max(first), limits
    """, HEMELB_FUSE="3,1,512,1")


def test_calls_on_the_default_stream_do_not_ask_whether_it_is_captured(stand_in):
    """The runtime answers that with an error while a blocking stream is being captured."""
    _run(stand_in, """
        g = wl.pipe()
        h = vessel(g)
        hip.stand_in_null_capture(906)  # hipErrorStreamCaptureImplicit
        buf = np.zeros((15, g.n_sites), dtype=np.float32)
        p = ctypes.c_void_p(buf.ctypes.data)
        t = ctypes.c_int64(0)
        L.check(lib.hemelb_lb_step(h, 5))
        L.check(lib.hemelb_lb_observables(h, p, None, None))
        L.check(lib.hemelb_lb_get_state(h, p, ctypes.byref(t)))
        L.check(lib.hemelb_lb_set_state(h, p, 0))
        assert t.value == 5
    """)


def test_a_device_without_room_for_several_steps_per_launch(stand_in):
    """Their third population buffer and groups are an extra: a handle that fits without
    them is created, steps one by one and takes what it takes without them."""
    _run(stand_in, """
        g = wl.pipe()
        os.environ["HEMELB_FUSE"] = "0"
        h = vessel(g)
        need = info(h).device_bytes
        assert need == hip.stand_in_live()
        L.check(lib.hemelb_lb_destroy(h))
        del os.environ["HEMELB_FUSE"]
        h = vessel(g)
        full = info(h).device_bytes
        assert full == hip.stand_in_live()
        L.check(lib.hemelb_lb_destroy(h))
        assert hip.stand_in_live() == 0 and full > need
        for limit in (need, need + (full - need) // 2, full - 1, full):
            hip.stand_in_limit(limit)
            h = vessel(g)
            fused = limit == full
            assert info(h).device_bytes == hip.stand_in_live() == (full if fused else need)
            hip.stand_in_clear()
            hip.stand_in_limit(2 * full)  # the first step makes its table of iolet values
            L.check(lib.hemelb_lb_step(h, 6))
            assert len(launches("k_fused_steps")) == (2 if fused else 0)
            assert len(launches("k_stream_collide")) == (0 if fused else 6)
            L.check(lib.hemelb_lb_destroy(h))
            assert hip.stand_in_live() == 0
    """)


@pytest.mark.parametrize("form,singles", [("0", 12), ("2,1,512,0", 0), ("3,1,512,1", 0)])
def test_launches_of_a_step_request(stand_in, form, singles):
    _run(stand_in, f"""
        h = vessel(wl.pipe())
        L.check(lib.hemelb_lb_step(h, 12))
        steps = int(os.environ["HEMELB_FUSE"][0])
        assert len(launches("k_stream_collide")) == {singles}
        assert len(launches("k_fused_steps")) == (12 // steps if steps else 0)
    """, HEMELB_FUSE=form)


@pytest.mark.parametrize("form", ["2,1,512,0", "3,1,512,1"])
@pytest.mark.parametrize("after", [1, 2, 5])
def test_cancel_between_launches_of_several_steps(stand_in, form, after):
    """A launch that another was to follow keeps no state before its last step, so a request
    that is cancelled behind it makes one more, single step: the outputs need that state."""
    _run(stand_in, f"""
        steps = int(os.environ["HEMELB_FUSE"][0])
        h = vessel(wl.pipe())
        cancel = THEN(lambda: lib.hemelb_lb_cancel(h) and None)
        hip.stand_in_at_launch(b"k_fused_steps", {after}, cancel)
        rc = lib.hemelb_lb_step(h, 20)
        assert rc == L.HEMELB_ECANCELLED, L.last_error()
        assert len(launches("k_fused_steps")) == {after} and len(launches("k_stream_collide")) == 1
        assert launches("k_stream_collide")[0] > launches("k_fused_steps")[-1]
        assert info(h).time == {after} * steps + 1
        assert f"cancelled after {{info(h).time}} of 20" in L.last_error()
        L.check(lib.hemelb_lb_step(h, steps))
        assert info(h).time == {after} * steps + 1 + steps
        # behind the last launch of a request nothing is missing
        hip.stand_in_clear()
        hip.stand_in_at_launch(b"k_fused_steps", 1, cancel)
        assert lib.hemelb_lb_step(h, steps) == 0
        assert lib.hemelb_lb_step(h, 1) == L.HEMELB_ECANCELLED
        assert not launches("k_stream_collide")
    """, HEMELB_FUSE=form)


@pytest.mark.parametrize("dim", [(1, 1, 1), (1, 1, 257), (2, 4097, (1 << 19) + 1),
                                 (1291, 1291, 1291), (1, 1, (1 << 31) - 1), (2, 2, (1 << 31) - 1)])
def test_distance_maps_of_more_cells_than_one_launch_dimension_takes(stand_in, dim):
    """A flat vessel's map may pass 2^32 cells (a bounding box may have 2^31 blocks, the map
    of reach one more along each axis); every cell gets a thread of each of the three passes."""
    out = _run(stand_in, f"""
        hip.stand_in_threads.restype = ctypes.c_uint64
        far = lib._ZN3hlb17launch_render_farEPKiPKhRA3_S0_PhS6_P12ihipStream_t
        null = ctypes.c_void_p(None)
        assert far(null, null, (ctypes.c_int32 * 3){dim}, null, null, null) == 0
        cells = {dim[0]} * {dim[1]} * {dim[2]}
        assert len(launches("k_far")) == 3
        assert cells <= hip.stand_in_threads() < cells + cells // 1024 + 256 + 256 * 1024
    """)
    assert out == ""
