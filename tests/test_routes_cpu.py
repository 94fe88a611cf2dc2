"""What the host side of libhough.so asks of the device, without one: a HIP runtime that runs nothing
(fake_hip.cpp) is loaded ahead of the library in a process of its own and writes down the kernels that
would be launched, in order, with the clears and waits between them."""
import json
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2607_04067_amd", "libhough.so")

PRELUDE = r"""
import ctypes, json, re, sys
FAKE = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
FAKE.fake_journal.restype = ctypes.c_char_p
L = ctypes.CDLL(sys.argv[2])
vp, i32, u32, f64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_uint32, ctypes.c_double
PERIODIC, DEDUP = 1, 2

class Params(ctypes.Structure):
    _fields_ = [("n_theta", i32), ("n_rho", i32), ("rho_min", f64), ("rho_max", f64), ("acc_type", i32),
                ("threshold", i32), ("rho_window", i32), ("max_peaks", i32), ("flags", i32), ("reserved", i32)]

class Plan(ctypes.Structure):
    _fields_ = [("waves", i32), ("groups", i32), ("per_cu", i32), ("lds", i32), ("window", i32)]

L.hough_split_workspace_bytes.restype = ctypes.c_size_t
L.hough_split_workspace_bytes.argtypes = [vp, u32]
X = vp(1 << 20)                                  # stands for a device array

def context(n_theta, n_rho, flags=0):
    c = vp()
    p = Params(n_theta, n_rho, -0.01, 0.01, 2, 10, 1, 64, flags, 0)
    rc = L.hough_config(ctypes.byref(p), ctypes.byref(c))
    assert rc == 0, rc
    return c

def plan(c):
    p = Plan()
    assert L.hough_get_batch_plan(c, ctypes.byref(p)) == 0
    return p.waves, p.groups, p.per_cu, p.window

def journal(call):
    # the call's status and what it asked for: kernels as name<template arguments>
    FAKE.fake_clear()
    rc = call()
    out = []
    for line in FAKE.fake_journal().decode().splitlines():
        w = line.split()
        if w[0] == "launch":
            name, args = re.search(r"\d(k_[a-z_0-9]+?)(?:I((?:L[ib]\d+E)+)|E)", w[1]).groups()
            out.append(name + ("<" + ",".join(re.findall(r"L[ib](\d+)E", args)) + ">" if args else ""))
        else:
            out.append(line)
    return rc, out

def batch(c, n):
    return journal(lambda: L.hough_run_batch(c, X, X, X, n, X, X, X, X, None))

def split(c, n, workspace=None, size=0, static=False):
    if static:
        return journal(lambda: L.hough_run_batch_split_static(c, X, X, X, None, None, n, X, X, X, X, None))
    return journal(lambda: L.hough_run_batch_split(c, X, X, X, None, None, n, X, X, X, X, workspace,
                                                   ctypes.c_size_t(size), None))
"""

SERVE = r"""
class Pool(ctypes.Structure):
    _fields_ = [("ctx", vp), ("x", vp), ("y", vp), ("offsets", vp), ("host_offsets", vp), ("n_events", u32),
                ("reserved", u32), ("host_x", vp), ("host_y", vp)]

class Config(ctypes.Structure):
    _fields_ = [("n_streams", i32), ("max_batch_events", i32), ("max_batch_hits", i32), ("plain", i32),
                ("copy_peaks", i32), ("small_batch_events", i32), ("split_batch_events", i32), ("reserved", i32),
                ("max_wait_us", f64)]

class Request(ctypes.Structure):
    _fields_ = [("arrival_us", f64), ("kind", i32), ("event", u32)]

class Result(ctypes.Structure):
    _fields_ = [("launch_us", f64), ("done_us", f64), ("n_peaks", u32), ("status", u32), ("batch_events", u32),
                ("slot", u32)]

def serve(c, n, small=64, split=16, streams=1):
    # n events that arrive together, as one batch
    off = (u32 * (n + 1))(*range(0, 3 * n + 1, 3))
    pool = (Pool * 1)(Pool(c, X, X, X, ctypes.cast(off, vp), n, 0, None, None))
    cfg = Config(streams, 4096, 1 << 16, 0, 0, small, split, 0, 0.0)
    req = (Request * n)(*[Request(0.0, 0, i) for i in range(n)])
    res = (Result * n)()
    rc, out = journal(lambda: L.hough_serve_run(pool, 1, ctypes.byref(cfg), req, u32(n), res, None, None, u32(0)))
    return rc, out, max(r.batch_events for r in res)
"""


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    if not os.path.exists(LIB):
        from paper_2607_04067_amd import build
        build.build()
    cxx = shutil.which("g++")
    assert cxx, "g++ not found"
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    fake = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run([cxx, "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                    "-I" + os.path.join(rocm, "include"), os.path.join(HERE, "fake_hip.cpp"), "-o", fake], check=True)

    def run(body: str, **values):
        """The value of `out` after `body`, run with the names of PRELUDE, SERVE and `values`."""
        code = PRELUDE + SERVE + "".join(f"{k} = {v!r}\n" for k, v in values.items()) + body
        code += "\nprint('OUT ' + json.dumps(out))\n"
        r = subprocess.run([sys.executable, "-c", code, fake, LIB], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr[-2000:]
        return json.loads([ln for ln in r.stdout.splitlines() if ln.startswith("OUT ")][-1][4:])

    return run


def test_zeros_are_in_place_before_a_kernel_can_read_them(routes):
    """The split form waits for slots that start at zero, so a context's are cleared and waited for in
    hough_config (its caller may launch on any stream), and a serving slot's workspace is cleared on
    the stream its launches go to."""
    log = routes("out = journal(lambda: context(360, 256) and 0)[1]")
    writes = [i for i, s in enumerate(log) if s in ("clear stream 0", "copy stream 0")]
    assert writes and "wait stream 0" in log[writes[-1]:]
    rc, log, n = routes("out = serve(context(360, 256), 4, streams=2)")
    assert rc == 0 and n == 4
    own = [s for s in log if s.startswith("clear stream")]
    assert "clear stream 1" in own and "clear stream 2" in own
    # a clear on the null stream is waited for before the first launch
    first = next(i for i, s in enumerate(log) if s.startswith("k_batch"))
    late = [i for i, s in enumerate(log[:first]) if s == "clear stream 0"]
    assert all("wait stream 0" in log[i:first] for i in late)


def test_serving_keeps_the_shapes_of_a_pool_nobody_tuned(routes):
    """A pool's context reports whole columns where its large batches take windows first: its serving
    copies run the same kernels, with one context per stream.  A shape its caller has set is copied;
    small batches keep the library's own shapes either way."""
    rc, alone = routes("out = batch(context(1000, 1000), 600)")
    assert rc == 0 and alone == ["k_order", "k_batch<8,1,0,1,1>", "k_batch<16,1,0,1,0>", "k_spill"]
    rc, log, n = routes("out = serve(context(1000, 1000), 600, split=0)")
    assert rc == 0 and n == 600
    # (a gathered batch keeps the caller's order)
    assert [s for s in log if s.startswith("k_")] == alone[1:]
    blocks = [s for s in log if s.startswith("malloc") and int(s.split()[1]) > 32 << 20]
    assert len(blocks) == 1
    rc, log, n = routes("""
c = context(1000, 1000)
assert L.hough_set_batch_plan(c, 12, 1, 1) == 0
out = serve(c, 600)""")
    assert rc == 0 and [s for s in log if s.startswith("k_")] == ["k_batch<12,1,0,1,0>", "k_spill"]
    for small, want in ((64, ["k_batch_split<16,0,0>", "k_spill"]), (1000, ["k_batch<16,1,0,0,0>", "k_spill"])):
        rc, log, n = routes("""
c = context(360, 256)
assert L.hough_set_batch_plan(c, 12, 1, 1) == 0
out = serve(c, n, small, 0)""", n=40 if small == 64 else 300, small=small)
        assert rc == 0 and [s for s in log if s.startswith("k_")] == want


# (n_theta, n_rho, flags, shape to set or None, events, kernels)
BATCH_ROUTES = [
    (360, 256, 0, None, 1, ["k_batch_split<16,0,0>", "k_spill"]),
    (360, 256, 0, None, 192, ["k_batch_split<8,0,0>", "k_spill"]),
    (360, 256, 0, None, 193, ["k_batch<8,1,0,0,0>", "k_spill"]),
    (360, 256, 0, None, 5000, ["k_order", "k_batch<8,1,0,0,0>", "k_spill"]),
    (720, 512, 0, None, 129, ["k_batch<12,1,0,0,0>", "k_spill"]),
    (1000, 2000, "PERIODIC", None, 64, ["k_batch_split<16,1,1>", "k_spill"]),
    (1000, 2000, "DEDUP", None, 64, ["k_dedup", "k_batch<16,1,0,1,1>", "k_spill"]),
    # windows from five theta tiles on
    (248, 700, 0, None, 600, ["k_order", "k_batch<16,1,0,0,0>", "k_spill"]),
    (249, 700, 0, None, 600, ["k_order", "k_batch<8,1,0,0,1>", "k_batch<16,1,0,0,0>", "k_spill"]),
    (249, 700, "PERIODIC", None, 600, ["k_order", "k_batch<8,1,1,0,1>", "k_batch<16,1,1,0,0>", "k_spill"]),
    # a shape the caller has set runs every batch, small ones too
    (360, 256, 0, (4, 2, 0), 1, ["k_batch<4,2,0,0,0>", "k_spill"]),
    (360, 256, 0, (6, 1, 3), 16, ["k_batch<6,1,0,0,0>", "k_spill"]),
    (360, 256, "PERIODIC", (12, 1, 0), 16, ["k_batch<12,1,1,0,0>", "k_spill"]),
    (360, 256, "DEDUP", (8, 1, 4), 100, ["k_dedup", "k_batch<8,1,0,0,0>", "k_spill"]),
    (720, 512, 0, (16, 2, 0), 40, ["k_batch<16,2,0,0,0>", "k_spill"]),
    (1000, 1000, 0, (8, 1, 2), 20, ["k_batch<8,1,0,1,1>", "k_spill"]),
    (1000, 1000, 0, (16, 1, 1), 600, ["k_order", "k_batch<16,1,0,1,0>", "k_spill"]),
    (1000, 2000, 0, (8, 1, 0), 20, ["k_batch<8,1,0,1,1>", "k_spill"]),
]


@pytest.mark.parametrize("n_theta,n_rho,flags,shape,events,kernels", BATCH_ROUTES)
def test_batch_routes(routes, n_theta, n_rho, flags, shape, events, kernels):
    rc, log = routes(f"""
c = context(n_theta, n_rho, {flags})
if shape: assert L.hough_set_batch_plan(c, *shape) == 0
out = batch(c, events)""", n_theta=n_theta, n_rho=n_rho, shape=shape, events=events)
    assert rc == 0 and log == kernels


def test_a_refused_shape_leaves_the_routes_alone(routes):
    out = routes("""
c = context(360, 256)
rc = L.hough_set_batch_plan(c, 5, 1, 0), L.hough_set_batch_plan(c, 8, 1, 90)
out = [rc, plan(c), batch(c, 16)]""")
    assert out[0] == [-1, -1] and out[1] == [8, 1, 4, 0] and out[2] == [0, ["k_batch_split<16,0,0>", "k_spill"]]


def test_the_latency_form_runs_by_tile_whatever_the_shape(routes):
    rc, log = routes("""
c = context(1000, 2000)
assert L.hough_set_batch_plan(c, 8, 1, 0) == 0
out = split(c, 16)""")
    assert rc == 0 and log == ["k_batch_split<16,0,1>", "k_spill"]


@pytest.mark.parametrize("flags", ["0", "PERIODIC"])
@pytest.mark.parametrize("n_rho,has", [(1109, True), (1110, False), (1120, False), (1121, False)])
def test_split_calls_on_tall_grids_need_no_workspace(routes, n_rho, has, flags):
    """Above 1,109 rows the latency form takes no workspace, and its static form any batch."""
    size, few, many, static = routes(f"""
c = context(130, n_rho, {flags})
out = [L.hough_split_workspace_bytes(c, 16), split(c, 16), split(c, 1000), split(c, 5000, static=True)]""", n_rho=n_rho)
    if has:
        assert size > 0 and few[0] == many[0] == -1 and static == [-5, []]
    else:
        assert size == 0 and few[0] == many[0] == static[0] == 0
        assert few[1][0].startswith("k_batch_split<16,") and any(s.startswith("k_batch<") for s in static[1])


def test_a_context_does_without_the_room_for_mapped_hits(routes):
    """Where the device cannot spare the 32 MiB a context is made without them (and batches run); where
    it cannot spare the rest either, none is."""
    out = routes("""
FAKE.fake_largest_malloc(ctypes.c_size_t(32 << 20))
out = [batch(context(360, 256), 1000)]
FAKE.fake_largest_malloc(ctypes.c_size_t(4096))
p, c = Params(360, 256, -0.01, 0.01, 2, 10, 1, 64, 0, 0), vp()
out.append([L.hough_config(ctypes.byref(p), ctypes.byref(c)), c.value])""")
    assert out[0] == [0, ["k_batch<8,1,0,0,0>", "k_spill"]] and out[1] == [-2, None]


@pytest.mark.parametrize("hits,waves", [(1, 16), (64 * 256, 16), (64 * 256 + 1, 8), (64 * 512 + 1, 4), (64 * 1024, 4),
                                        (64 * 1024 + 1, 2), (64 * 2048 + 1, 1), (10**6, 1), (2**32 - 1, 1)])
def test_retention_of_one_event_fills_the_chip(routes, hits, waves):
    """The waves that share 64 hits, by the hits per CU (256 of them here)."""
    out = routes("out = journal(lambda: L.hough_retain(context(720, 512), X, X, u32(hits), X, X, u32(99999), X, None))",
                 hits=hits)
    assert out[0] == 0 and out[1][-1] == f"k_retain<{waves}>"
