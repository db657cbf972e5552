"""The library's host side over a stand-in HIP runtime (hip_stub.cpp, preloaded
into a child process): in which order a handle lets go of what its graphs were
captured through, and what a handle holds after a capture that failed.  No
kernel runs."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

CHILD = r"""
import ctypes, sys, types
import numpy as np
sys.modules["torch"] = types.ModuleType("torch")     # the binding only loads its HIP runtime
from paper_1709_00821_amd import _lib as L, workloads as W
from paper_1709_00821_amd.plasma import make_desc
from paper_1709_00821_amd.plasma2d import make_desc2
lib, stub, STREAM = L.lib(), ctypes.CDLL(sys.argv[1]), 64     # any stream but the null one
stub.stub_waits.restype = stub.stub_launches.restype = stub.stub_bad_grids.restype = ctypes.c_long

def long_1d(**kw):
    p = W.slab_c1(n=300000, slab=(100000, 200000), src=5000, probes=(3000, 250000), n_freqs=4)
    d, keep = make_desc(p, "f64", "tiled", stream_handle=STREAM, **kw)
    h = ctypes.c_void_p()
    L.check(lib.fdtd_plasma_create(ctypes.byref(d), None, 0, ctypes.byref(h)))
    return h

def grid_2d():
    p = W.cylinder_2d("tm", n=400, steps=10)
    d, keep = make_desc2(p, "f64", STREAM)
    h = ctypes.c_void_p()
    L.check2(lib.fdtd2d_create(ctypes.byref(d), None, 0, ctypes.byref(h)))
    return h

def done(h, fn):
    v = ctypes.c_int64()
    assert fn(h, ctypes.byref(v)) == 0
    return v.value
"""

ORDER = CHILD + r"""
for make, run, destroy in ((long_1d, lib.fdtd_plasma_run, lib.fdtd_plasma_destroy),
                           (grid_2d, lib.fdtd2d_run, lib.fdtd2d_destroy)):
    h = make()
    for T in (100, 130, 100):
        assert run(h, T) == 0
    assert stub.stub_live() == 5              # a side stream, two events, two graphs
    assert destroy(h) == 0
    assert stub.stub_live() == 0 and stub.stub_misuses() == 0, stub.stub_misuses()
assert stub.stub_waits() > 0 and stub.stub_bad_grids() == 0
"""

FAILED = CHILD + r"""
what = sys.argv[2]
for make, run, step, count, destroy in (
        (lambda: long_1d(checkpoint=200), lib.fdtd_plasma_run, lib.fdtd_plasma_step, lib.fdtd_plasma_steps_done,
         lib.fdtd_plasma_destroy),
        (grid_2d, lib.fdtd2d_run, lib.fdtd2d_step, lib.fdtd2d_steps_done, lib.fdtd2d_destroy)):
    h = make()
    assert step(h, 20) == 0
    before = stub.stub_launches()
    assert step(h, 20) == 0
    pass_ = stub.stub_launches() - before     # the launches of 20 steps inside a sample window
    if what == "hipGraphLaunch":
        assert run(h, 100) == 0               # a graph that is there already
        assert run(h, 40) == 0
    stub.stub_fail(what.encode())
    assert run(h, 100) == L.E_DEVICE
    assert done(h, count) == 40               # nothing ran: the state is the one before
    before = stub.stub_launches()
    assert step(h, 20) == 0
    assert stub.stub_launches() - before == pass_, "the step of a run that failed"
    assert run(h, 100) == 0 and done(h, count) == 100
    assert run(h, 7) == 0 and done(h, count) == 7
    destroy(h)
    assert stub.stub_live() == 0 and stub.stub_misuses() == 0
"""

EVENTS = CHILD + r"""
what = sys.argv[2]
for make, step, err, destroy in ((long_1d, lib.fdtd_plasma_step, lib.fdtd_plasma_last_error, lib.fdtd_plasma_destroy),
                                 (grid_2d, lib.fdtd2d_step, lib.fdtd2d_last_error, lib.fdtd2d_destroy)):
    h = make()
    assert step(h, 10) == 0
    stub.stub_fail(what.encode())
    assert step(h, 10) == L.E_DEVICE          # launches beside each other without their wait
    assert step(h, 10) == L.E_STATE
    destroy(h)
"""


SIZES = CHILD + r"""
rng = np.random.default_rng(1)
up = lambda b: (max(b, 16) + 255) // 256 * 256
for mode, nx, ny, prec, P, F in (("tm", 40, 50, "f32", 0, 1), ("te", 300, 310, "f64", 9, 64), ("te", 64, 2000, "f32", 4096, 3),
                                 ("tm", 2, 200000, "f64", 2, 16)):
    wp2 = np.zeros((1 if mode == "tm" else 2, nx, ny))
    wp2[:, nx // 3:nx // 2 + 1, 5:ny // 2] = 1e21
    nc, nh, es = len(wp2), 3 - len(wp2), 8 if prec == "f64" else 4
    S = int(np.any(wp2 > 0, axis=0).sum())
    p = W.Problem2D(mode=mode, nx=nx, ny=ny, d=75e-6, dt=1e-13, wp2=wp2, nu=wp2 * 0, src=(1, 1), src_tau=1e-12, src_t0=1e-12,
                    src_amp=1.0, probes=np.stack([rng.integers(0, k, P) for k in (nc, nx, ny)], axis=1), freqs=np.arange(1.0, F + 1))
    d, keep = make_desc2(p, prec, STREAM)
    # one copy of the fields and currents, the plasma, the probes, their window, spectra and twiddles
    enough = ((nc + nh) * up(es * nx * ny) + 2 * up(8 * nx) + 3 * nc * up(8 * S) + up(24 * max(P, 1)) + up(8 * F) +
              up(8 * max(P, 1) * 2048) + 2 * up(16 * max(P, 1) * F) + up(16 * 1024 * F))
    mem = (ctypes.c_char * (enough + 256))()
    at = (ctypes.addressof(mem) + 255) // 256 * 256
    h = ctypes.c_void_p()
    assert lib.fdtd2d_create(ctypes.byref(d), ctypes.c_void_p(at), enough, ctypes.byref(h)) == 0, lib.fdtd2d_last_error()
    assert lib.fdtd2d_run(h, 40) == 0 and lib.fdtd2d_step(h, 9) == 0
    lib.fdtd2d_destroy(h)
    full = ctypes.c_size_t()
    assert lib.fdtd2d_workspace_bytes(ctypes.byref(d), ctypes.byref(full)) == 0
    stub.stub_limit(ctypes.c_long(full.value - 1))     # a card one byte short of two copies
    assert lib.fdtd2d_create(ctypes.byref(d), None, 0, ctypes.byref(h)) == (0 if nx > 3 else L.E_DEVICE)
    stub.stub_limit(ctypes.c_long(0))
    if h: lib.fdtd2d_destroy(h)
assert stub.stub_misuses() == 0 and stub.stub_bad_grids() == 0
"""


KERNELS = CHILD + r"""
stub.stub_launched.restype = ctypes.c_long
def taken(p, prec="f64", exec="tiled", steps=64, **kw):
    d, keep = make_desc(p, prec, exec, stream_handle=STREAM, **kw)
    h = ctypes.c_void_p()
    L.check(lib.fdtd_plasma_create(ctypes.byref(d), None, 0, ctypes.byref(h)))
    stub.stub_forget()
    assert lib.fdtd_plasma_step(h, steps) == 0
    lib.fdtd_plasma_destroy(h)
    return {k: stub.stub_launched(k.encode()) for k in ("k_spanI", "k_groupI", "k_tiledI", "k_step")}

def long_grids(ns, plasma):
    out = []
    for n in ns:
        p = W.large_c2(n=n, n_freqs=3, cpml=8)
        wp2 = np.full(n, p.wp2.max() / 40) if plasma else np.zeros(n)
        wp2[:100] = wp2[-100:] = 0.0
        out.append(p.copy(wp2=wp2, src_cell=n // 2, probes=np.array([n // 2 - 700, n // 2 + 900])))
    return out

# the grids of the span tests become spans beside segments, with 256-node tiles they stay tiles
plasma, vacuum = long_grids((1500007, 1511111, 1489999), True), long_grids((1900001, 1850011, 1799999), False)
for prec, K in (("f64", 64), ("f32", 60)):
    t = taken(plasma, prec, steps=K, tile_cells=512, steps_per_pass=K)
    assert t["k_spanI"] == 1 and t["k_groupI"] == 1, t
    t = taken(vacuum, prec, steps=K, tile_cells=512, vacuum_tile_cells=1024, steps_per_pass=K)
    assert t["k_spanI"] >= 1 and t["k_groupI"] == 1, t
    t = taken(plasma, prec, steps=K, tile_cells=256, steps_per_pass=K)
    assert t["k_spanI"] == 0 and t["k_tiledI"] >= 1, t
# the grids of the group tests: segments alone, or resident; with layers too thick for a segment, tiles
for n in (245, 801, 1569, 2900):
    p = W.random_slab(np.random.default_rng(n), n)
    for ex in ("auto", "tiled", "resident"):
        t = taken(p, exec=ex, steps=48)
        assert t["k_groupI"] == 1 and t["k_tiledI"] == 0, (n, ex, t)
p = W.random_slab(np.random.default_rng(1), 2900, bc="cpml", cpml_cells=120)
t = taken(p)
assert t["k_groupI"] == 0 and t["k_tiledI"] > 0, t
assert taken(p.copy(cpml_cells=6), "f32", steps=48)["k_groupI"] == 1
# a batch whose role tiles fill the GPU keeps them
few, many = ([W.slab_c1(n=2000, slab=(800, 1100), src=200, probes=(100, 1800), n_freqs=2)] * k for k in (300, 900))
assert taken(few, steps=48)["k_groupI"] == 1 and taken(many)["k_groupI"] == 0
"""

STATIC = CHILD + r"""
stub.stub_launched.restype = ctypes.c_long
MB16 = 16 << 20
def plan(ns, fill):                       # fill: the unused table of layers, 32 B a node, to come near the limit
    ps = [W.slab_c1(n=n, slab=(n // 3, n // 2), src=8, probes=(4,), n_freqs=2).copy(cpml_cells=fill) for n in ns]
    d, keep = make_desc(ps, "f64", "tiled", stream_handle=STREAM)
    b = ctypes.c_size_t()
    L.check(lib.fdtd_plasma_workspace_bytes(ctypes.byref(d), ctypes.byref(b)))
    return d, keep, b.value
def kernels(d):
    h = ctypes.c_void_p()
    rc = lib.fdtd_plasma_create_static(ctypes.byref(d), ctypes.byref(h))
    if rc: return rc
    stub.stub_forget()
    assert lib.fdtd_plasma_step(h, 40) == 0
    lib.fdtd_plasma_destroy(h)
    return stub.stub_launched(b"k_groupI"), stub.stub_launched(b"k_tiledI")
# 90 short grids: their segments' table is 90 x 8 bytes longer than the tiles'
ns = [380] * 90
while plan(ns, 1)[2] > MB16 - 200000: ns = [n - 8 for n in ns]
d, keep, b = plan(ns, 1)
assert kernels(d) == (1, 0), (kernels(d), b, ns[0])               # room to spare: segments
fill = 1
for _ in range(2):                        # (the transform's wider scratch space goes first)
    fill += (MB16 - plan(ns, fill)[2]) // 32 + 128
    while plan(ns, fill)[2] > MB16: fill -= 8
d, keep, b = plan(ns, fill)
assert MB16 - 256 < b <= MB16, (b, MB16 - b, fill)
assert kernels(d)[1] > 0 and kernels(d)[0] == 0, (kernels(d), b)     # the tiles' table still fits, the segments' does not: tiles
d, keep, b = plan(ns, fill + 8)
assert b > MB16 and kernels(d) == L.E_WORKSPACE
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = tmp_path_factory.mktemp("stub") / "hip_stub.so"
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-w", os.path.join(HERE, "hip_stub.cpp"), "-o", str(so)], check=True)
    return str(so)


def child(code, stub, *args):
    from paper_1709_00821_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    r = subprocess.run([sys.executable, "-c", code, stub, *args], cwd=ROOT, capture_output=True, text=True,
                       env={**os.environ, "LD_PRELOAD": stub, "PYTHONPATH": ROOT}, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


def test_graphs_go_before_what_they_were_captured_through(stub):
    child(ORDER, stub)


@pytest.mark.parametrize("what", ["hipStreamBeginCapture", "hipStreamEndCapture", "hipGraphInstantiate",
                                  "hipGraphLaunch"])
def test_a_run_that_was_not_captured_leaves_the_state(stub, what):
    child(FAILED, stub, what)


@pytest.mark.parametrize("what", ["hipEventRecord", "hipStreamWaitEvent"])
def test_a_step_whose_streams_did_not_wait_is_reported(stub, what):
    child(EVENTS, stub, what)


def test_the_kernels_a_problem_takes(stub):
    """The bit-for-bit tests of spans and segments compare them with tiles only
    if the problems take them."""
    child(KERNELS, stub)


def test_the_static_workspace_at_its_limit(stub):
    """Where the table of segments would push a problem past the static
    workspace and that of the plain tiles does not, it runs as tiles."""
    child(STATIC, stub)


def test_2d_takes_a_workspace_of_one_copy_of_the_fields(stub):
    child(SIZES, stub)
