"""GPU parity of the 2D Yee-RKETD library (TM and TE) against the 2D oracle
(through the C ABI): FP64 fields and probe spectra within 1e-12 of the
oracle's scale, FP32 storage (FP64 registers, rounded every step) within its
stated error; step composition and graph replay bit for bit."""
import sys
import zlib

import numpy as np
import pytest

import oracle
from paper_1709_00821_amd import workloads as W

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def G():
    import torch
    assert torch.cuda.is_available()
    from paper_1709_00821_amd import plasma2d
    return plasma2d


def rel(a, b, floor=0.0):
    s = max(float(np.max(np.abs(b))), floor)
    return float(np.max(np.abs(a - b)) / s) if s > 0 else float(np.max(np.abs(a)))


def errs(F, o):
    # pulse-scale floors: the source peaks at 1 V/m
    eE = rel(F["E"], o["E"], 1e-2)
    eH = rel(F["H"], o["H"], 1e-2 / 376.73)
    eJ = rel(F["J"], o["J"], 1e-6)
    return eE, eH, eJ


@pytest.mark.parametrize("mode,px,py", [("tm", False, False), ("te", False, False), ("tm", True, False),
                                        ("te", False, True), ("tm", True, True), ("te", True, True)])
def test_random_2d_matches_oracle(G, mode, px, py):
    rng = np.random.default_rng(zlib.crc32(f"{mode}{px}{py}".encode()))
    nx, ny = int(rng.integers(40, 200)), int(rng.integers(40, 200))
    p = W.random_2d(rng, mode, nx, ny, periodic_x=px, periodic_y=py)
    T = 400
    say(f"case 2d {mode} {nx}x{ny} periodic=({px},{py}) steps={T}")
    o = oracle.run2d(p, T)
    for prec, tol in (("f64", 1e-12), ("f32", 2e-5)):
        with G.FdtdPlasma2D(p, precision=prec) as h:
            h.run(T)
            X = h.spectra()
            F = h.fields()
        ex = rel(X, o["X"])
        ef = errs(F, o)
        say(f"2d {mode} {prec}: spectra {ex:.2e} fields E {ef[0]:.2e} H {ef[1]:.2e} J {ef[2]:.2e}")
        assert ex <= tol and max(ef) <= tol * 10, prec
    assert np.max(np.abs(o["J"])) > 0


@pytest.mark.parametrize("mode", ["tm", "te"])
def test_cylinder_2d_matches_oracle(G, mode):
    """The benchmark's plasma-cylinder problem scaled to 192^2 (cylinder radius
    n/8 with its Gaussian edge, PEC walls, soft point source, 8 probes)."""
    p = W.cylinder_2d(mode, n=192, n_freqs=16)
    T = 600
    say(f"case 2d cylinder {mode} n=192 steps={T}")
    o = oracle.run2d(p, T)
    for prec, tol in (("f64", 1e-12), ("f32", 2e-5)):
        with G.FdtdPlasma2D(p, precision=prec) as h:
            h.run(T)
            X = h.spectra()
            F = h.fields()
        ex = rel(X, o["X"])
        ef = errs(F, o)
        say(f"2d cylinder {mode} {prec}: spectra {ex:.2e} fields {max(ef):.2e}")
        assert ex <= tol and max(ef) <= tol * 10, prec


@pytest.mark.parametrize("mode", ["tm", "te"])
@pytest.mark.parametrize("nx,ny,px,py", [(2, 2, True, True), (3, 113, True, False), (16, 112, False, False),
                                         (17, 225, False, True), (33, 49, False, False), (600, 121, True, True),
                                         (1100, 800, False, False)])
def test_tile_edges_match_oracle(G, mode, nx, ny, px, py):
    """Grids at the edges of the register tiles (one output row or column more
    than a tile, grids shorter than the halo on periodic axes, and enough tiles
    for the tall shape), plasma in the middle third of the columns, probes in
    the corners and inside, the source on the last cell a wall allows; a step
    count that is no whole number of passes."""
    rng = np.random.default_rng(zlib.crc32(f"{mode}{nx}{ny}{px}{py}".encode()))
    nc = 1 if mode == "tm" else 2
    dt = 0.5 * 75e-6 / W.C0
    tau, t0, amp = W.pulse_params(dt, 4.0)
    wp2 = np.zeros((nc, nx, ny))
    wp2[:, :, ny // 3:2 * ny // 3 + 1] = rng.uniform(0, (2 * np.pi * 40e9) ** 2, (nc, nx, 2 * ny // 3 + 1 - ny // 3))
    corners = [(i, j) for i in (0, nx // 2, nx - 1) for j in (0, ny // 2, ny - 1)]
    p = W.Problem2D(mode=mode, nx=nx, ny=ny, d=75e-6, dt=dt, wp2=wp2, nu=rng.uniform(1e9, 5e10, (nc, nx, ny)),
                    src=(nx - 1, ny - 1), src_tau=tau, src_t0=t0, src_amp=amp,
                    probes=np.array([(nc - 1, i, j) for i, j in corners], np.int64),
                    freqs=np.linspace(1e9, 1e11, 5), periodic_x=px, periodic_y=py)
    T = 83
    say(f"case 2d tile edges {mode} {nx}x{ny} periodic=({px},{py})")
    o = oracle.run2d(p, T, kind="omp")
    for prec, tol in (("f64", 1e-12), ("f32", 2e-5)):
        with G.FdtdPlasma2D(p, precision=prec) as h:
            h.run(T)
            X, F = h.spectra(), h.fields()
            h.step(5).step(8)               # the other copy of the fields, and a short pass
            G2 = h.fields()
        with G.FdtdPlasma2D(p, precision=prec) as h:
            h.step(T + 13)
            F2 = h.fields()
        assert rel(X, o["X"]) <= tol and max(errs(F, o)) <= tol * 10, prec
        for k in ("E", "H", "J"):
            assert np.array_equal(G2[k], F2[k]), (prec, k)


@pytest.mark.parametrize("mode,nx,ny,px,py", [("tm", 70, 90, False, False), ("te", 97, 130, True, False),
                                              ("te", 820, 1040, False, True)])
def test_2d_dense_probes_match_fields(G, mode, nx, ny, px, py):
    """Probes on every cell of a block (both E components in TE) that crosses
    tiles of plasma and vacuum, waves and lanes, some given twice and in no
    order: after one step their spectra at f = 0 are dt times the E fields, and
    after 21 those of the oracle."""
    rng = np.random.default_rng(nx)
    p = W.random_2d(rng, mode, nx, ny, periodic_x=px, periodic_y=py)
    nc = 1 if mode == "tm" else 2
    i0, j0 = int(rng.integers(0, nx - 40)), int(rng.integers(0, ny - 50))
    pr = np.array([(c, i, j) for c in range(nc) for i in range(i0, i0 + 40) for j in range(j0, j0 + 50)], np.int64)
    pr = np.concatenate([pr, pr[rng.integers(0, len(pr), 90)]])[:4096]
    p = p.copy(probes=pr[rng.permutation(len(pr))], freqs=np.array([0.0, 3e10]), src=(i0 + 20, j0 + 25))
    say(f"case 2d dense probes {mode} {nx}x{ny}")
    for prec in ("f64", "f32"):
        with G.FdtdPlasma2D(p, precision=prec) as h:
            X, E = h.step(1).spectra(), h.fields()["E"]
            want = p.dt * E[tuple(p.probes.T)]
            assert np.any(want) and np.array_equal(X[:, 0], want), prec
            h.step(20)
            X = h.spectra()
        ref = oracle.run2d(p, 21, kind="omp")["X"]
        assert rel(X, ref) <= (1e-12 if prec == "f64" else 2e-5), prec


class OneCopy:
    """The smallest workspace the library takes for p, through the C ABI."""

    def __init__(self, G, p, precision):
        import ctypes
        import re
        import torch
        from paper_1709_00821_amd import _lib as L
        st = torch.cuda.Stream()
        self.d, self.keep = G.make_desc2(p, precision, st.cuda_stream)
        self.p, self.st, self.L, h = p, st, L.lib(), ctypes.c_void_p()
        full = ctypes.c_size_t()
        assert self.L.fdtd2d_workspace_bytes(ctypes.byref(self.d), ctypes.byref(full)) == 0
        self.ws = torch.empty(full.value, dtype=torch.uint8, device="cuda")
        at = ctypes.c_void_p(self.ws.data_ptr())
        assert self.L.fdtd2d_create(ctypes.byref(self.d), at, 256, ctypes.byref(h)) == L.E_WORKSPACE
        need = int(re.search(rb"needs (\d+)", self.L.fdtd2d_last_error()).group(1))
        self.need, self.full = need, full.value
        assert self.L.fdtd2d_create(ctypes.byref(self.d), at, need - 1, ctypes.byref(h)) == L.E_WORKSPACE
        assert self.L.fdtd2d_create(ctypes.byref(self.d), at, need, ctypes.byref(h)) == 0
        self.h, self.problem, self.desc = h, p, self.d

    def result(self, G):
        f = G.FdtdPlasma2D
        return f.spectra(self), f.fields(self)


@pytest.mark.parametrize("mode,nx,ny,px,py", [("tm", 70, 90, False, False), ("te", 33, 200, True, False),
                                              ("te", 64, 48, False, True), ("tm", 3, 140000, True, False),
                                              ("te", 2, 131100, False, True)])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_2d_in_place_steps_bitwise(G, mode, nx, ny, px, py, prec):
    """Steps taken one by one in place (a workspace that holds one copy of the
    fields, grids of two or three rows, the odd steps of any composition) against
    passes of tiles: the same spectra and fields, and the oracle's."""
    rng = np.random.default_rng(nx + ny)
    wide = nx < 4
    p = W.random_2d(rng, mode, max(nx, 4), ny if not wide else 400, periodic_x=px, periodic_y=py)
    if wide:                                  # the long way round: the random grid's rows, then vacuum
        w, v = np.zeros((p.ncomp, nx, ny)), np.full((p.ncomp, nx, ny), 1e10)
        w[:, :, 100:500], v[:, :, 100:500] = p.wp2[:, :nx], p.nu[:, :nx]
        pr = p.probes.copy()
        pr[:, 1], pr[:, 2] = pr[:, 1] % nx, 100 + pr[:, 2]
        p = p.copy(nx=nx, ny=ny, wp2=w, nu=v, probes=pr, src=(nx - 1, 300))
    say(f"case 2d in place {mode} {nx}x{ny} {prec}")
    T = 45
    one = OneCopy(G, p, prec)
    assert one.need < one.full or wide
    L = one.L
    assert L.fdtd2d_run(one.h, 19) == 0 and L.fdtd2d_run(one.h, T) == 0      # captured, in place
    X1, F1 = one.result(G)
    assert L.fdtd2d_run(one.h, 19) == 0 and L.fdtd2d_step(one.h, T - 19) == 0
    X2, F2 = one.result(G)
    assert L.fdtd2d_destroy(one.h) == 0
    with G.FdtdPlasma2D(p, precision=prec) as h:
        h.run(T)
        Xa, Fa = h.spectra(), h.fields()
        h.run(9)                              # one pass, one step in place
        h.run(10).run(9).step(1).step(2).step(3).step(1).step(T - 16)
        Xb, Fb = h.spectra(), h.fields()
    for X, F in ((X2, F2), (Xa, Fa), (Xb, Fb)):
        assert np.array_equal(X1, X)
        for k in ("E", "H", "J"):
            assert np.array_equal(F1[k], F[k]), k
    o = oracle.run2d(p, T, kind="omp")
    tol = 1e-12 if prec == "f64" else 2e-5
    assert rel(Xa, o["X"]) <= tol and max(errs(Fa, o)) <= 10 * tol


def test_2d_allocates_what_fits_when_torch_has_no_room(G, monkeypatch):
    """The Python handle without torch memory for its workspace."""
    import torch
    p = W.random_2d(np.random.default_rng(2), "tm", 90, 70)
    with G.FdtdPlasma2D(p) as h:
        X = h.run(30).spectra()

    def full(*a, **kw):
        raise torch.cuda.OutOfMemoryError("no room")
    monkeypatch.setattr(G.torch, "empty", full)
    with G.FdtdPlasma2D(p) as h:
        assert h.workspace is None and np.array_equal(h.run(30).spectra(), X)


def test_2d_step_composition_and_replay(G):
    p = W.random_2d(np.random.default_rng(5), "te", 70, 90)
    say("case 2d step composition")
    with G.FdtdPlasma2D(p) as a, G.FdtdPlasma2D(p) as b:
        a.step(1000).step(0).step(2500)      # crosses a 2048-sample window
        b.step(3500)
        assert a.steps_done() == b.steps_done() == 3500
        assert np.array_equal(a.spectra(), b.spectra())
        fa, fb = a.fields(), b.fields()
        for k in ("E", "H", "J"):
            assert np.array_equal(fa[k], fb[k])
        b.run(3500)
        X1 = b.spectra()
        b.run(3500)
        assert np.array_equal(b.spectra(), X1) and np.array_equal(X1, a.spectra())
        for k, v in b.fields().items():
            assert np.array_equal(v, fa[k])


def test_2d_errors(G):
    from paper_1709_00821_amd import _lib as L
    p = W.random_2d(np.random.default_rng(6), "tm", 30, 30)
    with G.FdtdPlasma2D(p) as h:
        with pytest.raises(L.FdtdError) as e:
            h.spectra()
        assert e.value.code == L.E_STATE


def _crop2(p, i0, i1, j0, j1):
    """The sub-box [i0, i1) x [j0, j1) of p as its own walled problem, the
    source and the probes inside it moved with it."""
    keep = [(k, c, i - i0, j - j0) for k, (c, i, j) in enumerate(p.probes) if i0 <= i < i1 and j0 <= j < j1]
    probes = np.array([q[1:] for q in keep], np.int64).reshape(-1, 3)
    q = p.copy(nx=i1 - i0, ny=j1 - j0, wp2=np.ascontiguousarray(p.wp2[:, i0:i1, j0:j1]),
               nu=np.ascontiguousarray(p.nu[:, i0:i1, j0:j1]), src=(p.src[0] - i0, p.src[1] - j0),
               probes=probes)
    return q, [k for k, *_ in keep]


@pytest.mark.parametrize("mode", ["tm", "te"])
def test_cylinder_2d_full_size_light_cone_matches_oracle(G, mode):
    """The 4096^2 benchmark problem in the benchmark's launch configuration
    (run(T), graph replay), T = 800 steps, against the oracle on the box of
    cells within T + 4 of the source: a step moves the fields one cell along
    each axis, so outside that box the full-size fields are exactly zero and
    inside it the box's walls, never reached, change nothing.  By step 800
    the pulse (half a cell a step) has entered the cylinder's Gaussian edge,
    320 cells from the source, so support cells carry current."""
    n, T = 4096, 800
    p = W.cylinder_2d(mode, n=n, n_freqs=16)
    si, sj = p.src
    r = T + 4
    i0, i1, j0, j1 = si - r, si + r + 1, sj - r, sj + r + 1
    q, inside = _crop2(p, i0, i1, j0, j1)
    assert q.wp2.any(), "the box must hold plasma"
    say(f"case 2d cylinder full size {mode} n={n} steps={T} box {q.nx}x{q.ny}")
    o = oracle.run2d(q, T, kind="omp")      # the OpenMP build: the same bits, sooner
    for prec, tol in (("f64", 1e-12), ("f32", 2e-5)):
        with G.FdtdPlasma2D(p, precision=prec) as h:
            h.run(T)
            F = h.fields()
            X = h.spectra()
        for k in ("E", "H", "J"):
            out = F[k].copy()
            out[:, i0:i1, j0:j1] = 0.0
            assert np.count_nonzero(out) == 0, (prec, k, "nonzero outside the light cone")
        Fin = {k: F[k][:, i0:i1, j0:j1] for k in ("E", "H", "J")}
        ef = errs(Fin, o)
        outside = [k for k in range(len(p.probes)) if k not in inside]
        assert np.all(X[outside] == 0)
        ex = rel(X[inside], o["X"]) if inside else 0.0
        say(f"2d full size {mode} {prec}: fields E {ef[0]:.2e} H {ef[1]:.2e} J {ef[2]:.2e} spectra {ex:.2e}")
        assert max(ef) <= tol * 10 and ex <= tol, prec
    assert np.max(np.abs(o["J"])) > 0
