"""Plane ranges of the 3D executor's slabs (csrc/slabs3d.h), on the CPU: the
header is compiled alone and its launches are played through for every grid
length, planes per thread and a few plane sizes."""
import ctypes
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PLAY = r"""
#include <vector>
#include "slabs3d.h"
using namespace fdtdp;
// 0, or what the n steps of a grid do wrong: 1 an empty launch, 2 planes outside
// the grid, 3 a plane advanced out of turn, 4 a plane left behind
extern "C" int play(int64_t nx, int64_t plane, int64_t ni, int n)
{
    const int64_t L = slab_planes(nx, plane, ni);
    if (L == 0) return 0;
    if (L % ni) return 5;
    std::vector<int> E(nx, 0), H(nx, 0);
    for (int64_t s = 0; s < nx; s += L)
        for (int t = 0; t < n; ++t) {
            const SlabRange r = slab_range(nx, L, s, t);
            if (r.ia >= r.ib) return 1;
            if (r.ia < 0 || r.ib > nx) return 2;
            for (int64_t i = r.ia; i < r.ib; ++i) {
                if (H[i] != t || E[i] != t || (i + 1 < nx && E[i + 1] != t)) return 3;
                H[i] = t + 1;
            }
            for (int64_t i = r.ia; i < r.ib; ++i) {
                if (E[i] != t || (i > 0 && H[i - 1] != t + 1)) return 3;
                E[i] = t + 1;
            }
        }
    for (int64_t i = 0; i < nx; ++i)
        if (E[i] != n || H[i] != n) return 4;
    return 0;
}
extern "C" int64_t planes(int64_t nx, int64_t plane, int64_t ni) { return slab_planes(nx, plane, ni); }
extern "C" int most() { return kSlabSteps; }
"""


def test_slab_ranges_hold_planes_and_advance_each_in_turn(tmp_path):
    src, so = tmp_path / "play.cpp", tmp_path / "play.so"
    src.write_text(PLAY)
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_1709_00821_amd", "csrc"), str(src), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    i64 = ctypes.c_int64
    lib.play.argtypes = [i64, i64, i64, ctypes.c_int]
    lib.planes.argtypes, lib.planes.restype = [i64, i64, i64], i64
    in_slabs = 0
    for nx in list(range(2, 131)) + [384, 1000]:
        for plane in (1 << 18, 1 << 20, 4 << 20, 8 << 20, 12 << 20, 64 << 20):
            for ni in range(1, 17):
                in_slabs += lib.planes(nx, plane, ni) > 0
                for n in (1, 2, 13, lib.most()):
                    assert lib.play(nx, plane, ni, n) == 0, (nx, plane, ni, n)
    assert in_slabs > 1000
    # the smallest grids in slabs, and what a thread of one plane gives them
    assert lib.planes(25, 9 << 20, 1) == lib.planes(30, 9 << 20, 1) == lib.most()
