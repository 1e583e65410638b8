"""Bounding boxes of footprints against the places that their lists reserve, at
radii a rounding off a multiple of 1/2 (cube roots are such radii) and centres
where both ends of a box round onto nodes.  The CPU test compiles the library's
own box arithmetic for the host; the GPU tests run such particles against the
FP64 oracle bit for bit, in runs whose lists are cut into segments."""
import ctypes
import itertools
import math
import os
import subprocess

import numpy as np
import pytest

from tests.parity_util import compare, make_pair

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1011_2613_amd", "csrc")

HOST = """
#include "internal.h"
extern "C" int extent(double R) { return lbimb::box_extent(R); }
extern "C" void boxes(int n, const double *c, const double *R, int *lo, int *hi) {
    for (int i = 0; i < n; i++) lbimb::box_axis(c[i], R[i], lo[i], hi[i]);
}
"""


def rounded(v, steps):
    for _ in range(abs(steps)):
        v = math.nextafter(v, math.inf if steps > 0 else -math.inf)
    return v


def test_boxes_fit_their_lists(tmp_path):
    """Every box holds at most extent(R) nodes per axis, hence at most
    extent(R_max)^D of them for R <= R_max, and every node left out lies where
    no sub-cell sample of eight per axis reaches the particle."""
    src, lib = tmp_path / "box.cpp", tmp_path / "box.so"
    src.write_text(HOST)
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-I", CSRC, str(src), "-o", str(lib)], check=True)
    L = ctypes.CDLL(str(lib))
    L.extent.argtypes = [ctypes.c_double]
    radii = [rounded(k / 2, s) for k in range(1, 125) for s in range(-6, 7) if rounded(k / 2, s) <= 62.0]
    radii += [k ** (1 / 3) for k in range(1, 1001)]
    centres = [rounded(b, s) for b in (0.0, 0.5, 7.5, 40.0, 40.5, 1000.5, 65534.5) for s in (-1, 0, 1)]
    c, R = (np.array(v) for v in zip(*itertools.product(centres, radii)))
    lo, hi = np.empty(len(c), np.int32), np.empty(len(c), np.int32)
    pd, pi = ctypes.POINTER(ctypes.c_double), ctypes.POINTER(ctypes.c_int)
    L.boxes(len(c), c.ctypes.data_as(pd), R.ctypes.data_as(pd), lo.ctypes.data_as(pi), hi.ctypes.data_as(pi))
    ext = np.array([L.extent(r) for r in R])
    assert np.all(ext == np.floor(2.0 * R + 1.0) + 1) and L.extent(62.0) == 126
    assert np.all(hi - lo + 1 <= ext)
    assert np.any(np.floor(c + R + 0.5) > hi)  # some boxes are narrowed
    reach = 0.5 - 0.5 / 8
    assert np.all(c - (lo - 1) - reach > R) and np.all(hi + 1 - c - reach > R)


CUBE = 125.0 ** (1.0 / 3.0)  # 4.999999999999999
CASES = [
    # dim, shape, radius, centres, samples, wall
    (3, (36, 34, 32), CUBE, [[20.5, 16.5, 14.5]], 4, False),
    (3, (40, 34, 32), CUBE, [[14.5, 15.5, 16.5], [24.5, 15.5, 16.5], [34.5, 28.5, 13.5]], 8, False),
    (3, (36, 30, 32), 7 - 2.0**-50, [[16.5, 23.5, 15.5]], 3, True),  # touches the upper wall
    (2, (260, 260), math.nextafter(60.5, 0), [[130.0, 125.0, 0.0]], 2, False),
    (2, (60, 64), 216.0 ** (1.0 / 3.0) * 2, [[28.5, 30.5, 0.0], [53.5, 45.5, 0.0]], 4, True),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(CASES)))
def test_rounded_radii_equal_the_oracle(gpu_lib, case):
    dim, shape, R, pos, S, wall = CASES[case]
    print("rounded radius", dim, shape, repr(R), len(pos), flush=True)
    n = len(pos)
    for c in np.array(pos)[:, :dim].ravel():  # these are the centres that round
        assert np.floor(c + R + 0.5) - np.ceil(c - R - 0.5) > np.floor(2.0 * R + 1.0)
    vel, om = np.full((n, 3), 0.004), np.full((n, 3), 5e-4)
    if dim == 2:
        vel[:, 2] = 0.0
        om[:, :2] = 0.0
    parts = (np.array(pos), vel, om, np.full(n, R), np.full(n, 6.0), np.ones(n, np.uint8))
    orc, gpu = make_pair(gpu_lib, dim, shape, 0.7, wall_y=wall, fluid_force=(1e-5, 0, 0), samples=S, kn=20.0,
                         particles=parts, max_radius=R)
    for steps in (1, 1, 4):
        orc.step(steps)
        gpu.step(steps)
        errs = compare(orc, gpu)
        assert all(e == 0.0 for e in errs.values()), errs
        assert np.array_equal(gpu.q(), orc.q()[:dim])
    # the sums over the lists: fluid and solid fractions of the nodes add up
    st = gpu.stats()
    assert np.allclose(st["mean_drag"][:dim], orc.forces()[0].mean(axis=0)[:dim], rtol=1e-13, atol=1e-18)
