"""The corrected quotient of the half-precision solid velocity (quotient_whole)
against the division of the host, which rounds correctly: the library's own
function, compiled for the host with the processor's fused multiply-add."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1011_2613_amd", "csrc")

HOST = """
#include <cstring>
#include "internal.h"
// wrong quotients of 1.m 2^e over the 2^23 significands m, every `step`-th
extern "C" long wrong(int den, int e, int step) {
    const float d = (float)den, inv = 1.0f / d;
    int bad = 0;
    for (uint32_t m = 0; m < (1u << 23); m += step) {
        const uint32_t u = (uint32_t)(e + 127) << 23 | m;
        float x;
        memcpy(&x, &u, 4);
        bad += (lbimb::quotient_whole(x, d, inv) != x / d) | (lbimb::quotient_whole(-x, d, inv) != -x / d);
    }
    return bad;
}
extern "C" long wrong_odd(int last) {
    long bad = 0;
#pragma omp parallel for schedule(dynamic, 4) reduction(+ : bad)
    for (int d = 1; d <= last; d += 2) bad += wrong(d, 0, 1);
    return bad;
}
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("quotient")
    src, lib = d / "quotient.cpp", d / "quotient.so"
    src.write_text(HOST)
    subprocess.run(["g++", "-O3", "-std=c++17", "-mavx2", "-mfma", "-ffp-contract=off", "-fno-math-errno", "-fopenmp",
                    "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC, str(src),
                    "-o", str(lib)], check=True)
    L = ctypes.CDLL(str(lib))
    L.wrong.restype = L.wrong_odd.restype = ctypes.c_long
    return L


def test_every_significand_over_every_odd_divisor(host):
    """Odd divisors up to 4 095: an even one differs by a power of two, which
    changes no rounding within the range."""
    assert host.wrong_odd(4095) == 0


@pytest.mark.parametrize("e", [-100, -99, 0, 99])
def test_ends_of_the_range(host, e):
    for den in (1, 2, 3, 7, 64, 511, 512, 1000, 1536, 2047, 2048, 4095, 4096):
        assert host.wrong(den, e, 1009) == 0, den
