"""The rotation of the initialization's eigensolver, compiled for the CPU: it annihilates the off-diagonal entry and is
orthogonal over the whole range of entries, also where their squares leave the range of fp64."""
import ctypes
import itertools
import os
import subprocess

import pytest

import paper_2510_24061_amd as fq

SHIM = """
#include <cmath>
using std::fabs; using std::fmax; using std::sqrt;
#define __host__
#define __device__
static double rsqrt(double x) { return 1.0 / sqrt(x); }
#include "jacobi_rotation.h"
extern "C" int rotation(double a, double b, double h, double* cs) { return falqon::jacobi_rotation(a, b, h, cs[0], cs[1]); }
"""


@pytest.fixture(scope="module")
def rotation(tmp_path_factory):
    d = tmp_path_factory.mktemp("rotation")
    (d / "shim.cpp").write_text(SHIM)
    csrc = os.path.join(os.path.dirname(fq.lib_path()), "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-shared", "-fPIC", "-I", csrc, "-o", str(d / "shim.so"),
                    str(d / "shim.cpp")], check=True)
    f = ctypes.CDLL(str(d / "shim.so")).rotation
    f.argtypes = [ctypes.c_double] * 3 + [ctypes.POINTER(ctypes.c_double)]

    def call(haa, hbb, hab):
        cs = (ctypes.c_double * 2)()
        return f(haa, hbb, hab, cs), cs[0], cs[1]
    return call


@pytest.mark.parametrize("exponent", [0, 60, -60, -100, -145, -155, -165, -200, -290])
def test_annihilates_at_every_size(rotation, exponent):
    for haa, hbb, hab in itertools.product([0.0, 1.0, 3.0], [0.0, 1.0, 7.0], [1.0, -2.0, 1e-3]):
        size = 10.0 ** exponent
        rotated, c, s = rotation(haa * size, hbb * size, hab * size)
        assert rotated
        assert abs(c * c + s * s - 1.0) < 1e-15                          # a few roundings of 1.1e-16
        off = c * s * (haa - hbb) + (c * c - s * s) * hab                # in units of size
        assert abs(off) < 2e-15 * max(haa, hbb, abs(hab))


def test_leaves_rounding_noise_alone(rotation):
    assert rotation(1.0, 4.0, 1e-17) == (0, 1.0, 0.0)
    assert rotation(0.0, 0.0, 0.0) == (0, 1.0, 0.0)
