"""The rotation of the initialization's eigensolver, compiled for the CPU from the header that the GPU's is compiled from: it
annihilates the off-diagonal entry up to the error of the estimates it starts from and is orthogonal over the whole range of
entries, also where their squares leave the range of fp64."""
import ctypes
import itertools
import os
import subprocess
from decimal import Decimal, localcontext

import pytest

import paper_2510_24061_amd as fq

SHIM = """
#include <cmath>
using std::fabs; using std::fma; using std::fmax;
#define __host__
#define __device__
#include "jacobi_rotation.h"
using namespace falqon;

static double off_rsqrt, off_reciprocal;
struct Off {                                                          // the GPU's estimates: off to either side
    static double rsqrt_of(double x) { return 1.0 / std::sqrt(x) * (1.0 + off_rsqrt); }
    static double reciprocal_of(double x) { return 1.0 / x * (1.0 + off_reciprocal); }
};
extern "C" void off(double a, double b) { off_rsqrt = a; off_reciprocal = b; }
extern "C" int rotation(double a, double b, double h, double* cst) { return jacobi_rotation<Off>(a, b, h, cst[0], cst[1], cst[2]); }
extern "C" double refined(double x) { return jacobi_rsqrt<Off>(x); }
"""
# The hardware's estimates are within 2^-24; here 2^-22, to either side.
OFF = [(a, b) for a in (-2.0 ** -22, 0.0, 2.0 ** -22) for b in (-2.0 ** -22, 0.0, 2.0 ** -22)]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("rotation")
    (d / "shim.cpp").write_text(SHIM)
    csrc = os.path.join(os.path.dirname(fq.lib_path()), "csrc")
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-shared", "-fPIC", "-I", csrc, "-o", str(d / "shim.so"),
                    str(d / "shim.cpp")], check=True)
    lib = ctypes.CDLL(str(d / "shim.so"))
    doubles = ctypes.POINTER(ctypes.c_double)
    lib.rotation.argtypes = [ctypes.c_double] * 3 + [doubles]
    lib.refined.argtypes, lib.refined.restype = [ctypes.c_double], ctypes.c_double
    lib.off.argtypes, lib.off.restype = [ctypes.c_double] * 2, None
    return lib


@pytest.mark.parametrize("off", OFF)
@pytest.mark.parametrize("exponent", [0, 60, -60, -100, -145, -155, -165, -200, -290])
def test_annihilates_at_every_size(lib, exponent, off):
    """Exact estimates leave roundings.  Others make the tangent t (1 + d) with |d| <= |off_rsqrt| + |off_reciprocal| to first
    order, and with t^2 hab + t (hbb - haa) = hab the entry becomes -d hab to first order."""
    lib.off(*off)
    cst = (ctypes.c_double * 3)()
    for haa, hbb, hab in itertools.product([0.0, 1.0, 3.0], [0.0, 1.0, 7.0], [1.0, -2.0, 1e-3]):
        size = 10.0 ** exponent
        assert lib.rotation(haa * size, hbb * size, hab * size, cst)
        c, s, t = cst
        assert abs(c * c + s * s - 1.0) < 1e-15                          # a few roundings of 1.1e-16
        assert abs(t) <= 1.0 + 2.0 ** -20 and s == t * c
        left = c * s * (haa - hbb) + (c * c - s * s) * hab               # in units of size
        assert abs(left) < 1.001 * (abs(off[0]) + abs(off[1])) * abs(hab) + 2e-15 * max(haa, hbb, abs(hab))


def test_leaves_rounding_noise_alone(lib):
    lib.off(0.0, 0.0)
    cst = (ctypes.c_double * 3)()
    for entries in [(1.0, 4.0, 1e-17), (0.0, 0.0, 0.0)]:
        assert lib.rotation(*entries, cst) == 0 and list(cst) == [1.0, 0.0, 0.0]


@pytest.mark.parametrize("off", OFF)
def test_refinement_of_an_estimate(lib, off):
    """A step of third order from 2^-22 leaves less than a rounding; what remains are the roundings of that step (three, halved
    where they meet a small correction): within 2 units of 2.2e-16."""
    lib.off(*off)
    for exponent in (-900, -451, -200, -1, 0, 1, 77, 300, 900):
        for mantissa in (1.0, 1.0 + 2.0 ** -52, 1.234567, 1.5, 1.999999999):
            x = mantissa * 2.0 ** exponent
            with localcontext() as c:
                c.prec = 60
                assert abs(Decimal(lib.refined(x)) * Decimal(x).sqrt() - 1) < Decimal(4.5e-16), x
