"""The rotation of the initialization's eigensolver, compiled for the CPU: it annihilates the off-diagonal entry and is
orthogonal over the whole range of entries, also where their squares leave the range of fp64."""
import ctypes
import itertools
import os
import subprocess
from decimal import Decimal, localcontext

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


# the GPU's estimates in place of the host's: within 2^-24 of the value there, 2^-22 here, off to either side
ESTIMATES = """
#include <cmath>
#define __host__
#define __device__
#include "jacobi_rotation.h"
static double off_rsqrt, off_reciprocal;
struct Off {
    static double rsqrt_of(double x) { return 1.0 / std::sqrt(x) * (1.0 + off_rsqrt); }
    static double reciprocal_of(double x) { return 1.0 / x * (1.0 + off_reciprocal); }
};
extern "C" void off(double a, double b) { off_rsqrt = a; off_reciprocal = b; }
extern "C" int rotation(double a, double b, double h, double* cs) { return falqon::jacobi_rotation<Off>(a, b, h, cs[0], cs[1]); }
extern "C" double refined(int which, double x)
{
    return which == 0 ? falqon::jacobi_rsqrt<Off>(x) : which == 1 ? falqon::jacobi_sqrt<Off>(x) : falqon::jacobi_reciprocal<Off>(x);
}
"""


@pytest.fixture(scope="module")
def estimated(tmp_path_factory):
    d = tmp_path_factory.mktemp("estimated")
    (d / "shim.cpp").write_text(ESTIMATES)
    csrc = os.path.join(os.path.dirname(fq.lib_path()), "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-shared", "-fPIC", "-I", csrc, "-o", str(d / "shim.so"),
                    str(d / "shim.cpp")], check=True)
    lib = ctypes.CDLL(str(d / "shim.so"))
    lib.rotation.argtypes = [ctypes.c_double] * 3 + [ctypes.POINTER(ctypes.c_double)]
    lib.refined.argtypes, lib.refined.restype = [ctypes.c_int, ctypes.c_double], ctypes.c_double
    lib.off.argtypes, lib.off.restype = [ctypes.c_double] * 2, None
    return lib


OFF = [(a, b) for a in (-2.0 ** -22, 0.0, 2.0 ** -22) for b in (-2.0 ** -22, 0.0, 2.0 ** -22)]


@pytest.mark.parametrize("off", OFF)
def test_refinement_of_an_estimate(estimated, off):
    """Two steps from 2^-22 leave less than a rounding; what remains are the roundings of the last step (three, halved
    where they meet a small correction): within 2 units of 2.2e-16."""
    estimated.off(*off)
    for exponent in (-900, -451, -200, -1, 0, 1, 77, 300, 900):
        for mantissa in (1.0, 1.0 + 2.0 ** -52, 1.234567, 1.5, 1.999999999):
            x = mantissa * 2.0 ** exponent
            with localcontext() as c:
                c.prec = 60
                root = Decimal(x).sqrt()
                for which, want in enumerate((1 / root, root, 1 / Decimal(x))):
                    assert abs(Decimal(estimated.refined(which, x)) / want - 1) < Decimal(4.5e-16), (which, x)


@pytest.mark.parametrize("off", OFF)
@pytest.mark.parametrize("exponent", [0, 60, -60, -100, -145, -155, -165, -200, -290])
def test_annihilates_from_estimates(estimated, exponent, off):
    estimated.off(*off)
    cs = (ctypes.c_double * 2)()
    for haa, hbb, hab in itertools.product([0.0, 1.0, 3.0], [0.0, 1.0, 7.0], [1.0, -2.0, 1e-3]):
        size = 10.0 ** exponent
        assert estimated.rotation(haa * size, hbb * size, hab * size, cs)
        c, s = cs
        assert abs(c * c + s * s - 1.0) < 1e-15
        assert abs(c * s * (haa - hbb) + (c * c - s * s) * hab) < 2e-15 * max(haa, hbb, abs(hab))
