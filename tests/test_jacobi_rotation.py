"""The rotation of the initialization's eigensolver, compiled for the CPU from the header that the GPU's is compiled from: it
annihilates the off-diagonal entry up to the error of the estimates it starts from and is orthogonal over the whole range of
entries, also where their squares leave the range of fp64, and the columns' lengths follow from it."""
import ctypes
import itertools
import os
import subprocess
from decimal import Decimal, localcontext

import numpy as np
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

// The eigensolver's sweeps over the columns v[c][.] in its order; returns the largest relative error of a followed length.
extern "C" double sweeps(double* v, int l, int count, double* cosine)
{
    double worst = 0.0;
    auto formed = [&](int c) { double s = 0.0; for (int e = 0; e < l; ++e) s = fma(v[c * l + e], v[c * l + e], s); return JacobiLength{s, s}; };
    auto check = [&](int c, double now) {
        long double s = 0.0L;
        for (int e = 0; e < l; ++e) s += static_cast<long double>(v[c * l + e]) * v[c * l + e];
        if (s > 1e-280L) worst = fmax(worst, static_cast<double>(std::fabs(now / s - 1.0L)));
    };
    auto at = [&](int pos, int round) { return pos == 0 ? 0 : (pos - 1 >= round ? pos - round : pos - round + l - 1); };
    JacobiLength* const length = new JacobiLength[l];
    for (int sweep = 0; sweep < count; ++sweep) {
        *cosine = 0.0;
        for (int c = 0; c < l; ++c) length[c] = formed(c);
        for (int round = 0; round < l - 1; ++round)
            for (int pair = 0; pair < l / 2; ++pair) {
                const int ca = at(pair, round), cb = at(l - 1 - pair, round);
                double *const a = v + ca * l, *const b = v + cb * l, hab = 0.0, c, s, tn;
                for (int e = 0; e < l; ++e) hab = fma(a[e], b[e], hab);
                *cosine = fmax(*cosine, hab == 0.0 ? 0.0 : fabs(hab) / std::sqrt(length[ca].now) / std::sqrt(length[cb].now));
                if (!jacobi_rotation<Off>(length[ca].now, length[cb].now, hab, c, s, tn)) continue;
                for (int e = 0; e < l; ++e) {
                    const double x = a[e], y = b[e];
                    a[e] = fma(c, x, -s * y);
                    b[e] = fma(s, x, c * y);
                }
                if (!jacobi_follow(c, tn, hab, length[ca], length[cb])) length[ca] = formed(ca), length[cb] = formed(cb);
                check(ca, length[ca].now), check(cb, length[cb].now);
            }
    }
    delete[] length;
    return worst;
}
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
    lib.sweeps.argtypes, lib.sweeps.restype = [doubles, ctypes.c_int, ctypes.c_int, doubles], ctypes.c_double
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


@pytest.mark.parametrize("decades", [0, 16, 60, 100])
@pytest.mark.parametrize("seed", range(4))
def test_lengths_follow_from_the_rotations(lib, decades, seed):
    """Columns of a triangular factor as the solver gets them, lengths from one size to `decades` decades apart, in any order:
    some absorb a long one and lose it again.  Bound: each of the l - 1 rotations of a sweep adds up to 16 roundings of
    1.1e-16 of the lengths that are carried (terms and sum, c twice, the entry, the column itself), and a length is formed anew
    below a thousandth of these: 1000 (l - 1) 16 1.1e-16 = 1.3e-10 at the worst.  After the solver's 48 sweeps the columns are orthogonal."""
    l = 72
    g = np.random.default_rng(100 * decades + seed)
    lib.off(2.0 ** -24, -2.0 ** -24)
    q = np.linalg.qr(g.normal(size=(l, l)))[0]
    size = 10.0 ** (-0.5 * decades * g.permutation(l) / (l - 1))
    lower = np.linalg.qr((q * size).T)[1].T if seed % 2 else np.tril(g.normal(size=(l, l))) * size[:, None]
    v = np.ascontiguousarray(lower)                                   # column c of L^T is row c of L
    cosine = ctypes.c_double()
    worst = lib.sweeps(v.ctypes.data_as(ctypes.POINTER(ctypes.c_double)), l, 48, ctypes.byref(cosine))
    assert worst < 1.3e-10 and cosine.value < 1e-8
