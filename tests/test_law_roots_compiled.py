"""The closures' roots of dsve_math.hpp itself, compiled for the host (host_math.cpp), from estimates as far
off as the hardware's (4e-7 for the FP32 exponential of a logarithm, 2^-24 for the FP64 root estimate) to
either side: against 80-bit values.

Tolerances in units u = 2^-53.  a^(-1/3): the step leaves 14/81 e^3 of e up to 3e-6 (nothing) and the
rounding of y^3, of the FMAs and of the sum: 3 u.  sqrt(a) = a rsqrt(a), the root from one step: 3 u.
a^1.1 = a^2 y^9: y good to 2 u and 77/2000 e^3 of e up to 1e-5 (0.4 u), nine times that, and the
products' own rounding, 13 u: 35 u.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
U = 2.0 ** -53


@pytest.fixture(scope="module")
def roots(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("math") / "libmath.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__",
                           "-I", os.path.join(ROOT, "paper_1912_04791_amd", "csrc"), "-I", "/opt/rocm/include",
                           os.path.join(ROOT, "tests", "host_math.cpp"), "-o", so])
    return ctypes.CDLL(so)


def worst(lib, name, a, exact, errs):
    f = getattr(lib, name)
    f.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_long, ctypes.c_double]
    out = np.empty_like(a)
    top = 0.0
    for err in errs:
        f(a.ctypes.data, out.ctypes.data, a.size, err)
        top = max(top, float(np.max(np.abs((out.astype(np.longdouble) - exact) / exact))))
    return top / U


def test_reciprocal_cube_root(roots):
    a = np.concatenate([np.logspace(-6, 4, 20001), np.linspace(0.01, 3.0, 2001)])
    exact = 1 / np.cbrt(a.astype(np.longdouble))
    assert worst(roots, "host_rcbrt", a, exact, (0.0, 4e-7, -4e-7)) <= 3


def test_power_1p1(roots):
    a = np.concatenate([np.logspace(-15, 3, 20001), np.linspace(0.5, 2.0, 2001)])
    exact = a.astype(np.longdouble) ** (np.longdouble(11) / 10)
    assert worst(roots, "host_pow_1p1", a, exact, (0.0, 4e-7, -4e-7)) <= 35


def test_square_root(roots):
    a = np.concatenate([np.logspace(-12, 6, 20001), np.linspace(0.5, 4.0, 2001)])
    exact = np.sqrt(a.astype(np.longdouble))
    assert worst(roots, "host_sqrt", a, exact, (0.0, 2.0 ** -24, -2.0 ** -24)) <= 3


def test_depths_outside_the_range_of_the_estimate(roots):
    # no transport where the stress vanishes with the depth, however small, and finite where it is large
    a = np.concatenate([np.logspace(-290, -10, 1401), np.logspace(30, 90, 301)])
    for name in ("host_mpm", "host_vanrijn"):
        f = getattr(roots, name)
        f.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_long, ctypes.c_double]
        out = np.empty_like(a)
        f(a.ctypes.data, out.ctypes.data, a.size, 0.0)
        assert np.isfinite(out).all() and (out[a < 1] == 0).all()
