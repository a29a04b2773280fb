"""Host checks of the closures' roots in dsve_math.hpp: one step of the third-order iteration for a^(-1/3)
and a^(-1/10) from an FP32 estimate, evaluated in FP64 as the kernels do.

Tolerances: the step leaves 14/81 e^3 (e to 3e-6) and 77/2000 e^3 (e to 1e-5), below 1e-16 even from
estimates degraded to 1e-6; what remains is the rounding of its handful of operations, below 4 ulp of
2^-53, and seven or nine times that in the powers.
"""
import numpy as np

ULP = 2.0 ** -53


def seeds(a, p):
    exact = a ** p
    y0 = np.exp2(np.float32(p) * np.log2(a.astype(np.float32))).astype(np.float64)
    return exact, (y0, exact * (1 + 1e-6), exact * (1 - 1e-6))


def test_reciprocal_cube_root_third_order():
    a = np.concatenate([np.logspace(-6, 4, 20001), np.linspace(0.01, 3.0, 2001)])
    exact, ys = seeds(a, -1.0 / 3.0)
    for y in ys:
        e = 1.0 - a.astype(np.longdouble) * (y * y * y)   # one rounding in the kernels (FMA)
        e = e.astype(np.float64)
        r = y + (y * e) * (e * (2.0 / 9.0) + 1.0 / 3.0)
        np.testing.assert_allclose(r, exact, rtol=4 * ULP, atol=0)


def test_tenth_root_third_order():
    a = np.concatenate([np.logspace(-15, 3, 20001), np.linspace(0.5, 2.0, 2001)])
    exact, ys = seeds(a, -0.1)
    for y in ys:
        y5 = (y * y) * (y * y) * y
        e = (1.0 - a.astype(np.longdouble) * (y5 * y5)).astype(np.float64)
        r = y + (y * e) * (e * 0.055 + 0.1)
        np.testing.assert_allclose(r, exact, rtol=4 * ULP, atol=0)
        r4 = (r * r) * (r * r)
        np.testing.assert_allclose((a * a) * (r4 * r4 * r), a ** 1.1, rtol=9 * 4 * ULP + 16 * ULP, atol=0)
