"""The growth factor of the step scalars against a fixed quadrature in long double.

D1(a) = E(a) I(a) / I(1), I(a) = int_0^a dx / (x E)^3 = int_0^sqrt(a) 2 s^4 /
(Om + OL s^6)^(3/2) ds; the reference takes 40 panels of 60 Gauss-Legendre
nodes.  The library stops at a relative error of 1e-14 for each of the two
integrals; with the roundings of E, the ratio and the sums: 1e-13.
"""
import ctypes as C

import numpy as np
import pytest

from paper_1507_05329_amd import _lib


def reference_D1(a, om):
    x, w = np.polynomial.legendre.leggauss(60)
    x, w = x.astype(np.longdouble), w.astype(np.longdouble)
    om, a = np.longdouble(om), np.longdouble(a)

    def integral(b):
        total = np.longdouble(0)
        for i in range(40):
            lo, hi = b * i / 40, b * (i + 1) / 40
            s = (lo + hi) / 2 + (hi - lo) / 2 * x
            total += ((hi - lo) / 2 * w * 2 * s**4 / (om + (1 - om) * s**6) ** np.longdouble(1.5)).sum()
        return total

    return np.sqrt(om / a**3 + 1 - om) * integral(np.sqrt(a)) / integral(np.longdouble(1))


@pytest.mark.parametrize("om", [0.01, 0.27, 0.7, 1.0])
@pytest.mark.parametrize("a", [1e-4, 0.02, 0.1, 0.51, 1.0, 4.0])
def test_growth_factor(om, a):
    lib = _lib.load()
    p = _lib.cola_params()
    lib.cola_params_default(C.byref(p), 32, 64, 100.0)
    p.omega_m = om
    out = np.zeros(10)
    assert lib.cola_step_scalars(C.byref(p), a, a, 1.1 * a, _lib.dptr(out)) == 0
    np.testing.assert_allclose([out[1], out[8]], [float(reference_D1(a, om)), float(reference_D1(1.1 * a, om))],
                               rtol=1e-13)
