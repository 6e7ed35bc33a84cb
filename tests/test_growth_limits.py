"""The step scalars at scale factors far outside any run: they return (0, or not a
number where the formulas overflow), also where an integrand is not a number."""
import subprocess
import sys

import pytest

from paper_1507_05329_amd import _lib

CODE = """
import ctypes as C
import numpy as np
from paper_1507_05329_amd import _lib
lib, p, out = _lib.load(), _lib.cola_params(), np.zeros(10)
lib.cola_params_default(C.byref(p), 32, 64, 100.0)
p.omega_m = {om}
assert lib.cola_step_scalars(C.byref(p), {a0}, {a0}, {a1}, _lib.dptr(out)) == 0
print(out[1], out[8])
"""


# zero: the quadrature's nodes all lie where the integrand has underflowed to 0
@pytest.mark.parametrize("om,a0,a1,zero", [(0.27, 0.5, 1e160, True), (0.27, 0.5, 1.7e308, True),
                                           (0.27, 1e160, 2e160, True), (1.0, 0.5, 1e160, False),
                                           (0.27, 1e-200, 1e-190, False)])
def test_scalars_return(om, a0, a1, zero):
    r = subprocess.run([sys.executable, "-c", CODE.format(om=om, a0=a0, a1=a1)], capture_output=True, text=True,
                       timeout=20, cwd=_lib.__file__.rsplit("/", 2)[0])
    assert r.returncode == 0, r.stderr
    assert not zero or float(r.stdout.split()[1]) == 0.0
