"""The 2LPT maps divide by |n|^2 with one correctly rounded quotient.

Waves of a quarter of the particle grid's frequency (n = np / 4) on a grid whose
side is a power of two pass the transforms exactly: every value they meet is 0 or
a power of two times the input, every twiddle that meets one is 1, -1, i or -i (to
6e-17).  With P = dq^3 the amplitude is 1, so the displacement is np^3 n fl(s / n2)
times sines and cosines of 0 or +-1, where s = nm / (2 pi np^3) in float32 and
fl(s / n2) is the one rounding: equality bit for bit.  A product with the hardware's
reciprocal of n2 = 3 n^2 (the float below 1 / n2) differs from it."""
import numpy as np
import pytest

from _progress import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def waves(np_side):
    i = np.arange(np_side)
    c, s = np.array([1.0, 0.0, -1.0, 0.0])[i % 4], np.array([0.0, 1.0, 0.0, -1.0])[i % 4]
    x, y, z = ((c[:, None, None], s[:, None, None]), (c[None, :, None], s[None, :, None]),
               (c[None, None, :], s[None, None, :]))
    ccc = x[0] * y[0] * z[0]
    gradient = np.stack([x[1] * y[0] * z[0], x[0] * y[1] * z[0], x[0] * y[0] * z[1]])   # -d/dx, -d/dy, -d/dz of ccc
    return ccc, gradient, x[0] * y[0] + z[0] + 0.0 * ccc


def fields(np_side, nm, noise):
    from paper_1507_05329_amd.sim import ColaSim
    sim = ColaSim(np_side, nm, float(np_side))      # dq = 1
    try:
        sim.init_from_noise(torch.from_numpy(noise.astype(np.float32).reshape(-1)).cuda(), np.array([1e-3, 1e3]),
                            np.array([1.0, 1.0]))
        st = sim.get_state()
        return [st[n].cpu().numpy().reshape(3, np_side, np_side, np_side) for n in ("psi1", "psi2")]
    finally:
        sim.close()


@pytest.mark.parametrize("np_side", [32, 64])
@pytest.mark.parametrize("order", [1, 2])
def test_one_rounding_in_the_division(np_side, order):
    say(f"[gpu] exact 2LPT division, order {order}, {np_side}^3")
    nm, n = 2 * np_side, np_side // 4
    ccc, gradient, pair = waves(np_side)
    s, n2 = np.float32(nm / (2.0 * np.pi) / np_side ** 3), np.float32(3 * n * n)
    assert s / n2 != s * np.nextafter(np.float32(1.0) / n2, np.float32(0.0))
    v = (s / n2) * np.float32(n * np_side ** 3)      # exact but for the quotient
    # order 1: psi1 = IDFT[i n s / n2 DFT(ccc)].  Order 2: phi = cos x cos y / (2 n^2) + cos z / n^2 has the
    # source cos x cos y cos z + Nyquist waves (zeroed), and psi2 = IDFT[-i n s / n2 DFT(source)]
    got = fields(np_side, nm, ccc if order == 1 else pair)[order - 1]
    want = (v * (-gradient if order == 1 else gradient)).astype(np.float32)
    some = want != 0
    assert np.array_equal(got[some], want[some])
    assert np.abs(got[~some]).max() < 1e-12 * v
