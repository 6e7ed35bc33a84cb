"""The adjoint of the 2LPT initial conditions against the forward map on large particle
grids (at 768 and 1024 a workgroup of its z pass holds one row), by dot products.

Psi1 is linear in the noise and Psi2 quadratic, so the derivatives along v at w are
J1 v = (Psi1(w + v) - Psi1(w - v)) / 2 and J2 v = (Psi2(w + v) - Psi2(w - v)) / 2 exactly.
<v, J^T J v> = |J v|^2, with dbar0 = J1 v in place of psi1bar D1 |J1 v|^2 + D2 <J1 v, J2 v>.
Both maps are float32 transforms with relative errors of some 1e-6: bar 1e-5."""
import pytest

from _progress import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import cosmology as cosmo  # noqa: E402
from paper_1507_05329_amd.inputs import bbks_table  # noqa: E402


def dot(a, b, piece=1 << 26):
    a, b = a.view(-1), b.view(-1)
    return sum(float(torch.dot(a[i:i + piece].double(), b[i:i + piece].double())) for i in range(0, a.numel(), piece))


@pytest.mark.parametrize("np_side", [256, 768, 1024])
def test_adjoint_is_the_transpose(np_side):
    from paper_1507_05329_amd.sim import ColaSim
    say(f"[gpu] transpose of the initial conditions {np_side}^3")
    table = bbks_table()
    sim = ColaSim(np_side, np_side, 2.5 * np_side)
    try:
        w, v = sim.noise(1), sim.noise(2)
        jv = []
        for sign in (1.0, -1.0):
            sim.init_from_noise(w + sign * v, *table)
            st = sim.get_state(("psi1", "psi2"))
            jv.append((st["psi1"], st["psi2"]))
            say(f"[gpu]   fields of w {'+' if sign > 0 else '-'} v")
        j1, j2 = (a.sub_(b).mul_(0.5) for a, b in zip(*jv))
        del jv, st
        sim.init_from_noise(w, *table)
        zero = torch.zeros_like(j1)
        n1, n2, n12 = dot(j1, j1), dot(j2, j2), dot(j1, j2)
        d1, d2 = cosmo.growth_D1(0.02, 0.27), cosmo.growth_D2(0.02, 0.27)
        for bars, want in (((zero, j1, zero), n1), ((zero, zero, j2), n2), ((j1, zero, zero), d1 * n1 + d2 * n12)):
            got = dot(sim.init_adjoint(w, *bars), v)
            say(f"[gpu]   <v, J^T u> / <J v, u> - 1 = {got / want - 1:.2e}")
            assert abs(got / want - 1) < 1e-5
    finally:
        sim.close()
