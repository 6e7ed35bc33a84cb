"""2LPT initial conditions at every kind of transform length and with P(k)
tables of two nodes and of more nodes than the device holds, against the
float64 oracle."""
import numpy as np
import pytest

from _progress import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import cosmology as cosmo, ic  # noqa: E402
from paper_1507_05329_amd.inputs import bbks_table, white_noise  # noqa: E402


def fields(np_side, nm, box, w, table):
    from paper_1507_05329_amd.sim import ColaSim
    sim = ColaSim(np_side, nm, box)
    try:
        sim.init_from_noise(torch.from_numpy(w).cuda(), *table)
        st = sim.get_state()
        return {n: st[n].cpu().numpy().astype(np.float64) for n in ("disp", "vres", "psi1", "psi2")}
    finally:
        sim.close()


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("np_side,nm", [(16, 32), (32, 32), (48, 96), (64, 96), (96, 96), (128, 192)])
def test_initial_conditions_by_length(np_side, nm):
    say(f"[gpu] 2LPT initial conditions {np_side}^3 / {nm}^3")
    box = 3.0 * np_side
    w, t = white_noise(np_side, np_side), bbks_table()
    got = fields(np_side, nm, box, w, t)
    p1, p2 = ic.initial_fields(w, box, *t)
    s = nm / box
    p1, p2 = p1 * s, p2 * s
    assert rel(got["psi1"], p1) < 1e-5 and rel(got["psi2"], p2) < 1e-4
    d = cosmo.growth_D1(0.02, 0.27) * p1 + cosmo.growth_D2(0.02, 0.27) * p2
    assert rel(got["disp"], d) < 1e-5 and not got["vres"].any()


@pytest.mark.parametrize("nk", [2, 3, 400000])
def test_table_sizes(nk):
    # a power law is the same function whatever the number of nodes
    say(f"[gpu] P(k) table of {nk} nodes")
    w = white_noise(5, 32)
    k0, p0 = np.array([1e-4, 50.0]), 1e3 * np.array([1e-4, 50.0]) ** -1.5
    k = np.geomspace(1e-4, 50.0, nk)
    ref = fields(32, 64, 100.0, w, (k0, p0))
    got = fields(32, 64, 100.0, w, (k, 1e3 * k ** -1.5))
    assert rel(got["psi1"], ref["psi1"]) < 1e-6 and rel(got["psi2"], ref["psi2"]) < 1e-6


@pytest.mark.parametrize("np_side,nm", [(16, 32), (32, 32), (48, 48), (64, 96), (96, 96), (128, 192)])
def test_initial_condition_adjoint_by_length(np_side, nm):
    from oracle import adjoint
    from paper_1507_05329_amd.sim import ColaSim
    say(f"[gpu] adjoint of the initial conditions {np_side}^3 / {nm}^3")
    box, t = 3.0 * np_side, bbks_table()
    w = white_noise(np_side + 1, np_side)
    d0, p1, p2 = np.random.default_rng(np_side).standard_normal((3, 3, np_side ** 3)).astype(np.float32)
    sim = ColaSim(np_side, nm, box)
    try:
        sim.init_from_noise(torch.from_numpy(w).cuda(), *t)
        got = sim.init_adjoint(*(torch.from_numpy(x).cuda() for x in (w, d0, p1, p2))).cpu().numpy().astype(np.float64)
    finally:
        sim.close()
    s = box / nm
    ref = adjoint.ic_adjoint(w.astype(np.float64), box, *t, (p1 + cosmo.growth_D1(0.02, 0.27) * d0) / s,
                             (p2 + cosmo.growth_D2(0.02, 0.27) * d0) / s)
    assert rel(got.ravel(), ref.ravel()) < 1e-4
