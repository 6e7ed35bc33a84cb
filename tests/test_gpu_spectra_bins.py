"""P(k), its adjoint and the velocity spectra at the bin counts and mesh sides
where their kernels change: one bin, the most bins that the one-pass kernel
takes, one more, and bins that begin inside the first shell."""
import numpy as np
import pytest

from _progress import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import adjoint, ic, pk  # noqa: E402
from paper_1507_05329_amd.inputs import bbks_table, step_edges, white_noise  # noqa: E402

L, NP, NM = 100.0, 32, 96


@pytest.fixture(scope="module")
def sim():
    from paper_1507_05329_amd.sim import ColaSim
    say("[gpu] create ColaSim np=32 nm=96")
    s = ColaSim(NP, NM, L)
    s.init_from_noise(torch.from_numpy(white_noise(11, NP)).cuda(), *bbks_table())
    s.run(step_edges()[:4])
    return s


def positions(sim):
    return ic.lattice(NP, L) + sim.get_state(("disp",))["disp"].cpu().numpy().astype(np.float64) * (L / NM)


def edges_of(nbins, ngrid):
    lo, hi = 2 * np.pi / L, np.pi * ngrid / L
    return np.linspace(0.5 * lo, 1.2 * hi, nbins + 1)  # past the Nyquist wavenumber: empty bins at the end


@pytest.mark.parametrize("nbins", [1, 2, 400, 512, 513])
@pytest.mark.parametrize("ngrid", [32, 96])
def test_pk_by_bin_count(sim, nbins, ngrid):
    say(f"[gpu] P(k), {nbins} bins on {ngrid}^3")
    e = edges_of(nbins, ngrid)
    km, p, n = sim.pk(e, ngrid)
    ko, po, no = pk.power_spectrum(positions(sim), L, ngrid, e)
    assert np.array_equal(n, no)
    ok = no > 0
    assert np.abs(km[ok] / ko[ok] - 1).max() < 1e-12
    assert np.abs(p[ok] / po[ok] - 1).max() < 1e-4
    assert np.isnan(p[~ok]).all() and np.isnan(km[~ok]).all()
    for _ in range(3):
        again = sim.pk(e, ngrid)
        assert all(a.tobytes() == b.tobytes() for a, b in zip(again, (km, p, n)))


@pytest.mark.parametrize("nbins", [1, 300, 600])
def test_pk_adjoint_by_bin_count(sim, nbins):
    say(f"[gpu] P(k) adjoint, {nbins} bins")
    e = edges_of(nbins, NM)
    cb = np.random.default_rng(2).standard_normal(nbins)
    d = sim.get_state(("disp",))["disp"]
    out = torch.zeros_like(d)
    sim.pk_adjoint(d, e, cb, out)
    ref = adjoint.pk_adjoint(positions(sim), L, NM, e, cb) * (L / NM)
    got = out.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(got - ref) / np.linalg.norm(ref) < 1e-4


@pytest.mark.parametrize("nbins", [1, 300, 512])
def test_velocity_spectra_agree_with_pk(sim, nbins):
    # the same density modes through both entry points: P_dd equals P(k) but for the
    # rounding of the weighted deposit, the mean |k| and the counts are those of P(k)
    e = edges_of(nbins, NM)
    km, p, n = sim.pk(e)
    kv, dd, _, _, nv = sim.pk_velocity(e, axis=1)
    assert np.array_equal(n, nv)
    ok = n > 0
    assert np.abs(kv[ok] / km[ok] - 1).max() < 1e-12
    assert np.abs(dd[ok] / p[ok] - 1).max() < 1e-4
