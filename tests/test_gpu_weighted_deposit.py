"""The weighted deposits (three components in the adjoint step, two in the velocity
spectra) against the float64 oracle where a workgroup takes many rounds: particles
crowded around one tile corner, so that a region's boundary segments hold more
records than the workgroup has threads and the region many thousands, next to empty
tiles; and weights of one component over a range of 2^40.

Positions keep 0.02 cells from the cell faces: the gradient of a CIC weight jumps
there, and float32 positions may fall on the other side.  Bars: 1e-4, as for every
chain of float32 transforms here."""
import numpy as np
import pytest

from _progress import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import adjoint, cola, cosmology as cosmo, ic, pk, velocity  # noqa: E402

OM, N_LPT, A0, A1, AV = 0.27, -2.5, 0.5, 0.598, 0.451


def crowded(np_side, nm, seed, crowd):
    """Displacements: most particles around the corner of a tile (crowd) or anywhere, 70% of the
    coordinates in cell 15 of a tile; the particles of the fullest region and of its boundary."""
    rng = np.random.default_rng(seed)
    n = np_side ** 3
    cell = 16 + rng.integers(0, 16, (3, n)) if crowd else rng.integers(0, nm, (3, n))
    cell = np.where(rng.random((3, n)) < 0.7, cell // 16 * 16 + 15, cell)
    u = cell + rng.uniform(0.02, 0.98, (3, n))
    q = np.stack(np.meshgrid(*([np.arange(np_side) * (nm / np_side)] * 3), indexing="ij")).reshape(3, -1)
    nt = nm // 16
    t, up = cell // 16, cell % 16 == 15
    region, own = np.zeros((nt, nt, nt), int), np.zeros((nt, nt, nt), int)
    for s in np.ndindex(2, 2, 2):                      # a cell on an upper face also feeds the next tile
        ok = np.all(up | (np.array(s)[:, None] == 0), axis=0)
        np.add.at(region, tuple(((t + np.array(s)[:, None]) % nt)[:, ok]), 1)
    np.add.at(own, tuple(t), 1)
    d = u + 0.5 - q + nm * rng.integers(-1, 2, (3, n))
    return d.astype(np.float32), region.max(), (region - own).max()


def wide(rng, shape):
    """Standard normals times 2^0 ... 2^-40."""
    return (rng.standard_normal(shape) * np.exp2(-rng.uniform(0.0, 40.0, shape[-1]))).astype(np.float32)


# 256 threads per tile at 32/64 and 32/96, 1024 at 48/48 and 64/64
@pytest.mark.parametrize("np_side,nm", [(32, 64), (32, 96), (48, 48), (64, 64)])
@pytest.mark.parametrize("crowd", [True, False])
@pytest.mark.parametrize("weights", ["normal", "wide"])
def test_adjoint_step_of_crowded_particles(np_side, nm, crowd, weights):
    from paper_1507_05329_amd.sim import ColaSim
    say(f"[gpu] adjoint step, crowd={crowd}, {weights} weights, {np_side}^3 / {nm}^3")
    d, region, boundary = crowded(np_side, nm, np_side + nm, crowd)
    if crowd:
        threads = 1024 if np_side ** 3 > 1024 * (nm // 16) ** 3 else 256
        assert boundary > 4 * threads and region > 8000
    rng = np.random.default_rng(nm)
    n, box = np_side ** 3, 3.0 * np_side
    db, vb = ((wide(rng, (3, n)), wide(rng, (3, n))) if weights == "wide" else
              (rng.standard_normal((3, n)).astype(np.float32), rng.standard_normal((3, n)).astype(np.float32)))
    if weights == "wide":
        db *= np.float32(2.0 ** -20)                    # the kick's weights are those of vb
    sim = ColaSim(np_side, nm, box)
    try:
        out = [torch.from_numpy(x).cuda() for x in (db, vb)]
        out += [torch.zeros_like(out[0]), torch.zeros_like(out[0])]
        start = torch.from_numpy(d).cuda()
        sim.set_state(start, *(torch.zeros_like(start) for _ in range(3)), A0, AV)
        sim.step_adjoint(A0, A1, AV, start, *out)
        got = [x.cpu().numpy().astype(np.float64) for x in out]
    finally:
        sim.close()
    s, z = box / nm, np.zeros((3, n))
    o = cola.State(np_side, nm, box, OM, N_LPT, ic.lattice(np_side, box), d * float(s), z, z, z, A0, AV)
    ref = [x * s for x in adjoint.step_adjoint(o, A1, db / s, vb / s)]
    for name, g, r in zip(("dbar", "vbar", "psi1bar", "psi2bar"), got, ref):
        assert np.linalg.norm(g - r) < 1e-4 * np.linalg.norm(r), name
    if weights == "wide":                               # what the heavy particles do to the light ones
        light = np.abs(vb).max(axis=0) < 2.0 ** -20
        assert light.sum() > n // 8
        g, r = got[0][:, light], ref[0][:, light]
        assert np.linalg.norm(g - r) < 1e-4 * np.linalg.norm(r)


@pytest.mark.parametrize("np_side,nm", [(32, 64), (48, 48)])
@pytest.mark.parametrize("crowd", [True, False])
@pytest.mark.parametrize("weights", ["normal", "wide"])
def test_velocity_spectra_of_crowded_particles(np_side, nm, crowd, weights):
    from paper_1507_05329_amd.sim import ColaSim
    say(f"[gpu] velocity spectra, crowd={crowd}, {weights} weights, {np_side}^3 / {nm}^3")
    d, _, _ = crowded(np_side, nm, 3 * np_side + nm, crowd)
    rng = np.random.default_rng(np_side)
    n, box, axis = np_side ** 3, 3.0 * np_side, 1
    v = wide(rng, (3, n)) if weights == "wide" else rng.standard_normal((3, n)).astype(np.float32)
    z = np.zeros((3, n), np.float32)
    sim = ColaSim(np_side, nm, box)
    edges = pk.linear_edges(box, nm, dk=2 * np.pi / box)
    try:
        sim.set_state(*(torch.from_numpy(x).cuda() for x in (d, v, z, z)), A0, A0)
        km, pdd, pdu, puu, cnt = sim.pk_velocity(edges, axis=axis)
    finally:
        sim.close()
    s = box / nm
    o = cola.State(np_side, nm, box, OM, N_LPT, ic.lattice(np_side, box), d * float(s), v * float(s), z, z, A0, A0)
    u = velocity.full_velocity(o)[axis] / (A0 * cosmo.adot(A0, OM))
    ko, dd, du, uu, no = pk.velocity_power(o.positions(), u, box, nm, edges, axis)
    assert np.array_equal(cnt, no)
    ok = no > 0
    assert np.abs(km[ok] / ko[ok] - 1).max() < 1e-12
    assert np.abs(pdd[ok] / dd[ok] - 1).max() < 1e-4 and np.abs(puu[ok] / uu[ok] - 1).max() < 1e-4
    assert (np.abs(pdu[ok] - du[ok]) / np.sqrt(dd[ok] * uu[ok])).max() < 1e-4
