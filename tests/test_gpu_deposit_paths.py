"""The tile sort and the mass deposit at the sizes where their kernels change:
meshes whose bucket scan takes one workgroup in one round, in several, and
several workgroups; tiles with many particles and with hardly any; particles
crowded on the faces, edges and corners of tiles, where the region's boundary
segments hold more records than a workgroup has threads.  Density bit for bit
against the FP32 replay; the weighted deposit (which sorts ids instead of
records) through the adjoint of the same state."""
import numpy as np
import pytest

from _progress import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import adjoint, cic_fp32, cola, ic  # noqa: E402
from paper_1507_05329_amd.inputs import bbks_table, seeded_normal, step_edges, white_noise  # noqa: E402


def faces(np_side, nm, seed, crowd):
    """Displacements that put most particles into cells 15 of their tiles along some axes (crowd: all
    of them around one tile corner), the others anywhere, some a whole box away."""
    rng = np.random.default_rng(seed)
    n = np_side ** 3
    q = np.stack(np.meshgrid(*([np.arange(np_side) * (nm / np_side)] * 3), indexing="ij")).reshape(3, -1)
    x = rng.uniform(0.0, nm, (3, n))
    tile = np.zeros((3, n)) + 16 if crowd else 16 * rng.integers(0, nm // 16, (3, n))
    on_face = (rng.random((3, n)) < 0.7)
    x = np.where(on_face, tile + 15.5 + rng.uniform(0.0, 1.0, (3, n)), tile + rng.uniform(0.0, 16.0, (3, n)) if crowd else x)
    x += nm * rng.integers(-1, 2, (3, n))
    return (x - q).astype(np.float32)


@pytest.mark.parametrize("np_side,nm", [(16, 32), (32, 32), (48, 48), (64, 64), (32, 96), (32, 128), (48, 192), (16, 384)])
@pytest.mark.parametrize("crowd", [False, True])
def test_density_on_tile_faces_bit_exact(np_side, nm, crowd):
    from paper_1507_05329_amd.sim import ColaSim
    say(f"[gpu] density of particles on tile faces, {np_side}^3 / {nm}^3")
    d = faces(np_side, nm, 7 * np_side + nm, crowd)
    sim = ColaSim(np_side, nm, 100.0)
    try:
        t = torch.from_numpy(d).cuda()
        got = [sim.density(disp=t).cpu().numpy() for _ in range(2)]
    finally:
        sim.close()
    ref = cic_fp32.density(d, np_side, nm)
    assert got[0].tobytes() == ref.tobytes() and got[1].tobytes() == ref.tobytes()


def test_sort_of_records_and_ids_together():
    # the recomputing adjoint sorts records and ids in one pass, the one with kept forces the ids alone
    from paper_1507_05329_amd.sim import ColaSim
    say("[gpu] records and ids in one sort")
    np_side, nm = 32, 64
    d = torch.from_numpy(faces(np_side, nm, 3, False)).cuda()
    z = torch.zeros_like(d)
    sim = ColaSim(np_side, nm, 100.0)
    out = []
    try:
        sim.set_state(d, z, z, z, 0.5, 0.451)
        slot = sim.force_slot()
        sim.step_keep(0.5, 0.598, slot)
        for kept in (None, slot):
            db, vb = torch.sin(d), torch.cos(d)
            p1, p2 = torch.zeros_like(d), torch.zeros_like(d)
            sim.step_adjoint(0.5, 0.598, 0.451, d, db, vb, p1, p2, slot=kept)
            out.append([x.cpu().numpy().tobytes() for x in (db, vb, p1, p2)])
    finally:
        sim.close()
    assert out[0] == out[1]


def test_non_finite_displacements_leave_the_other_particles():
    # a NaN or infinite displacement adds nothing that is not a number to the mesh
    from paper_1507_05329_amd.sim import ColaSim
    say("[gpu] density with non-finite displacements")
    np_side, nm = 16, 32
    d = faces(np_side, nm, 5, False)
    keep = d.copy()
    bad = np.array([3, 700, 4000])
    d[0, bad[0]], d[1, bad[1]], d[2, bad[2]] = np.nan, np.inf, -np.inf
    sim = ColaSim(np_side, nm, 100.0)
    try:
        got = sim.density(disp=torch.from_numpy(d).cuda()).cpu().numpy()
    finally:
        sim.close()
    assert np.isfinite(got).all()
    # the sum misses exactly the three particles (weights of NaN are taken as 0)
    mass = (got.astype(np.float64) + 1.0).sum() * np_side ** 3 / nm ** 3
    assert abs(mass - (np_side ** 3 - 3)) < 1e-3
    assert np.isfinite(keep).all()


def adjoint_of(np_side, nm, seed, edit=None):
    """One adjoint step from a state after two steps, and the oracle's."""
    from paper_1507_05329_amd.sim import ColaSim
    box, e = 3.0 * np_side, step_edges()
    sim = ColaSim(np_side, nm, box)
    try:
        sim.init_from_noise(torch.from_numpy(white_noise(seed, np_side)).cuda(), *bbks_table())
        sim.run(e[:3])
        st = sim.get_state()
        db, vb = (seeded_normal(seed + k, (3, np_side ** 3)) for k in (1, 2))
        if edit:
            edit(db, vb)
        out = [torch.from_numpy(db).cuda(), torch.from_numpy(vb).cuda()]
        out += [torch.zeros_like(out[0]), torch.zeros_like(out[0])]
        sim.step_adjoint(e[2], e[3], st["a_v"], st["disp"], *out)
        got = [x.cpu().numpy().astype(np.float64) for x in out]
    finally:
        sim.close()
    s = box / nm
    h = {n: st[n].cpu().numpy().astype(np.float64) * s for n in ("disp", "vres", "psi1", "psi2")}
    o = cola.State(np_side, nm, box, 0.27, -2.5, ic.lattice(np_side, box), h["disp"], h["vres"], h["psi1"], h["psi2"],
                   st["a_x"], st["a_v"])
    return got, [x * s for x in adjoint.step_adjoint(o, e[3], db / s, vb / s)] if edit is None else None


@pytest.mark.parametrize("np_side,nm", [(32, 32), (48, 48), (64, 64), (16, 96), (48, 128)])
def test_weighted_deposit_in_the_adjoint_step(np_side, nm):
    say(f"[gpu] adjoint step {np_side}^3 / {nm}^3")
    got, ref = adjoint_of(np_side, nm, np_side)
    for g, r in zip(got, ref):
        assert np.linalg.norm(g - r) / np.linalg.norm(r) < 1e-4


def test_weights_of_any_size():
    # cotangents 1e-30 and 1e30 times as large give results 1e-30 and 1e30 times as large; one that
    # is not finite leaves none finite of what depends on the transforms, and the others untouched
    say("[gpu] weighted deposit of small, large and non-finite weights")
    base, _ = adjoint_of(32, 64, 9, lambda db, vb: None)
    for f in (2.0 ** -100, 2.0 ** 90):
        def scale(db, vb):
            db *= np.float32(f)
            vb *= np.float32(f)
        got, _ = adjoint_of(32, 64, 9, scale)
        for g, r in zip(got, base):
            assert np.linalg.norm(g / f - r) / np.linalg.norm(r) < 1e-5
    for bad in (np.inf, np.nan):
        def spoil(db, vb):
            vb[1, 77] = bad
        got, _ = adjoint_of(32, 64, 9, spoil)
        assert not np.isfinite(got[0]).any()
        assert np.isfinite(np.delete(got[1], 77, axis=1)).all() and not np.isfinite(got[1][1, 77])
