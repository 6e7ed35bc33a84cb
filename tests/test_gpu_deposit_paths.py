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

from oracle import cic_fp32  # noqa: E402


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
