"""Displacements that are not finite leave the density of the other particles as it is,
node by node: the replay without them, on the contrast scale of all particles."""
import numpy as np
import pytest

from _progress import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import cic_fp32  # noqa: E402


# 256 and 1024 threads per tile, the latter with particles past a thread's first two
@pytest.mark.parametrize("np_side,nm", [(16, 32), (48, 96), (48, 48)])
def test_other_particles_keep_their_nodes(np_side, nm):
    from paper_1507_05329_amd.sim import ColaSim
    say(f"[gpu] density beside non-finite displacements, {np_side}^3 / {nm}^3")
    rng = np.random.default_rng(nm)
    n = np_side ** 3
    d = rng.uniform(-3.0, 3.0, (3, n)).astype(np.float32)
    bad = rng.choice(n, 60, replace=False)
    for j, i in enumerate(bad):
        d[j % 3, i] = (np.nan, np.inf, -np.inf)[(j // 3) % 3]
    d[:, bad[:2]] = np.nan
    sim = ColaSim(np_side, nm, 100.0)
    try:
        got = sim.density(disp=torch.from_numpy(d).cuda()).cpu().numpy()
    finally:
        sim.close()
    rest = np.setdiff1d(np.arange(n), bad)
    rho = cic_fp32._to_rho(cic_fp32.node_sums(d[:, rest], np_side, nm, rest)).reshape(nm, nm, nm)
    assert got.tobytes() == cic_fp32._contrast(rho, np_side, nm).tobytes()
