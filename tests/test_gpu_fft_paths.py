"""The forward z transform's two forms (plain and nontemporal accesses, by the
bytes of the launch's meshes).

A batch of five 96^3/192^3 mocks (165 MB of mesh: more than half of the
last-level cache) takes the nontemporal form, each mock alone (33 MB) the
plain one; the arithmetic is the same, so the states are equal bit for bit.
Single meshes of either form are compared element
by element with FP64 transforms in test_gpu_lengths.py.
"""
import pytest

from _progress import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1507_05329_amd.inputs import bbks_table, step_edges  # noqa: E402


@pytest.mark.parametrize("mocks", [3, 5])
def test_batch_across_the_cache_size_equals_single_mocks(mocks):
    from paper_1507_05329_amd.sim import ColaBatch, ColaSim
    say(f"[gpu] {mocks} mocks 96/192 against single runs")
    table, e = bbks_table(), step_edges()
    specs = [dict(np=96, nmesh=192, box=300.0, seed=11 + m) for m in range(mocks)]
    b = ColaBatch(specs)
    seq = [ColaSim(96, 192, 300.0) for _ in specs]
    try:
        for m, s, sp in zip(b.mocks, seq, specs):
            m.init_2lpt(sp["seed"], *table)
            s.init_2lpt(sp["seed"], *table)
        for i in range(3):
            b.step(e[i], e[i + 1])
            for s in seq:
                s.step(e[i], e[i + 1])
            torch.cuda.synchronize()
            for m, s in zip(b.mocks, seq):
                a, c = m.get_state(), s.get_state()
                assert torch.equal(a["disp"], c["disp"]) and torch.equal(a["vres"], c["vres"])
    finally:
        b.close()
        for s in seq:
            s.close()
