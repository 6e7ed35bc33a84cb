"""State copies and the density of the new state in one captured graph: replayed with
new contents in the same buffers, equal to the eager calls bit for bit each time."""
import pytest

from _progress import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("np_side,nm,shift", [(32, 64, 0), (48, 96, 1)])
def test_state_and_density_under_capture(np_side, nm, shift):
    from paper_1507_05329_amd.sim import ColaSim
    say(f"[gpu] captured state copies {np_side}^3 / {nm}^3, shift {shift}")
    stream = torch.cuda.Stream()
    gen = torch.Generator("cuda").manual_seed(np_side)
    with torch.cuda.stream(stream):
        sim = ColaSim(np_side, nm, 100.0, stream=stream)
        n = 3 * np_side ** 3
        arrays = [torch.zeros(n + shift, device="cuda")[shift:].view(3, -1) for _ in range(4)]
        back = [torch.zeros(n + shift, device="cuda")[shift:].view(3, -1) for _ in range(2)]
        out = torch.empty((nm, nm, nm), device="cuda")
        assert all(t.data_ptr() % 16 == 4 * shift for t in arrays + back)
        sim.set_state(*arrays, 0.5, 0.5)
        sim.density(out=out)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            sim.set_state(*arrays, 0.5, 0.5)
            sim.density(out=out)
            sim.get_state(("vres", "psi2"), out=dict(zip(("vres", "psi2"), back)))
        for _ in range(4):
            for a in arrays:
                a.copy_(torch.randn(a.shape, generator=gen, device="cuda"))
            graph.replay()
            stream.synchronize()
            got = out.clone()
            assert torch.equal(back[0], arrays[1]) and torch.equal(back[1], arrays[3])
            assert torch.equal(got, sim.density(disp=arrays[0].clone()))
        stream.synchronize()
        sim.close()
