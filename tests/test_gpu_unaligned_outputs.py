"""The cotangent of the noise in a buffer that is only 4-byte aligned: the z pass
that writes pairs of floats takes 8-byte aligned buffers, any other gets the same
values by single floats.  Bit for bit, and nothing beside the array is written."""
import pytest

from _progress import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1507_05329_amd.inputs import bbks_table, white_noise  # noqa: E402


@pytest.mark.parametrize("np_side,nm", [(16, 32), (48, 96)])
@pytest.mark.parametrize("shift", [1, 2, 3])
def test_noise_cotangent_at_an_odd_float(np_side, nm, shift):
    from paper_1507_05329_amd import _lib
    from paper_1507_05329_amd.sim import ColaSim, _ptr
    say(f"[gpu] noise cotangent {np_side}^3, shift {shift}")
    n = np_side ** 3
    sim = ColaSim(np_side, nm, 3.0 * np_side)
    try:
        w = torch.from_numpy(white_noise(np_side, np_side)).cuda()
        sim.init_from_noise(w, *bbks_table())
        gen = torch.Generator("cuda").manual_seed(shift)
        bars = [torch.randn((3, n), generator=gen, device="cuda") for _ in range(3)]
        want = sim.init_adjoint(w, *bars)
        flat = torch.full((n + 8,), 7.0, device="cuda")
        out = flat[shift:shift + n]
        assert out.data_ptr() % 8 == 4 * (shift % 2)
        _lib.check(sim.lib.cola_init_2lpt_adjoint(sim.ctx, _ptr(w), *(_ptr(b) for b in bars), _ptr(out)), sim.ctx,
                   "init_2lpt_adjoint")
        torch.cuda.synchronize()
        assert torch.equal(out, want.view(-1))
        assert bool((flat[:shift] == 7.0).all()) and bool((flat[shift + n:] == 7.0).all())
    finally:
        sim.close()
