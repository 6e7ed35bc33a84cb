"""State arrays in and out: one launch for the arrays of a call.

Full and partial sets, vectors of 4 and single floats (a buffer that is only
4-byte aligned), a source that is the destination, and a copy that a
stream-ordered sequence would see in order (one state array into another).
Copies are compared bit for bit.
"""
import ctypes

import pytest

from _progress import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

NAMES = ("disp", "vres", "psi1", "psi2")


def offset_like(t, shift):
    flat = torch.zeros(t.numel() + shift, dtype=t.dtype, device=t.device)[shift:]
    return flat.view(t.shape)


@pytest.mark.parametrize("np_side", [16, 48, 256])
@pytest.mark.parametrize("shift", [0, 1, 4])
def test_state_round_trip(np_side, shift):
    from paper_1507_05329_amd.sim import ColaSim
    say(f"[gpu] state copies np={np_side} shift={shift}")
    s = ColaSim(np_side, 2 * np_side, 100.0)
    gen = torch.Generator("cuda").manual_seed(np_side + shift)
    try:
        ref = []
        for _ in NAMES:
            t = offset_like(s.particles(), shift)
            t.copy_(torch.randn(t.shape, generator=gen, device="cuda"))
            ref.append(t)
        s.set_state(*ref, 0.5, 0.5)
        out = {n: offset_like(s.particles(), shift) for n in NAMES}
        got = s.get_state(out=out)
        for n, t in zip(NAMES, ref):
            assert torch.equal(got[n], t), n
        # some arrays only: the others keep their values
        new = torch.randn(ref[1].shape, generator=gen, device="cuda")
        s.set_state(None, new, None, None, 0.6, 0.6)
        got = s.get_state()
        for n, t in zip(NAMES, (ref[0], new, ref[2], ref[3])):
            assert torch.equal(got[n], t), n
        only = s.get_state(("psi2",))
        assert set(only) == {"psi2", "a_x", "a_v"} and torch.equal(only["psi2"], ref[3])
    finally:
        s.close()


def test_overlapping_copies_keep_their_order():
    """The same buffer for two outputs holds the later array, as sequential copies leave it."""
    from paper_1507_05329_amd.sim import ColaSim
    say("[gpu] state copies into one buffer")
    s = ColaSim(32, 64, 100.0)
    try:
        ref = [torch.randn_like(s.particles()) for _ in NAMES]
        s.set_state(*ref, 0.5, 0.5)
        one = s.particles()
        ax, av = ctypes.c_double(), ctypes.c_double()
        p = ctypes.c_void_p(one.data_ptr())
        assert s.lib.cola_get_state(s.ctx, p, p, p, p, ctypes.byref(ax), ctypes.byref(av)) == 0
        torch.cuda.synchronize()
        assert torch.equal(one, ref[3])
    finally:
        s.close()
