"""The order of the additions in the one-pass spectra, pinned bit for bit.

A host replay of the sums of |k| with the order that the kernel states: lanes along
nz, runs of one bin along the rows, the runs that end in a row handed over in lane
order, then the waves and the chunks.  In a box of 2 pi the fundamental is 1, so
|k| = sqrt(n2) and every addition is one IEEE operation."""
import math

import numpy as np
import pytest

from _progress import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

WAVES, MAX_CHUNKS, PARTIALS = 4, 1024, 3 * 4096 * 64


def threshold(e, strict=False):
    n = max(int(e * e) - 2, 0)
    while not (math.sqrt(n) > e if strict else math.sqrt(n) >= e):
        n += 1
    return n


def mean_k(ng, edges):
    """Mean |k| per bin and the mode counts, added as the kernel adds."""
    nb, h = len(edges) - 1, ng // 2
    nchunk = min(max(min(ng * ng // (16 * WAVES), MAX_CHUNKS), 1), PARTIALS // (nb * 3))
    nw, nrows = nchunk * WAVES, ng * ng
    per = -(-nrows // nw)
    thr = np.array([threshold(e) for e in edges])
    lo, hi = thr[0], min(thr[-1], threshold(math.pi * ng / (2.0 * math.pi), strict=True))
    acc, cnt = np.zeros((nw, nb)), np.zeros((nw, nb), np.int64)
    wave = np.arange(nw)
    for z0 in range(0, h + 1, 64):
        nz = z0 + np.arange(64)
        run, nrun, cur = np.zeros((nw, 64)), np.zeros((nw, 64), np.int64), np.full((nw, 64), -1)

        def hand_over(out):
            for w, lane in zip(*np.nonzero(out)):          # lane order within a wave
                acc[w, cur[w, lane]] += run[w, lane]
                cnt[w, cur[w, lane]] += nrun[w, lane]
            run[out], nrun[out] = 0.0, 0

        for i in range(per):
            r = wave * per + i
            sx, sy = r // ng, r % ng
            sx, sy = np.where(sx < h, sx, sx - ng), np.where(sy < h, sy, sy - ng)
            p2 = sx * sx + sy * sy
            visit = (r < np.minimum((wave + 1) * per, nrows)) & (p2 + z0 * z0 < hi)
            n2 = p2[:, None] + nz[None, :] ** 2
            half = (nz[None, :] > 0) | (sy[:, None] > 0) | ((sy[:, None] == 0) & (sx[:, None] > 0))
            counted = visit[:, None] & (nz[None, :] <= h) & (n2 >= lo) & (n2 < hi) & half
            b = np.where(counted, np.searchsorted(thr, n2, side="right") - 1, -1)
            hand_over(visit[:, None] & (nrun > 0) & (b != cur))
            cur = np.where(counted, b, cur)
            run += np.where(counted, np.sqrt(n2.astype(np.float64)), 0.0)
            nrun += counted
        hand_over(nrun > 0)
    chunk = np.zeros((nchunk, nb))
    for w in range(WAVES):
        chunk += acc[w::WAVES]
    s = np.zeros((256, nb))
    for c in range(nchunk):
        s[c % 256] += chunk[c]
    o = 128
    while o:
        s[:o] += s[o:2 * o]
        o //= 2
    n = cnt.sum(axis=0)
    with np.errstate(invalid="ignore"):
        return s[0] / n, n


@pytest.mark.parametrize("ng,nbins", [(32, 1), (32, 9), (96, 5), (96, 300), (192, 1), (192, 40), (192, 400)])
def test_mean_k_in_the_stated_order(ng, nbins):
    from paper_1507_05329_amd.sim import ColaSim
    say(f"[gpu] mean |k| in order, {nbins} bins on {ng}^3")
    edges = np.linspace(0.7, 0.49 * ng, nbins + 1) if nbins < 40 else np.geomspace(0.7, 0.55 * ng, nbins + 1)
    sim = ColaSim(32, ng, 2.0 * math.pi)
    try:
        z = sim.particles().zero_()
        sim.set_state(z, z, z, z, 0.5, 0.5)
        km, _, n = sim.pk(edges)
        _, _, _, _, nv = sim.pk_velocity(edges, axis=0) if nbins <= 300 else (None,) * 4 + (n,)
    finally:
        sim.close()
    want, modes = mean_k(ng, edges)
    assert np.array_equal(n, modes) and np.array_equal(nv, modes)
    assert np.array_equal(km, want, equal_nan=True)
