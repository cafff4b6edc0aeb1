"""Output stores of the predistortion body: whole wavefronts through LDS,
the last wavefront of a firing, positions off 16-byte alignment and ring wrap
directly.  Every tile shape gives the same bits, and the oracle's values."""
import numpy as np
import pytest

from helpers import DPD_TOL, rel_rms_per_firing, say
from oracle import dpd as odpd
from workloads import dpd_random

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [255, 256, 257, 511, 512, 513, 1024, 2050, 4096])
@pytest.mark.parametrize("M", [4, 16, 11])
def test_shapes_give_the_same_bits(r, M):
    from paper_1611_03226_amd.graph import Graph
    n, cap = 67, 1 << 18
    w = dpd_random(50 + r, n_firings=n, r=r, n_branches_max=6, n_taps=M, ctrl_low=0)
    outs = []
    for tile in ((256, 4, 0), (1024, 4, 0), (512, 8, 0), (2048, 8, 0)):
        say(f"stores r={r} M={M} tile={tile}")
        with Graph(0) as G:
            G.set_tile(*tile)
            ch = G.dpd_chain(w.h, r, cap_x=cap, cap_ctrl=256, cap_y=cap)
            y = np.zeros(n * r, np.complex64)
            at = 0
            while at < n:                                # batches that cross the rings' ends
                k = min(n - at, max(1, cap // (2 * r) - 1), 66)
                G.push(ch.ctrl, w.ctrl[at:at + k])
                G.push(ch.x, w.x[at * r:(at + k) * r])
                assert G.fire(ch.actor, k) == k
                assert G.pop(ch.y, y[at * r:(at + k) * r]) == k * r
                at += k
            G.sync()
            outs.append(y)
    for y in outs[1:]:
        assert np.array_equal(outs[0], y)
    worst, _, bad = rel_rms_per_firing(outs[0], odpd.run_dpd(w.x, w.ctrl, w.h, r, w.n_delay), r)
    assert worst <= DPD_TOL and bad == 0


def test_many_instances_of_large_tiles():
    """4096 outputs a tile (stored directly: no room for the buffer) and 2048
    (through LDS), several instances in one launch."""
    from paper_1611_03226_amd.graph import Graph
    r, nf = 8195, [3, 70, 1]
    ws = [dpd_random(60 + i, n_firings=n, r=r, n_branches_max=6, n_taps=8, ctrl_low=0) for i, n in enumerate(nf)]
    outs = []
    for tile in ((4096, 8, 0), (2048, 8, 0), (256, 4, 0)):
        say(f"instances tile={tile}")
        with Graph(0) as G:
            G.set_tile(*tile)
            chains = [G.dpd_chain(w.h, r, cap_x=1 << 20, cap_ctrl=128, cap_y=1 << 20) for w in ws]
            for ch, w in zip(chains, ws):
                G.push(ch.ctrl, w.ctrl)
                G.push(ch.x, w.x)
            G.fire_many([ch.actor for ch in chains], nf, persistent=True, graph=False)
            ys = [np.zeros(w.x.size, np.complex64) for w in ws]
            for ch, y in zip(chains, ys):
                assert G.pop(ch.y, y) == y.size
            G.sync()
            outs.append(np.concatenate(ys))
    assert np.array_equal(outs[0], outs[1]) and np.array_equal(outs[0], outs[2])
