"""Tap counts that are not compiled in (a run-time tap loop): the edges of its
four- and eight-tap turns, one tap, the largest count, both tile shapes, ring
wrap and unaligned output pairs, against the oracle."""
import numpy as np
import pytest

from helpers import DPD_TOL, rel_rms_per_firing, run_dpd_chain, say
from oracle import dpd as odpd
from workloads import dpd_random

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 2, 3, 5, 6, 7, 9, 10, 12, 13, 15, 17, 24, 31, 32])
@pytest.mark.parametrize("hist", ["branch", "shared"])
def test_tap_counts_match_oracle(M, hist):
    from paper_1611_03226_amd.graph import Graph
    for B, r, n, cap in ((10, max(M, 37), 70, 0), (13, 300, 9, 1024)):
        say(f"taps M={M} B={B} r={r} {hist}")
        w = dpd_random(700 + M, n_firings=n, r=r, n_branches_max=B, n_taps=M, n_delay=1, ctrl_low=0)
        with Graph(0) as G:
            y, _ = run_dpd_chain(G, w, hist=hist, batches=[3] * (n // 3) + ([n % 3] if n % 3 else []) if cap else [n],
                                 cap_x=cap)
        ref = odpd.run_dpd(w.x, w.ctrl, w.h, w.r, w.n_delay, hist=hist)
        worst, _, bad = rel_rms_per_firing(y, ref, r)
        assert worst <= DPD_TOL and bad == 0


@pytest.mark.parametrize("M", [4, 8, 16, 10, 31])
@pytest.mark.parametrize("control", ["count", "mask"])
def test_large_tiles_equal_small_ones(M, control):
    """The batch size selects eight outputs per thread; the same batch with
    four per thread, and fired in two parts (output positions off 16-byte
    alignment), gives the same bits."""
    from paper_1611_03226_amd.graph import Graph
    r, n, B = 2051, 260, 10
    say(f"large tiles M={M} {control}")
    w = dpd_random(90 + M, n_firings=n, r=r, n_branches_max=B, n_taps=M, ctrl_low=0)
    rng = np.random.default_rng(M)
    ctrl = rng.integers(0, 1 << B, n).astype(np.int32) if control == "mask" else w.ctrl
    outs = []
    for tile, parts in ((None, [n]), ((1024, 4, 0), [n]), (None, [259, 1])):
        with Graph(0) as G:
            if tile:
                G.set_tile(*tile)
            ch = G.dpd_chain(w.h, r, control=control, cap_x=1 << 20, cap_ctrl=512, cap_y=1 << 20)
            G.push(ch.ctrl, ctrl)
            G.push(ch.x, w.x)
            for k in parts:
                assert G.fire(ch.actor, k) == k
            y = np.zeros(n * r, np.complex64)
            assert G.pop(ch.y, y) == n * r
            G.sync()
            outs.append(y)
    assert np.array_equal(outs[0], outs[1]) and np.array_equal(outs[0], outs[2])
