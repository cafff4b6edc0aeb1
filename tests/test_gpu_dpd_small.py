"""Batches of at most 64 firings (one launch) beside larger ones (scan, head
pass and body): the same bits for every way of cutting a control sequence into
batches around 64, with the same tables, history carried over reactivations,
errors reported, and all tap counts, histories and control modes."""
import numpy as np
import pytest

from helpers import DPD_TOL, rel_rms_per_firing, say
from oracle import dpd as odpd
from workloads import dpd_random

pytestmark = pytest.mark.gpu


def _fire(w, ctrl, hist, control, batches, tables=False):
    from paper_1611_03226_amd import dfhip as D
    from paper_1611_03226_amd.graph import Graph
    n = len(ctrl)
    y = np.zeros(n * w.r, np.complex64)
    with Graph(0) as G:
        p2 = 1 << int(n * w.r + w.n_delay).bit_length()
        ch = G.dpd_chain(w.h, w.r, w.n_delay, history=hist, control=control, cap_x=p2, cap_ctrl=256, cap_y=p2)
        G.push(ch.ctrl, ctrl)
        G.push(ch.x, w.x)
        tab = []
        for k in batches:
            assert G.fire(ch.actor, k) == k
            if tables:
                tab.append(D.df_debug_last_batch(G.g, ch.actor, w.n_branches_max, 256))
        assert G.pop(ch.y, y) == n * w.r
        G.sync()
    return y, tab


@pytest.mark.parametrize("M", [1, 4, 8, 16, 10, 17, 32])
@pytest.mark.parametrize("hist,control", [("branch", "count"), ("shared", "count"), ("branch", "mask")])
def test_batches_around_64_are_bit_identical(M, hist, control):
    for B, r in ((10, 40), (16, 1100)):
        n = 130
        say(f"small batches M={M} B={B} r={r} {hist} {control}")
        w = dpd_random(50 + M, n_firings=n, r=r, n_branches_max=B, n_taps=M, n_delay=2, ctrl_low=0)
        rng = np.random.default_rng(M + B)
        ctrl = rng.integers(0, 1 << B, n).astype(np.int32) if control == "mask" else w.ctrl
        outs = [_fire(w, ctrl, hist, control, b)[0] for b in ([130], [64, 64, 2], [65, 65], [1] * 5 + [63, 62], [3, 64, 63])]
        for o in outs[1:]:
            assert np.array_equal(o, outs[0])
        if control == "count":
            ref = odpd.run_dpd(w.x, ctrl, w.h, w.r, w.n_delay, hist=hist)
            assert rel_rms_per_firing(outs[0], ref, r)[0] <= DPD_TOL


@pytest.mark.parametrize("hist", ["branch", "shared"])
@pytest.mark.parametrize("n", [1, 2, 63, 64])
def test_tables_match_oracle(hist, n):
    say(f"small batch tables n={n} {hist}")
    w = dpd_random(60 + n, n_firings=n, r=16, n_branches_max=7, n_taps=8, ctrl_low=0)
    _, tab = _fire(w, w.ctrl, hist, "count", [n], tables=True)
    rates, offs, prev = odpd.firing_tables(w.ctrl, 7, w.r, hist=hist)[:3]
    for got, want in zip(tab[0], (rates, offs, prev)):
        assert np.array_equal(got, want)


def test_bad_device_token_is_an_empty_set_and_reported():
    import torch
    from paper_1611_03226_amd import dfhip as D
    from paper_1611_03226_amd.graph import Graph
    say("small batch with an out-of-range token")
    w = dpd_random(77, n_firings=9, r=50, n_branches_max=5, n_taps=8, ctrl_low=1)
    bad, zero = w.ctrl.copy(), w.ctrl.copy()
    bad[4], zero[4] = 6, 0
    y = np.zeros(9 * 50, np.complex64)
    with Graph(0) as G:
        ch = G.dpd_chain(w.h, w.r, cap_x=512, cap_ctrl=16, cap_y=512)
        G.push(ch.ctrl, torch.from_numpy(bad).cuda())
        G.push(ch.x, w.x)
        G.fire(ch.actor, 9)
        G.pop(ch.y, y)
        with pytest.raises(D.DFError) as e:
            G.sync()
        assert e.value.code == D.DF_ECONTROL
    assert np.array_equal(y, _fire(w, zero, "branch", "count", [9])[0])
