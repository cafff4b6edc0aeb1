"""Emitted-count read-back of the motion actor: batches replayed from a
captured graph between eager ones, and the status call's synchronisation."""
import numpy as np
import pytest

from helpers import say
from oracle import motion as omo

pytestmark = pytest.mark.gpu


def _frames(n, W, H, seed):
    return np.random.default_rng(seed).integers(0, 256, (n, H, W)).astype(np.uint8)


@pytest.mark.parametrize("order", ["erer", "eerr", "rere"])
def test_counts_include_replayed_batches(order):
    """Batches run eagerly (e) and by replay (r): a pop moves the frames of
    every batch that ran, also behind an eager batch fired after the capture."""
    import torch
    from paper_1611_03226_amd.graph import Graph
    say(f"motion counts over replays {order}")
    W, H, k = 70, 33, 4
    frames = _frames(k * (len(order) + 1), W, H, 5)
    s = torch.cuda.Stream()
    with Graph(0, stream=s) as G:
        mc = G.motion_chain(W, H, permille=0, self_delay=False, cap_in=64, cap_out=64)
        G.push(mc.cur, frames)
        G.push(mc.prev, frames)
        assert G.fire(mc.actor, k) == k                  # the scratch is there before the capture
        G.sync()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            assert G.fire(mc.actor, k) == k
        for o in order:
            if o == "e":
                assert G.fire(mc.actor, k) == k
            else:
                with torch.cuda.stream(s):
                    g.replay()
        out = np.zeros((len(frames) + 1, H, W), np.uint8)
        assert G.pop(mc.mask, out) == len(frames)
        assert G.status(mc.index)[1] == len(frames)
        G.sync()
    ref, idx = omo.run_motion(frames, permille=0)
    assert len(idx) == len(frames) and np.array_equal(out[:-1], ref)


def test_status_synchronises():
    """The status of a channel with a data-dependent producer waits for the
    graph's stream, also behind a pop that did not have to."""
    import torch
    from paper_1611_03226_amd.graph import Graph
    say("motion status waits for the stream")
    W, H, k = 64, 48, 6
    frames = _frames(k, W, H, 6)
    s = torch.cuda.Stream()
    with Graph(0, stream=s) as G:
        mc = G.motion_chain(W, H, permille=0, cap_in=16, cap_out=16)
        dst = torch.zeros(k, H, W, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        for pop_first in (False, True):
            G.push(mc.cur, frames[:k // 2])
            assert G.fire(mc.actor, k // 2) == k // 2
            if pop_first:
                assert G.pop(mc.mask, dst) == k
            with torch.cuda.stream(s):
                torch.cuda._sleep(200_000_000)           # about a tenth of a second
            assert G.status(mc.mask)[1] == (k if pop_first else k // 2)
            assert s.query()
        G.sync()
