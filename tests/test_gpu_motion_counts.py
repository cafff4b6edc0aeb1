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


@pytest.mark.parametrize("self_delay", [True, False])
def test_batch_beyond_one_launch(self_delay):
    """More firings than one launch's grid rows, in one batch and in batches of
    a few thousand: the same masks and indices, and the right state behind."""
    import torch
    from paper_1611_03226_amd.graph import Graph
    n, H, W = 65600, 5, 9
    say(f"motion batch of {n} firings, self_delay={self_delay}")
    frames = np.repeat(np.random.default_rng(3).integers(0, 256, (1, H, W)), n, 0).astype(np.uint8)
    frames[1::7, 1:4, 2:6] ^= 0x80
    frames[65533:65537] = np.random.default_rng(4).integers(0, 256, (4, H, W)) // 128 * 255
    out = []
    for step in (n, 4100):
        with Graph(0) as G:
            mc = G.motion_chain(W, H, self_delay=self_delay, cap_in=1 << 17, cap_out=1 << 17)
            G.push(mc.cur, frames)
            if not self_delay:
                G.push(mc.prev, frames)
            for k in range(0, n, step):
                assert G.fire(mc.actor, min(step, n - k)) == min(step, n - k)
            m, i = np.zeros((n, H, W), np.uint8), np.zeros(n, np.int64)
            got = G.pop(mc.mask, m)
            assert G.pop(mc.index, i) == got
            G.sync()
            out.append((m[:got], i[:got]))
    assert np.array_equal(out[0][1], out[1][1]) and np.array_equal(out[0][0], out[1][0])
    lo = 65520
    ref_m, ref_i = omo.run_motion(frames[lo:])           # its first frame sees the zero frame
    late = out[0][1] > lo
    assert np.array_equal(out[0][1][late], ref_i[ref_i > 0] + lo)
    assert np.array_equal(out[0][0][late], ref_m[ref_i > 0])


def test_many_actors_share_the_page_locked_words():
    """More motion actors than one page has words, some destroyed and made again
    in between: every actor pops its own frames."""
    from paper_1611_03226_amd.graph import Graph
    say("300 motion actors")
    W, H = 32, 6
    f = _frames(5, W, H, 9)
    ref = {n: omo.run_motion(f[:n], permille=0)[0] for n in range(1, 6)}
    graphs = []

    def make(k):
        G = Graph(0)
        chains = [G.motion_chain(W, H, permille=0, cap_in=8, cap_out=8) for _ in range(30)]
        for i, mc in enumerate(chains):
            n = 1 + (i + k) % 5
            G.push(mc.cur, f[:n])
            assert G.fire(mc.actor, n) == n
        return G, chains, k

    for k in range(10):
        graphs.append(make(k))
    for k in (1, 4, 8):
        graphs[k][0].close()
        graphs[k] = make(k + 2)
    for G, chains, k in graphs:
        for i, mc in enumerate(chains):
            n, out = 1 + (i + k) % 5, np.zeros((8, H, W), np.uint8)
            assert G.pop(mc.mask, out) == n
            assert np.array_equal(out[:n], ref[n])
        G.close()
