"""Motion actor over the shapes its bits pass selects (frames per wavefront,
band heights), frame widths that start rows at any byte, and the emitted-count
read-back, bit for bit against the oracle."""
import numpy as np
import pytest

from helpers import say
from oracle import motion as omo
from workloads import motion as gen_motion

pytestmark = pytest.mark.gpu


def _run(frames, self_delay, batches):
    from paper_1611_03226_amd.graph import Graph
    n, H, W = frames.shape
    masks, idx = np.zeros((n, H, W), np.uint8), np.zeros(n, np.int64)
    got = 0
    with Graph(0) as G:
        mc = G.motion_chain(W, H, self_delay=self_delay, cap_in=1 << (n + 1).bit_length(), cap_out=1 << n.bit_length())
        G.push(mc.cur, frames)
        if not self_delay:
            G.push(mc.prev, frames)
        for k, b in enumerate(batches):
            assert G.fire(mc.actor, b) == b
            if k % 2:                                    # counts of two batches read at once, and of one
                m = G.pop(mc.mask, masks[got:])
                assert G.pop(mc.index, idx[got:]) == m
                got += m
        m = G.pop(mc.mask, masks[got:])
        assert G.pop(mc.index, idx[got:]) == m
        assert G.status(mc.mask)[1] == G.status(mc.index)[1] == got + m
        G.sync()
    return masks[:got + m], idx[:got + m]


@pytest.mark.parametrize("W,H,n", [(1, 3, 5), (5, 9, 7), (31, 40, 6), (33, 17, 9), (63, 8, 5), (64, 33, 11), (99, 70, 20),
                                   (1985, 33, 4), (1983, 65, 3), (320, 240, 26), (333, 251, 40), (320, 96, 700),
                                   (1920, 64, 1100), (1920, 64, 2100)])
@pytest.mark.parametrize("self_delay", [True, False])
def test_shapes_bit_exact(W, H, n, self_delay):
    say(f"motion {W}x{H}x{n} self_delay={self_delay}")
    if n > 100:                                          # many frames: noise blocks, cheap to make
        rng = np.random.default_rng(n + W)
        frames = np.repeat(rng.integers(0, 256, (1, H, W)), n, 0).astype(np.uint8)
        for t in range(0, n, 3):
            frames[t, t % (H - 8):t % (H - 8) + 8, (5 * t) % (W - 40):(5 * t) % (W - 40) + 40] ^= 0x80
        frames[n - 1, -1, -1] ^= 0x40
    else:
        s = max(2, min(W, H) // 3)
        frames = gen_motion(seed=W + H + n, n_frames=n, width=W, height=H, rect_min=min(2, s), rect_max=s, segment=2).frames
    masks, idx = _run(frames, self_delay, [n] if n > 100 else [n // 3, n // 3, n - 2 * (n // 3)])
    ref_m, ref_i = omo.run_motion(frames)
    assert np.array_equal(idx, ref_i) and np.array_equal(masks, ref_m)
