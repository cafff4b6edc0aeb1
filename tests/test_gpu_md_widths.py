"""Frame widths at the edges of the strip layout (a last strip that overlaps
its neighbour, 0..4 pixels right of a strip, rows and frames that start at any
byte), bit for bit against the oracle."""
import numpy as np
import pytest

from helpers import say
from oracle import md_paper as omd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W", [1, 3, 4, 8, 12, 15, 16, 17, 18, 19, 20, 21, 22, 23, 31, 32, 33, 34, 35, 36, 47, 49, 50, 51,
                               63, 65, 94, 333, 854])
@pytest.mark.parametrize("H", [3, 16, 21])
@pytest.mark.parametrize("chain", [False, True])
def test_widths_bit_exact(W, H, chain):
    from paper_1611_03226_amd.graph import Graph
    say(f"pipeline {W}x{H} chain={chain}")
    rng = np.random.default_rng(1000 * W + H)
    frames = rng.integers(0, 256, (12, H, W)).astype(np.uint8)
    frames[1::2] = np.clip(frames[0::2].astype(int) + rng.integers(-30, 31, (6, H, W)), 0, 255)
    out = np.zeros_like(frames)
    with Graph(0) as G:
        p = G.paper_motion_pipeline(W, H, 20, 4, cap=16)
        G.push(p.inp, frames)
        for n in (2, 1):
            if chain:
                assert p.fire_chain(G, n) == n
            else:
                p.fire_all(G, n)
        assert G.pop(p.out, out) == 12
        G.sync()
    assert np.array_equal(out, omd.paper_motion_direct(frames, 20))
