"""df_stream_dpd on both sides of the control-token size from which their copies
leave the graph's stream, page-locked and pageable, with rings of exactly two
batches, so that every token slot is reused while batches are in flight: the
bits of pushing, firing and popping batch by batch."""
import numpy as np
import pytest

from helpers import say
from workloads import complex_gaussian, dpd_coeffs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [2048, 4096, 8192, 16384])
@pytest.mark.parametrize("pinned", [True, False])
def test_streamed_tokens(nb, pinned):
    import torch
    from paper_1611_03226_amd import dfhip as D
    from paper_1611_03226_amd.graph import Graph
    r, B, M, n_batches = 8, 6, 8, 7
    say(f"stream_dpd of {nb} tokens a batch, pinned={pinned}")
    rng = np.random.default_rng(nb)
    n = nb * n_batches
    h = dpd_coeffs(rng, B, M)

    def host(a):
        t = torch.from_numpy(np.ascontiguousarray(a))
        return (t.pin_memory() if pinned else t).numpy()

    x, c = host(complex_gaussian(rng, n * r)), host(rng.integers(0, B + 1, n).astype(np.int32))
    y, ref = host(np.zeros(n * r, np.complex64)), np.zeros(n * r, np.complex64)
    with Graph(0) as G, Graph(0) as S:
        a, b = (g.dpd_chain(h, r, cap_x=2 * nb * r, cap_ctrl=2 * nb, cap_y=2 * nb * r) for g in (G, S))
        D.df_stream_dpd(G.g, a.actor, x, c, y, n_batches, nb)
        for k in range(n_batches):
            s = slice(k * nb * r, (k + 1) * nb * r)
            S.push(b.ctrl, c[k * nb:(k + 1) * nb])
            S.push(b.x, x[s])
            assert S.fire(b.actor, nb) == nb
            assert S.pop(b.y, ref[s]) == nb * r
        G.sync()
        S.sync()
    assert np.array_equal(y, ref)
