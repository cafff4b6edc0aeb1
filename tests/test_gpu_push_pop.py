"""Device push and pop (one kernel for the copy and the counter): tokens of
odd byte sizes, runs that wrap, both sides at any alignment, sizes at the
edges of a thread's and a workgroup's share and of the streamed form, and the
paper's channel layout, against the host's view of the same tokens."""
import numpy as np
import pytest

from helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("elems,cap,counts", [(1, 64, [1, 15, 16, 17, 33, 64]), (3, 32, [1, 5, 21, 32]), (77, 64, [53, 64, 64]),
                                              (4096, 16, [1, 15, 16]), (4099, 8, [3, 8, 5]),
                                              (1 << 20, 128, [65, 63, 127, 128])])
@pytest.mark.parametrize("offset", [0, 1, 7])
def test_bytes_through_a_ring(elems, cap, counts, offset):
    import torch
    from paper_1611_03226_amd import dfhip as D
    from paper_1611_03226_amd.graph import Graph
    say(f"push/pop tokens of {elems} bytes, capacity {cap}, offset {offset}")
    with Graph(0) as G:
        f = D.df_fifo_create(G.g, D.DF_U8, elems, cap)
        done = 0
        for k, n in enumerate(counts):
            src = torch.randint(0, 256, (n * elems + 16,), dtype=torch.uint8, device="cuda")
            dst = torch.full((n * elems + 32,), 7, dtype=torch.uint8, device="cuda")
            torch.cuda.synchronize()
            G.push(f, src[offset:offset + n * elems])
            assert G.pop(f, dst[8 + offset:8 + offset + n * elems]) == n
            G.sync()
            done += n
            assert torch.equal(dst[8 + offset:8 + offset + n * elems], src[offset:offset + n * elems])
            assert bool((dst[:8 + offset] == 7).all()) and bool((dst[8 + offset + n * elems:] == 7).all())
            assert D.df_fifo_status(G.g, f) == (done, done, cap)


@pytest.mark.parametrize("delay", [0, 1])
def test_paper_layout_from_device_equals_from_host(delay):
    import torch
    from paper_1611_03226_amd import dfhip as D
    from paper_1611_03226_amd.graph import Graph
    say(f"paper layout, delay {delay}, device push and pop")
    rate, elems = 3, 21
    rng = np.random.default_rng(delay)
    with Graph(0) as G, Graph(0) as R:
        init = rng.integers(0, 256, (delay, elems)).astype(np.uint8) if delay else None
        f, q = (D.df_fifo_create_paper(g.g, D.DF_U8, elems, rate, delay, init) for g in (G, R))
        for k in range(9):
            t = rng.integers(0, 256, (rate, elems)).astype(np.uint8)
            d, out, ref = torch.from_numpy(t).cuda(), torch.zeros(rate, elems, dtype=torch.uint8, device="cuda"), np.zeros_like(t)
            torch.cuda.synchronize()
            G.push(f, d)
            R.push(q, t)
            assert G.pop(f, out) == R.pop(q, ref) == rate
            G.sync()
            assert np.array_equal(out.cpu().numpy(), ref)
            if k:                                        # every slot of the layout has been written
                assert k < 3 or np.array_equal(D.df_debug_read_slots(G.g, f), D.df_debug_read_slots(R.g, q))
