"""Pushes and pops whose buffer is declared device memory but is not, or ends
before the tokens do: the runtime copy serves page-locked host memory and
refuses a range past an allocation's end, so that no kernel runs into it."""
import ctypes as C

import numpy as np
import pytest

from helpers import say

pytestmark = pytest.mark.gpu


def _push(D, G, f, ptr, n):
    return D._lib.df_push(G.g, f, ptr, n, 1)


def test_pinned_host_memory_as_device_memory():
    import torch
    from paper_1611_03226_amd import dfhip as D
    from paper_1611_03226_amd.graph import Graph
    say("push / pop of page-locked host memory declared device memory")
    src = torch.arange(1000, dtype=torch.int64).pin_memory()
    dst = torch.zeros(1000, dtype=torch.int64).pin_memory()
    with Graph(0) as G:
        f = G.fifo(D.DF_I64, 1, 1024)
        got = C.c_int64()
        assert _push(D, G, f, src.data_ptr(), 1000) == D.DF_OK
        assert D._lib.df_pop(G.g, f, dst.data_ptr(), 1000, 1, C.byref(got)) == D.DF_OK and got.value == 1000
        G.sync()
    assert torch.equal(src, dst)


@pytest.mark.parametrize("pop", [False, True])
def test_range_past_the_allocation_is_refused(pop):
    """An allocation of 4 MiB of its own, tokens for 6 MiB."""
    import torch
    from paper_1611_03226_amd import dfhip as D
    from paper_1611_03226_amd.graph import Graph
    say(f"range past the end of an allocation, pop={pop}")
    hip = C.CDLL("libamdhip64.so")
    buf = C.c_void_p()
    assert hip.hipMalloc(C.byref(buf), C.c_size_t(4 << 20)) == 0
    try:
        n = 6 << 17
        with Graph(0) as G:
            f = G.fifo(D.DF_I64, 1, 1 << 20)
            if pop:
                G.push(f, np.arange(n, dtype=np.int64))
                got = C.c_int64(7)
                st = D._lib.df_pop(G.g, f, buf, n, 1, C.byref(got))
            else:
                st = _push(D, G, f, buf, n)
            assert st == D.DF_EDEVICE
            hip.hipGetLastError()                        # the refused call's, else the next launch would report it
    finally:
        hip.hipFree(buf)
    torch.cuda.synchronize()                             # and nothing is left to fail


def test_push_and_pop_are_capturable():
    """The buffer checks ask nothing that a stream capture forbids."""
    import torch
    from paper_1611_03226_amd import dfhip as D
    from paper_1611_03226_amd.graph import Graph
    say("push and pop under capture")
    s = torch.cuda.Stream()
    src = torch.arange(100, dtype=torch.int64, device="cuda")
    dst = torch.zeros(100, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    with Graph(0, stream=s) as G:
        f = G.fifo(D.DF_I64, 1, 128)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            G.push(f, src)
            assert G.pop(f, dst) == 100
        assert int(dst.abs().sum()) == 0
        with torch.cuda.stream(s):
            g.replay()
        G.sync()
    assert torch.equal(src, dst)
