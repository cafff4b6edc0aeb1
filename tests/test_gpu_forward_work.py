"""Forward and coefficient adjoint in the caller's scratch: the same bits as
the allocating calls, buffers checked, a changed control tensor reported, and
the same results through saved-tensor hooks and on a side stream."""
import numpy as np
import pytest

from helpers import say
from workloads import complex_gaussian, dpd_coeffs

pytestmark = pytest.mark.gpu


def _case(S, nf, r, B, M):
    import torch
    rng = np.random.default_rng(S + nf + M)
    x, g = (torch.from_numpy(complex_gaussian(rng, (S, nf * r))).cuda() for _ in range(2))
    h = torch.from_numpy(dpd_coeffs(rng, B, M)).cuda()
    ctrl = torch.from_numpy(rng.integers(0, B + 1, (S, nf)).astype(np.int32)).cuda()
    return x, g, h, ctrl


@pytest.mark.parametrize("S,nf,r,B,M", [(3, 7, 40, 5, 8), (2, 600, 33, 10, 16), (1, 3, 5000, 16, 11)])
@pytest.mark.parametrize("hist", [0, 1])
def test_same_bits_as_the_allocating_calls(S, nf, r, B, M, hist):
    import torch
    from paper_1611_03226_amd import dfhip as D
    say(f"forward work S={S} nf={nf} r={r} B={B} M={M} hist={hist}")
    x, g, h, ctrl = _case(S, nf, r, B, M)
    for c in (ctrl, None):
        y0, y1 = torch.empty_like(x), torch.empty_like(x)
        D.df_dpd_forward(x, c, h, y0, r, hist)
        work = torch.empty(D.df_dpd_forward_work_bytes(S, nf * r, r, B, M, c is not None), dtype=torch.uint8, device="cuda")
        tables = None if c is None else torch.empty(D.df_dpd_tables_bytes(S, nf * r, r, B), dtype=torch.uint8, device="cuda")
        D.df_dpd_forward_work(x, c, h, y1, r, tables, work, hist)
        torch.cuda.synchronize()
        assert torch.equal(y0, y1)
        if c is None:
            continue
        aw = torch.empty(D.df_dpd_coeff_adjoint_work_bytes(S, nf * r, r, B, M), dtype=torch.uint8, device="cuda")
        g0, g1 = torch.empty_like(h), torch.empty_like(h)
        D.df_dpd_coeff_adjoint(x, c, g, g0, r, aw, hist)
        D.df_dpd_coeff_adjoint_tables(x, tables, g, g1, r, aw)
        torch.cuda.synchronize()
        assert torch.equal(g0, g1)
        for bad in ((tables[:-8], work), (tables, work[:-8])):
            with pytest.raises(D.DFError):
                D.df_dpd_forward_work(x, c, h, y1, r, *bad, hist)
        with pytest.raises(D.DFError):
            D.df_dpd_coeff_adjoint_tables(x, tables[:-8], g, g1, r, aw)


def test_layer_hooks_streams_and_changed_control():
    import torch
    from paper_1611_03226_amd.autograd import DPDFunction
    say("layer through saved-tensor hooks and a side stream")
    x, g, h, ctrl = _case(4, 9, 64, 6, 12)

    def grads():
        hh = h.clone().requires_grad_(True)
        y = DPDFunction.apply(x, hh, 64, ctrl)
        y.backward(g)
        return y.detach(), hh.grad

    y0, g0 = grads()
    with torch.autograd.graph.save_on_cpu():
        y1, g1 = grads()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        y2, g2 = grads()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    for y, gr in ((y1, g1), (y2, g2)):
        assert torch.equal(y, y0) and torch.equal(gr, g0)
    hh = h.clone().requires_grad_(True)
    y = DPDFunction.apply(x, hh, 64, ctrl)
    ctrl[0, 0] = 1
    with pytest.raises(RuntimeError):
        y.backward(g)
