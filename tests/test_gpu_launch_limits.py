"""Stateless calls of so many short rows that one workgroup per row, or per
few firings, would be more threads than a launch has: every row equals the
same row of a call of its own few rows."""
import numpy as np
import pytest

from helpers import DPD_TOL, say
from oracle import dpd as odpd

pytestmark = pytest.mark.gpu


# 2^22 rows of 16 branches: a scan of 1024 threads a row; 2^25 firings of
# three taps: a head pass of 256 threads for two firings
@pytest.mark.parametrize("S,nf,r,B,M", [((1 << 22) + 3, 1, 1, 16, 1), ((1 << 19) + 1, 64, 2, 1, 3)])
def test_many_short_rows(S, nf, r, B, M):
    import torch
    from paper_1611_03226_amd import dfhip as D
    say(f"{S} rows of {nf} firings of {r}, {B} branches, {M} taps")
    g = torch.Generator(device="cuda").manual_seed(S)
    x = torch.view_as_complex(torch.randn(S, nf * r, 2, device="cuda", generator=g) * 0.5)
    ctrl = torch.randint(0, B + 1, (S, nf), device="cuda", generator=g, dtype=torch.int32)
    h = torch.view_as_complex(torch.randn(B, M, 2, device="cuda", generator=g) * 0.3)
    y = torch.empty_like(x)
    D.df_dpd_forward(x, ctrl, h, y, r)
    for at in (0, S // 2, S - 1000):
        part = slice(at, at + 1000)
        ref = torch.empty_like(x[part])
        D.df_dpd_forward(x[part].contiguous(), ctrl[part].contiguous(), h, ref, r)
        assert torch.equal(y[part], ref)
    last = slice(S - 20, S)
    want = odpd.run_dpd_streams(x[last].cpu().numpy(), ctrl[last].cpu().numpy(), h.cpu().numpy(), r, "branch")
    assert np.linalg.norm(y[last].cpu().numpy() - want) <= DPD_TOL * np.linalg.norm(want)
