"""Stateless calls with control tokens at the edges of the one-launch scan
(rows of 1, 63..65, 511..513 firings, one and many branches), against the
oracle: forward, coefficient adjoint and network form."""
import numpy as np
import pytest

from helpers import DPD_TOL, say
from oracle import dpd as odpd
from oracle import pa as opa
from workloads import complex_gaussian, dpd_coeffs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,nf", [(1, 1), (5, 1), (3, 63), (2, 64), (2, 65), (2, 511), (1, 512), (2, 513), (300, 2)])
@pytest.mark.parametrize("B,M,hist", [(1, 4, "branch"), (16, 9, "branch"), (7, 8, "shared")])
def test_rows_match_oracle(S, nf, B, M, hist):
    import torch
    from paper_1611_03226_amd import dfhip as D
    say(f"scan rows S={S} nf={nf} B={B} M={M} {hist}")
    rng = np.random.default_rng(S * 1000 + nf + B)
    r = 12
    x = complex_gaussian(rng, (S, nf * r))
    g = complex_gaussian(rng, (S, nf * r))
    h = dpd_coeffs(rng, B, M)
    ctrl = rng.integers(-1, B + 2, (S, nf)).astype(np.int32)     # out-of-range tokens count as 0
    valid = np.where((ctrl >= 0) & (ctrl <= B), ctrl, 0).astype(np.int32)
    dev = [torch.from_numpy(a).cuda() for a in (x, ctrl, h, g)]
    y, yn = torch.empty_like(dev[0]), torch.empty_like(dev[0])
    H = D.DF_HIST_SHARED if hist == "shared" else D.DF_HIST_BRANCH
    D.df_dpd_forward(dev[0], dev[1], dev[2], y, r, H)
    grad = torch.empty(B, M, dtype=torch.complex64, device="cuda")
    work = torch.empty(D.df_dpd_coeff_adjoint_work_bytes(S, nf * r, r, B, M), dtype=torch.uint8, device="cuda")
    D.df_dpd_coeff_adjoint(dev[0], dev[1], dev[3], grad, r, work, H)
    if hist == "branch":
        D.df_dpd_forward_network(dev[0], dev[1], dev[2], yn, r)
    torch.cuda.synchronize()
    ref = odpd.run_dpd_streams(x, valid, h, r, hist)
    n = np.linalg.norm(ref)
    assert np.linalg.norm(y.cpu().numpy() - ref) <= DPD_TOL * max(n, 1e-30)
    if hist == "branch":
        assert np.linalg.norm(yn.cpu().numpy() - ref) <= DPD_TOL * max(n, 1e-30)
    gref = opa.dpd_coeff_vjp_streams(x, valid, g, B, M, r, hist)
    assert np.linalg.norm(grad.cpu().numpy() - gref) <= DPD_TOL * max(np.linalg.norm(gref), 1e-30)
