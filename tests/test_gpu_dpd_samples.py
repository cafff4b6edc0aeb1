"""Batches that run sample by sample (short firings, tap counts that are not
compiled in): bit for bit what the same firings give in batches of at most 64,
which run in tiles, infinities and NaN among the samples; and the oracle, also
for stateless rows with and without control tokens."""
import numpy as np
import pytest

from helpers import DPD_TOL, rel_rms_per_firing, say
from oracle import dpd as odpd
from workloads import complex_gaussian, dpd_coeffs

pytestmark = pytest.mark.gpu


def _pow2(n):
    return 1 << max(0, int(n - 1).bit_length())


@pytest.mark.parametrize("B,M,r", [(1, 1, 1), (4, 1, 7), (2, 2, 1), (3, 3, 2), (16, 5, 4), (6, 7, 6), (10, 9, 8), (6, 12, 11)])
@pytest.mark.parametrize("control,hist", [("count", "branch"), ("mask", "branch"), ("count", "shared")])
@pytest.mark.parametrize("special", [False, True])
def test_one_batch_equals_small_batches(B, M, r, control, hist, special):
    from paper_1611_03226_amd.graph import Graph
    n, delay = 30011, 1 if M > 1 else 0
    say(f"samples B={B} M={M} r={r} {control} {hist} special={special}")
    rng = np.random.default_rng(100 * B + M)
    x = complex_gaussian(rng, n * r, rms=0.6)
    if special:
        at = rng.integers(0, n * r, 40)
        x[at] = np.array([np.inf, -np.inf, np.nan, 1e30])[rng.integers(0, 4, 40)] + 1j * x[at].imag
    h = dpd_coeffs(rng, B, M)
    ctrl = rng.integers(0, 1 << B if control == "mask" else B + 1, n).astype(np.int32)
    outs = []
    for step in (n, 61):
        y = np.zeros(n * r, np.complex64)
        with Graph(0) as G:
            ch = G.dpd_chain(h, r, delay, history=hist, control=control, cap_x=_pow2(n * r + delay), cap_ctrl=_pow2(n),
                             cap_y=_pow2(n * r))
            G.push(ch.ctrl, ctrl)
            G.push(ch.x, x)
            for k in range(0, n, step):
                assert G.fire(ch.actor, min(step, n - k)) == min(step, n - k)
            assert G.pop(ch.y, y) == n * r
            G.sync()
        outs.append(y)
    assert np.array_equal(outs[0].view(np.float32), outs[1].view(np.float32), equal_nan=True)
    if not special:
        m = 400
        ref = odpd.run_dpd(x[:m * r], ctrl[:m], h, r, n_delay=delay, hist=hist, control=control)[:m * r]
        worst, _, bad0 = rel_rms_per_firing(outs[0][:m * r], ref, r)
        assert worst <= DPD_TOL and bad0 == 0


@pytest.mark.parametrize("B,M,S,L", [(4, 7, 3, 1000), (1, 1, 5000, 1), (16, 5, 3000, 4), (10, 12, 700, 64), (16, 32, 2, 40),
                                     (3, 2, 1, 257), (5, 4, 64, 33), (2, 3, 9, 100001)])
def test_rows_match_oracle(B, M, S, L):
    import torch
    from paper_1611_03226_amd import dfhip as D
    say(f"rows B={B} M={M} {S}x{L}")
    rng = np.random.default_rng(S + L)
    x, h = complex_gaussian(rng, (S, L), rms=0.6), dpd_coeffs(rng, B, M)
    buf = torch.zeros(S * L + 2, dtype=torch.complex64, device="cuda")
    y = buf[1:1 + S * L].view(S, L)                      # nothing outside may be written
    D.df_dpd_forward(torch.from_numpy(x).cuda(), None, torch.from_numpy(h).cuda(), y, L)
    torch.cuda.synchronize()
    ref = odpd.run_dpd_streams(x, np.full((S, 1), B, np.int32), h, L)
    assert np.linalg.norm(y.cpu().numpy() - ref) <= DPD_TOL * np.linalg.norm(ref)
    assert buf[0].item() == 0 and buf[-1].item() == 0


@pytest.mark.parametrize("B,M", [(10, 16), (16, 4), (5, 8), (10, 12), (3, 31)])
def test_rows_equal_larger_batches(B, M):
    """Rows give the same bits alone (sample by sample) and among so many that
    they run in tiles."""
    import torch
    from paper_1611_03226_amd import dfhip as D
    say(f"rows alone and among others B={B} M={M}")
    S, L = 20000, 300
    g = torch.Generator(device="cuda").manual_seed(B)
    x = torch.view_as_complex(torch.randn(S, L, 2, device="cuda", generator=g) * 0.4)
    x[7, 5], x[9, 0], x[11, 299] = float("inf"), float("nan"), 1e30
    h = torch.from_numpy(dpd_coeffs(np.random.default_rng(M), B, M)).cuda()
    y, few = torch.empty_like(x), torch.empty_like(x[:50])
    D.df_dpd_forward(x, None, h, y, L)
    D.df_dpd_forward(x[:50].contiguous(), None, h, few, L)
    assert np.array_equal(y[:50].cpu().numpy().view(np.float32), few.cpu().numpy().view(np.float32), equal_nan=True)


@pytest.mark.parametrize("B,M,S,nf,r", [(3, 3, 300, 100, 2), (6, 7, 40, 200, 6), (1, 1, 50, 600, 3)])
@pytest.mark.parametrize("hist", ["branch", "shared"])
def test_rows_with_tokens_match_oracle(B, M, S, nf, r, hist):
    import torch
    from paper_1611_03226_amd import dfhip as D
    say(f"rows with tokens B={B} M={M} {S}x{nf}x{r} {hist}")
    rng = np.random.default_rng(S + nf)
    x, h = complex_gaussian(rng, (S, nf * r), rms=0.6), dpd_coeffs(rng, B, M)
    c = rng.integers(-1, B + 2, (S, nf)).astype(np.int32)
    valid = np.where((c >= 0) & (c <= B), c, 0).astype(np.int32)
    y = torch.empty(S, nf * r, dtype=torch.complex64, device="cuda")
    D.df_dpd_forward(torch.from_numpy(x).cuda(), torch.from_numpy(c).cuda(), torch.from_numpy(h).cuda(), y, r,
                     D.DF_HIST_SHARED if hist == "shared" else D.DF_HIST_BRANCH)
    torch.cuda.synchronize()
    pick = [0, S // 2, S - 1]
    ref = odpd.run_dpd_streams(x[pick], valid[pick], h, r, hist)
    assert np.linalg.norm(y[pick].cpu().numpy() - ref) <= DPD_TOL * np.linalg.norm(ref)
