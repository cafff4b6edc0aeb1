"""Amplifier model kernels: loss and stored error, the input adjoint with and
without the loss's scale, at the edges of a thread's four samples, a
workgroup's run and a row, unaligned rows and other orders and taps than the
compiled four by four, against the FP64 oracle; and adaptation_loss against
the same expression in torch operations."""
import numpy as np
import pytest

from helpers import say
from oracle import pa as opa
from workloads import complex_gaussian
from workloads.gen import pa_coeffs

pytestmark = pytest.mark.gpu

# a value is a sum of at most Q (2K + 4) products of FP32 factors, each with a
# relative rounding of 2^-24: below 1e-5 of the terms' size at K = 5, Q = 7
TOL = 1e-5


def _t(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("K,Q", [(4, 4), (1, 1), (4, 3), (5, 7), (2, 4), (4, 32)])
@pytest.mark.parametrize("S,L", [(1, 40), (3, 45), (2, 255), (5, 256), (1, 1027), (2, 1024), (3, 4099)])
def test_loss_and_adjoints(K, Q, S, L):
    import torch
    from paper_1611_03226_amd import dfhip as D
    say(f"pa loss K={K} Q={Q} {S}x{L}")
    rng = np.random.default_rng(K * 1000 + Q * 100 + L)
    a = pa_coeffs(rng, K, Q, sigma=0.1)
    u, x, g = (complex_gaussian(rng, (S, L), rms=0.7) for _ in range(3))
    ref = opa.pa_forward(u, a) - x
    buf = torch.zeros(S * L + 1, dtype=torch.complex64, device="cuda")
    e = buf[1:].view(S, L)                               # 8 bytes off a 16-byte boundary
    loss = torch.zeros((), device="cuda")
    work = torch.empty(D.df_mp_loss_work_bytes(), dtype=torch.uint8, device="cuda")
    D.df_mp_loss(_t(u), _t(a), _t(x), e, loss, work)
    only = torch.zeros((), device="cuda")
    D.df_mp_loss(_t(u), _t(a), _t(x), None, only, work)
    gl = torch.full((), -0.75, device="cuda")
    Gu, Gp = (torch.zeros(S, L, dtype=torch.complex64, device="cuda") for _ in range(2))
    D.df_mp_loss_adjoint(_t(u), _t(a), e, gl, Gu)
    D.df_mp_input_adjoint(_t(u), _t(a), _t(g), Gp)
    torch.cuda.synchronize()
    scale = np.sqrt(np.mean(np.abs(ref) ** 2))
    assert np.abs(e.cpu().numpy() - ref).max() <= TOL * (scale + np.abs(ref).max())
    want = float(np.sum(np.abs(ref) ** 2))
    assert abs(loss.item() - want) <= TOL * want and only.item() == loss.item()
    for got, up in ((Gu, -1.5 * e.cpu().numpy().astype(np.complex128)), (Gp, g)):
        r = opa.pa_input_vjp(u, a, up)
        assert np.linalg.norm(got.cpu().numpy() - r) <= TOL * np.linalg.norm(r)


def test_short_rows_and_empty():
    import torch
    from paper_1611_03226_amd import dfhip as D
    say("pa rows of 3..9 samples, empty batch")
    rng = np.random.default_rng(9)
    a = pa_coeffs(rng, 4, 4, sigma=0.1)
    work = torch.empty(D.df_mp_loss_work_bytes(), dtype=torch.uint8, device="cuda")
    for L in range(3, 10):
        u, x = (complex_gaussian(rng, (70, L)) for _ in range(2))
        e = torch.empty(70, L, dtype=torch.complex64, device="cuda")
        loss = torch.empty((), device="cuda")
        D.df_mp_loss(_t(u), _t(a), _t(x), e, loss, work)
        ref = opa.pa_forward(u, a) - x
        assert np.linalg.norm(e.cpu().numpy() - ref) <= TOL * np.linalg.norm(ref)
        assert abs(loss.item() - np.sum(np.abs(ref) ** 2)) <= TOL * np.sum(np.abs(ref) ** 2)
    z = torch.empty(0, 8, dtype=torch.complex64, device="cuda")
    loss = torch.ones((), device="cuda")
    D.df_mp_loss(z, _t(a), z, z, loss, work)
    assert loss.item() == 0.0
    with pytest.raises(D.DFError):                       # shorter than the model's memory, as the forward refuses it
        D.df_mp_loss(_t(u[:, :2]), _t(a), _t(u[:, :2]), None, loss, work)


@pytest.mark.parametrize("x_grad", [False, True])
def test_adaptation_loss_equals_torch_expression(x_grad):
    import torch
    from paper_1611_03226_amd.autograd import DPDFunction, PAFunction, adaptation_loss
    say(f"adaptation loss vs torch expression, x_grad={x_grad}")
    rng = np.random.default_rng(4)
    x = _t(complex_gaussian(rng, (3, 2051), rms=0.3)).requires_grad_(x_grad)
    a = _t(pa_coeffs(rng))
    h = _t((0.02 * rng.standard_normal((6, 9)) + 0.01j * rng.standard_normal((6, 9))).astype(np.complex64))
    out = []
    for fused in (True, False):
        hh = h.clone().requires_grad_(True)
        x.grad = None
        if fused:
            loss = adaptation_loss(x, hh, a, 2051)
        else:
            e = PAFunction.apply(DPDFunction.apply(x, hh, 2051), a) - x
            loss = (e.real * e.real + e.imag * e.imag).sum()
        (3.0 * loss).backward()
        out.append((loss.detach(), hh.grad, x.grad))
    assert abs(out[0][0] - out[1][0]) <= TOL * out[1][0]
    assert (out[0][1] - out[1][1]).norm() <= TOL * out[1][1].norm()
    assert (out[0][2] is None) == (not x_grad)
    if x_grad:
        assert torch.equal(out[0][2], out[1][2])
    with torch.no_grad():
        assert torch.equal(adaptation_loss(x, h, a, 2051), adaptation_loss(x, h, a, 2051))


@pytest.mark.parametrize("h_grad", [False, True])
def test_adaptation_loss_with_a_variable_amplifier(h_grad):
    """A model whose coefficients require a gradient is fixed all the same: the
    backward runs and leaves none there, as PAFunction's does."""
    from paper_1611_03226_amd.autograd import adaptation_loss
    say(f"adaptation loss, a requires grad, h_grad={h_grad}")
    rng = np.random.default_rng(11)
    x = _t(complex_gaussian(rng, (2, 300), rms=0.3))
    a0 = _t(pa_coeffs(rng))
    h0 = _t((0.02 * rng.standard_normal((4, 8)) + 0j).astype(np.complex64))
    a, h = a0.clone().requires_grad_(True), h0.clone().requires_grad_(h_grad)
    loss = adaptation_loss(x, h, a, 300)
    loss.backward()
    assert a.grad is None
    hr = h0.clone().requires_grad_(True)
    ref = adaptation_loss(x, hr, a0, 300)
    ref.backward()
    assert loss.item() == ref.item()
    if h_grad:
        assert (h.grad - hr.grad).norm() == 0


@pytest.mark.parametrize("K,Q,S,L", [(4, 4, 1, 1 << 21), (4, 4, 512, 4099), (4, 4, 3, 200003), (4, 4, 9000, 61),
                                     (5, 4, 2, 300001), (3, 7, 20001, 31), (8, 16, 7, 80001), (1, 1, 1, 600000)])
def test_large_batches(K, Q, S, L):
    """Batches large enough for the forms with several samples per thread: the
    run form's rows at and off a run's length, the sample-wise forms with rows
    that end anywhere in a thread's samples."""
    import torch
    from paper_1611_03226_amd import dfhip as D
    say(f"pa loss large K={K} Q={Q} {S}x{L}")
    rng = np.random.default_rng(K * 1000 + Q * 100 + S)
    a = pa_coeffs(rng, K, Q, sigma=0.1)
    u, x, g = (complex_gaussian(rng, (S, L), rms=0.7) for _ in range(3))
    ref = opa.pa_forward(u, a) - x
    e, Gp = (torch.zeros(S, L, dtype=torch.complex64, device="cuda") for _ in range(2))
    loss = torch.zeros((), device="cuda")
    work = torch.empty(D.df_mp_loss_work_bytes(), dtype=torch.uint8, device="cuda")
    du, da, dx, dg = _t(u), _t(a), _t(x), _t(g)
    D.df_mp_loss(du, da, dx, e, loss, work)
    D.df_mp_input_adjoint(du, da, dg, Gp)
    torch.cuda.synchronize()
    scale = np.sqrt(np.mean(np.abs(ref) ** 2))
    assert np.abs(e.cpu().numpy() - ref).max() <= TOL * (scale + np.abs(ref).max())
    want = float(np.sum(np.abs(ref) ** 2))
    assert abs(loss.item() - want) <= TOL * want
    r = opa.pa_input_vjp(u, a, g)
    err = np.abs(Gp.cpu().numpy() - r)
    assert np.linalg.norm(err) <= TOL * np.linalg.norm(r)
    D.df_mp_input_adjoint(du, da, dg, du)                # in place of u, as a caller may
    assert torch.equal(du, Gp)


@pytest.mark.parametrize("K,Q,S,L", [(1, 1, 3, 501), (4, 4, 5, 999), (4, 4, 700, 1003), (3, 6, 300, 2500)])
def test_error_of_a_close_model(K, Q, S, L):
    """With one real coefficient the error sample is one fused product onto -x:
    its own rounding is 2^-24 of the sample, however much larger the two parts
    are, and twice that leaves room for nothing at the parts' size."""
    import torch
    from paper_1611_03226_amd import dfhip as D
    say(f"pa loss close K={K} Q={Q} {S}x{L}")
    rng = np.random.default_rng(L)
    a = np.zeros((K, Q), np.complex64)
    a[0, 0] = np.float32(1) / np.float32(3)
    u = complex_gaussian(rng, (S, L), rms=0.7).astype(np.complex64)
    x = (u / 3 * (1 + 1e-3 * rng.standard_normal((S, L)))).astype(np.complex64)
    e, loss = torch.zeros(S, L, dtype=torch.complex64, device="cuda"), torch.zeros((), device="cuda")
    work = torch.empty(D.df_mp_loss_work_bytes(), dtype=torch.uint8, device="cuda")
    D.df_mp_loss(_t(u), _t(a), _t(x), e, loss, work)
    torch.cuda.synchronize()
    ref = (u.astype(np.complex128) * np.float64(a[0, 0].real) - x).view(np.float64)
    assert np.all(np.abs(e.cpu().numpy().view(np.float32) - ref) <= 2.0 ** -23 * np.abs(ref))
