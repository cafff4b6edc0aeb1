"""Performance cases: the work that users of this library have it do, each
through its public entry points.

listed() gives fixed cases over the range of use, draw() further ones of the
same ranges, prepare() what a program holds before a pass (inputs, the graph
with its actors and channels), run() one pass, exact() its result in 64 bits
by plain torch, and work() the bytes and operations a pass cannot do without.

Kinds:
  dpd        one predistortion actor: push control tokens and samples, fire
             the batch, pop the outputs
  instances  many predistortion actors of uneven length, fired as one batch
             (persistent kernel, captured graph)
  stream     host arrays through one predistortion actor, transfers overlapped
  motion     motion actor: push frames, fire, pop the emitted masks and the
             frame numbers
  pipeline   Gauss -> Thres -> Med on 8-bit frames: push, fire, pop
  adapt      one coefficient adaptation step through a power-amplifier model:
             loss and coefficient gradients
  layer      a predistortion layer with control tokens inside a larger
             program: forward and coefficient gradients for a given upstream
             gradient
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1611_03226_amd import autograd as A
from paper_1611_03226_amd import dfhip as D
from paper_1611_03226_amd.graph import Graph


def listed():
    return [
        # the smallest call in use: one short chain of 64 firings, where the
        # launches and the host's part count
        {"name": "dpd_chain", "kind": "dpd", "firings": 64, "r": 256, "branches": 5, "taps": 8, "control": "count",
         "history": "branch", "delay": 4, "lowest": 1, "host_control": False},
        # predistortion of a long recording: 2^24 samples, reconfigured every 4096
        {"name": "dpd_scale", "kind": "dpd", "firings": 4096, "r": 4096, "branches": 10, "taps": 16,
         "control": "count", "history": "branch", "delay": 0, "lowest": 1, "host_control": False},
        # arbitrary filter sets chosen on the host per firing, firing size not
        # a power of two
        {"name": "dpd_mask", "kind": "dpd", "firings": 777, "r": 1000, "branches": 10, "taps": 16, "control": "mask",
         "history": "branch", "delay": 0, "lowest": 1, "host_control": True},
        # the paper's predistortion filters (Sec. 4.2): 10 taps, 2..10 active
        # branches, reconfigured every 65536 samples
        {"name": "dpd_ten_taps", "kind": "dpd", "firings": 32, "r": 65536, "branches": 10, "taps": 10,
         "control": "count", "history": "branch", "delay": 0, "lowest": 2, "host_control": False},
        # a base station's antennas and carriers: independent actors of uneven
        # length in one batch
        {"name": "instances", "kind": "instances", "count": 128, "r": 1024, "median": 16384, "branches": 10,
         "taps": 16},
        # samples that arrive and leave through host memory
        {"name": "stream_host", "kind": "stream", "batches": 4, "firings": 256, "r": 4096, "branches": 10,
         "taps": 16},
        # motion detection on full-HD video with data-dependent emission
        {"name": "motion_1080p", "kind": "motion", "frames": 120, "width": 1920, "height": 1080, "self_delay": True},
        # small video of odd width, the previous frame over its own channel
        {"name": "motion_odd", "kind": "motion", "frames": 24, "width": 333, "height": 251, "self_delay": False},
        # the paper's motion pipeline (Sec. 4.1): 320x240 frames, token rate 4,
        # the chain fired as one
        {"name": "pipeline_320x240", "kind": "pipeline", "firings": 1024, "rate": 4, "width": 320, "height": 240,
         "chain": True},
        # the same actors fired one by one on widescreen video whose width is
        # not a multiple of 4
        {"name": "pipeline_854x480", "kind": "pipeline", "firings": 16, "rate": 4, "width": 854, "height": 480,
         "chain": False},
        # coefficient adaptation over 64 captured streams: forward, amplifier
        # model, loss and backward
        {"name": "adapt", "kind": "adapt", "streams": 64, "length": 65536, "branches": 10, "taps": 16},
        # a smaller adaptation layer under reconfiguration: forward and backward
        {"name": "layer_control", "kind": "layer", "streams": 6, "firings": 40, "r": 500, "branches": 6, "taps": 12,
         "history": "branch"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["dpd", "dpd", "dpd", "instances", "stream", "motion", "motion", "pipeline", "pipeline",
                       "adapt", "layer"])
    taps = rng.choice([4, 8, 16, 16, rng.randint(1, 32)])
    branches = rng.choice([5, 10, rng.randint(1, 16)])
    if kind == "dpd":
        r = _log(rng, max(16, taps), 65536)
        n = _log(rng, 4, max(4, min(8192, (1 << 22) // r)))
        return {"kind": kind, "firings": n, "r": r, "branches": branches, "taps": taps,
                "control": rng.choice(["count", "count", "mask"]), "history": rng.choice(["branch", "branch", "shared"]),
                "delay": rng.choice([0, 0, 1, 4]), "lowest": rng.choice([0, 1]),
                "host_control": rng.choice([False, True])}
    if kind == "instances":
        return {"kind": kind, "count": _log(rng, 8, 128), "r": rng.choice([256, 1000, 1024, 2048]),
                "median": _log(rng, 4096, 32768), "branches": branches, "taps": rng.choice([4, 8, 16])}
    if kind == "stream":
        return {"kind": kind, "batches": rng.randint(2, 6), "firings": _log(rng, 16, 256), "r": _log(rng, 256, 4096),
                "branches": branches, "taps": rng.choice([8, 10, 16])}
    if kind in ("motion", "pipeline"):
        w = rng.choice([16 * rng.randint(8, 120), rng.randint(100, 1920)])
        h = max(16, int(w * rng.uniform(0.5, 0.8)))
        n = _log(rng, 4, max(4, min(1024, (1 << 28) // (w * h))))
        if kind == "motion":
            return {"kind": kind, "frames": n, "width": w, "height": h, "self_delay": rng.choice([True, False])}
        rate = rng.choice([1, 4, 4])
        return {"kind": kind, "firings": max(1, n // rate), "rate": rate, "width": w, "height": h,
                "chain": rng.choice([True, False])}
    if kind == "adapt":
        s = _log(rng, 1, 64)
        return {"kind": kind, "streams": s, "length": _log(rng, 1000, (1 << 22) // s), "branches": min(branches, 10),
                "taps": min(taps, 16)}
    s = _log(rng, 1, 32)
    r = _log(rng, max(64, taps), 8192)
    return {"kind": kind, "streams": s, "firings": _log(rng, 2, max(2, min(256, (1 << 21) // (s * r)))), "r": r,
            "branches": branches, "taps": taps, "history": rng.choice(["branch", "branch", "shared"])}


# ------------------------------------------------------------------ inputs

DEV = "cuda"


def _pow2(n):
    return 1 << max(0, int(n - 1).bit_length())


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _normal(g, *shape, rms=1.0):
    return torch.view_as_complex(torch.randn(*shape, 2, device=DEV, generator=g) * (rms / math.sqrt(2.0)))


def _ofdm(g, n):
    """Band-limited Gaussian signal (80 % of the band) clipped at 10 dB above RMS, unit RMS."""
    m = _pow2(n)
    s = torch.fft.fft(_normal(g, m))
    s[torch.fft.fftfreq(m, device=DEV).abs() > 0.4] = 0
    x = torch.fft.ifft(s)[:n]
    x = x / x.abs().square().mean().sqrt()
    mag = x.abs()
    x = torch.where(mag > 10.0 ** 0.5, x * (10.0 ** 0.5 / mag), x)
    return (x / x.abs().square().mean().sqrt()).contiguous()


def _coeffs(g, branches, taps):
    """Coefficients with a unit linear tap, branch b scaled so that every order contributes comparably."""
    h = 0.1 * torch.view_as_complex(torch.randn(branches, taps, 2, device=DEV, generator=g))
    f = [1.0] + [1.0 / math.sqrt(math.factorial(2 * b + 1)) for b in range(1, branches)]
    h = h * torch.tensor(f, device=DEV)[:, None]
    h[0, 0] = 1.0
    return h.contiguous()


def _control(g, c, n, mask):
    hi = (1 << c["branches"]) if mask else c["branches"] + 1
    return torch.randint(min(c.get("lowest", 1), hi - 1), hi, (n,), device=DEV, generator=g, dtype=torch.int32)


def _dpd_inputs(c, seed):
    g = _gen(seed)
    n = c["firings"] * c.get("batches", 1)
    N = n * c["r"]
    x = _ofdm(g, N) if N >= 1 << 18 else _normal(g, N)
    return x, _control(g, c, n, c.get("control") == "mask"), _coeffs(g, c["branches"], c["taps"])


def _instance_inputs(c, seed):
    g = _gen(seed)
    rng = np.random.default_rng(c["count"])          # a program's instances keep their lengths
    raw = np.exp(rng.normal(math.log(c["median"]), 1.0, size=c["count"]))
    nf = np.clip(raw // c["r"], 1, 262144 // c["r"]).astype(np.int64)
    B = rng.integers(1, c["branches"] + 1, size=c["count"]).astype(np.int32)
    h = torch.stack([_coeffs(g, c["branches"], c["taps"]) for _ in range(c["count"])])
    return _normal(g, int(nf.sum()) * c["r"]), nf, B, h


def _frames(c, seed):
    """Static texture, 0..8 moving textured rectangles (their number changes every 20 frames), noise of sigma 3."""
    g = _gen(seed)
    rng = np.random.default_rng(seed)
    W, H = c["width"], c["height"]
    n = c["frames"] if "frames" in c else c["firings"] * c["rate"]
    bg = torch.randint(0, 256, (H, W), device=DEV, generator=g, dtype=torch.uint8)
    out = bg.expand(n, H, W).contiguous()
    big = max(4, min(H, W) // 4)
    size = rng.integers(max(2, big // 8), big + 1, size=(8, 2))
    pos = rng.random((8, 2)) * (np.array([H, W]) - size)
    vel = rng.uniform(-6, 6, size=(8, 2))
    tex = [torch.randint(0, 256, (int(s[0]), int(s[1])), device=DEV, generator=g, dtype=torch.uint8) for s in size]
    seen = rng.integers(0, 9, size=n // 20 + 1)
    for t in range(n):
        for k in range(int(seen[t // 20])):
            lim = np.array([H, W]) - size[k]
            q = (pos[k] + vel[k] * t) % (2 * lim + 2)
            y, x = np.minimum(np.where(q > lim, 2 * lim + 1 - q, q), lim).clip(0).astype(int)
            out[t, y:y + size[k][0], x:x + size[k][1]] = tex[k]
    per = max(1, (1 << 27) // (W * H))
    for t in range(0, n, per):
        v = out[t:t + per]
        v.copy_((v.float() + 3.0 * torch.randn(v.shape, device=DEV, generator=g)).round_().clamp_(0, 255))
    return out


def _adapt_inputs(c, seed):
    """Streams at RMS 0.25, a predistorter near identity, a fixed amplifier model of orders 1..7 and 4 delays."""
    g = _gen(seed)
    x = _normal(g, c["streams"], c["length"], rms=0.25)
    h = 0.01 * torch.view_as_complex(torch.randn(c["branches"], c["taps"], 2, device=DEV, generator=g))
    h[0, 0] = 1.0
    a = 0.05 * torch.view_as_complex(torch.randn(4, 4, 2, device=DEV, generator=g))
    a[0, 0] = 1.0
    return x, h.contiguous(), a.contiguous()


def _layer_inputs(c, seed):
    g = _gen(seed)
    S, n = c["streams"], c["firings"]
    x = _normal(g, S, n * c["r"], rms=0.7)
    ctrl = _control(g, c, S * n, False).view(S, n)
    return x, ctrl, _coeffs(g, c["branches"], c["taps"]), _normal(g, S, n * c["r"])


# ------------------------------------------------------------------ a program's state and one pass of it

def prepare(case, seed):
    c = case
    k = c["kind"]
    st = {"kind": k, "case": c}
    if k in ("dpd", "stream"):
        x, ctrl, h = _dpd_inputs(c, seed)
        n, r = ctrl.numel(), c["r"]
        held = n * r + c.get("delay", 0) if k == "dpd" else 2 * c["firings"] * r
        fired = n if k == "dpd" else 2 * c["firings"]
        G = Graph(0)
        ch = G.dpd_chain(h.cpu().numpy(), r, c.get("delay", 0), history=c.get("history", "branch"),
                         control=c.get("control", "count"), cap_x=_pow2(held), cap_ctrl=_pow2(fired),
                         cap_y=_pow2(held))
        st.update(G=G, ch=ch, n=n)
        if k == "dpd":
            st.update(x=x, ctrl=ctrl.cpu().numpy() if c["host_control"] else ctrl, y=torch.empty_like(x))
        else:
            def pinned(t):
                return torch.empty(t.shape, dtype=t.dtype, pin_memory=True).copy_(t)
            st["keep"] = [pinned(x), pinned(ctrl), pinned(torch.zeros_like(x))]
            st["x"], st["ctrl"], st["y"] = (t.numpy() for t in st["keep"])
    elif k == "instances":
        x, nf, B, h = _instance_inputs(c, seed)
        r = c["r"]
        hh = h.cpu().numpy()
        G = Graph(0)
        st.update(G=G, nf=[int(v) for v in nf], x=[], ctrl=[], y=[], ch=[], out=torch.empty_like(x))
        at = 0
        for i, m in enumerate(st["nf"]):
            st["ch"].append(G.dpd_chain(hh[i], r, cap_x=_pow2(m * r), cap_ctrl=_pow2(m), cap_y=_pow2(m * r)))
            st["x"].append(x[at:at + m * r])
            st["y"].append(st["out"][at:at + m * r])
            st["ctrl"].append(torch.full((m,), int(B[i]), dtype=torch.int32, device=DEV))
            at += m * r
        st["actors"] = [ch.actor for ch in st["ch"]]
    elif k == "motion":
        f = _frames(c, seed)
        n = c["frames"]
        G = Graph(0)
        mc = G.motion_chain(c["width"], c["height"], self_delay=c["self_delay"], cap_in=_pow2(n + 1),
                            cap_out=_pow2(n))
        st.update(G=G, ch=mc, frames=f, n=n, mask=torch.zeros_like(f),
                  index=torch.zeros(n, dtype=torch.int64, device=DEV))
    elif k == "pipeline":
        f = _frames(c, seed)
        G = Graph(0)
        p = G.paper_motion_pipeline(c["width"], c["height"], 20, c["rate"], cap=_pow2(f.shape[0] + 1))
        st.update(G=G, ch=p, frames=f, out=torch.empty_like(f))
    elif k == "adapt":
        x, h, a = _adapt_inputs(c, seed)
        st.update(x=x, h=h.requires_grad_(True), a=a)
    else:
        x, ctrl, h, g = _layer_inputs(c, seed)
        st.update(x=x, ctrl=ctrl, h=h.requires_grad_(True), g=g)
    return st


def run(state):
    s, k = state, state["kind"]
    if k == "dpd":
        G, ch = s["G"], s["ch"]
        G.push(ch.ctrl, s["ctrl"])
        G.push(ch.x, s["x"])
        G.fire(ch.actor, s["n"])
        G.pop(ch.y, s["y"])
        return s["y"]
    if k == "instances":
        G = s["G"]
        for ch, x, ctrl in zip(s["ch"], s["x"], s["ctrl"]):
            G.push(ch.ctrl, ctrl)
            G.push(ch.x, x)
        G.fire_many(s["actors"], s["nf"], persistent=True, graph=True)
        for ch, y in zip(s["ch"], s["y"]):
            G.pop(ch.y, y)
        return s["out"]
    if k == "stream":
        c = s["case"]
        D.df_stream_dpd(s["G"].g, s["ch"].actor, s["x"], s["ctrl"], s["y"], c["batches"], c["firings"])
        return s["y"]
    if k == "motion":
        G, ch = s["G"], s["ch"]
        G.push(ch.cur, s["frames"])
        if ch.prev >= 0:
            G.push(ch.prev, s["frames"])
        G.fire(ch.actor, s["n"])
        m = G.pop(ch.mask, s["mask"])
        i = G.pop(ch.index, s["index"])
        return {"mask": s["mask"], "index": s["index"], "emitted": [m, i]}
    if k == "pipeline":
        G, p, n = s["G"], s["ch"], s["case"]["firings"]
        G.push(p.inp, s["frames"])
        if s["case"]["chain"]:
            p.fire_chain(G, n)
        else:
            p.fire_all(G, n)
        G.pop(p.out, s["out"])
        return s["out"]
    s["h"].grad = None
    if k == "adapt":
        loss = A.adaptation_loss(s["x"], s["h"], s["a"], s["case"]["length"])
        loss.backward()
        return {"loss": loss.detach(), "grad": s["h"].grad}
    hist = D.DF_HIST_SHARED if s["case"]["history"] == "shared" else D.DF_HIST_BRANCH
    y = A.DPDFunction.apply(s["x"], s["h"], s["case"]["r"], s["ctrl"], hist)
    y.backward(s["g"])
    return {"y": y.detach(), "grad": s["h"].grad}


# ------------------------------------------------------------------ results in 64 bits

def _branch_parts(x, sets, r, b, shared):
    """Rows of x [S, n*r] as branch b's filter sees them: (per row) the samples of its stream, and where its active
    firings' samples lie in that stream and in the row."""
    S, N = x.shape
    t = torch.arange(N, device=x.device)
    for s in range(S):
        on = ((sets[s] >> b) & 1).bool().repeat_interleave(r)
        if not bool(on.any()):
            continue
        at = t[on]
        yield (s, x[s], at, at) if shared else (s, x[s][on], torch.arange(at.numel(), device=x.device), at)


def _dpd64(x, sets, h, r, shared):
    """y [S, N] and, per (branch, row), the branch's stream, in complex128."""
    x, h = x.to(torch.complex128), h.to(torch.complex128)
    y = torch.zeros_like(x)
    for b in range(h.shape[0]):
        for s, u, here, at in _branch_parts(x, sets, r, b, shared):
            psi = u * u.abs().square() ** b
            acc = torch.zeros_like(u)
            for m in range(min(h.shape[1], u.numel())):
                acc[m:] += h[b, m] * psi[:u.numel() - m]
            y[s, at] += acc[here]
    return y


def _coeff_grad64(x, sets, g, B, M, r, shared):
    x, g = x.to(torch.complex128), g.to(torch.complex128)
    out = torch.zeros(B, M, dtype=torch.complex128, device=x.device)
    for b in range(B):
        for s, u, here, at in _branch_parts(x, sets, r, b, shared):
            psi = u * u.abs().square() ** b
            gu = torch.zeros_like(u)
            gu[here] = g[s, at]
            for m in range(min(M, u.numel())):
                out[b, m] += (gu[m:] * psi[:u.numel() - m].conj()).sum()
    return out


def _sets(ctrl, mask):
    ctrl = ctrl.long()
    return ctrl if mask else (1 << ctrl) - 1


def exact(case, seed):
    c = case
    k = c["kind"]
    if k in ("motion", "pipeline"):
        return None                      # whole bytes and frame numbers
    if k in ("dpd", "stream"):
        x, ctrl, h = _dpd_inputs(c, seed)
        d = c.get("delay", 0)
        x = torch.cat([x.new_zeros(d), x])[:x.numel()]
        y = _dpd64(x[None], _sets(ctrl, c.get("control") == "mask")[None], h, c["r"], c.get("history") == "shared")[0]
        return y if k == "dpd" else y.cpu().numpy()
    if k == "instances":
        x, nf, B, h = _instance_inputs(c, seed)
        out, at = [], 0
        for i, m in enumerate(nf):
            m = int(m)
            sets = torch.full((1, m), (1 << int(B[i])) - 1, device=DEV)
            out.append(_dpd64(x[None, at:at + m * c["r"]], sets, h[i], c["r"], False)[0])
            at += m * c["r"]
        return torch.cat(out)
    if k == "adapt":
        x, h, a = _adapt_inputs(c, seed)
        S, N = x.shape
        a = a.to(torch.complex128)
        sets = torch.full((S, 1), (1 << c["branches"]) - 1, device=DEV)
        u = _dpd64(x, sets, h, N, True).requires_grad_(True)
        v = 0
        for i in range(4):
            psi = u * (u.real.square() + u.imag.square()) ** i
            for q in range(min(4, N)):
                v = v + torch.nn.functional.pad(torch.view_as_real(a[i, q] * psi[:, :N - q]), (0, 0, q, 0))
        e = v - torch.view_as_real(x.to(torch.complex128))
        loss = e.square().sum()
        gu, = torch.autograd.grad(loss, u)
        return {"loss": loss.detach(), "grad": _coeff_grad64(x, sets, gu, c["branches"], c["taps"], N, True)}
    x, ctrl, h, g = _layer_inputs(c, seed)
    sets, shared = _sets(ctrl, False), c["history"] == "shared"
    return {"y": _dpd64(x, sets, h, c["r"], shared),
            "grad": _coeff_grad64(x, sets, g, c["branches"], c["taps"], c["r"], shared)}


# ------------------------------------------------------------------ least work of a pass

def work(case):
    """Bytes: inputs read once, outputs written once.  Operations of a sample with B active branches and M taps:
    |x|^2 (3), per tap the real-argument polynomial of B complex coefficients (4 (B - 1)) and a complex
    multiply-add (8)."""
    c = case
    k = c["kind"]

    def per_sample(B, M):
        return 3.0 + M * (4.0 * B + 4.0)

    if k in ("dpd", "stream", "layer"):
        n = c["firings"] * c.get("batches", c.get("streams", 1))
        N = n * c["r"]
        mean = c["branches"] / 2 if c.get("control") == "mask" else (c.get("lowest", 1) + c["branches"]) / 2
        f = N * per_sample(mean, c["taps"])
        if k == "layer":
            return {"bytes": 24.0 * N + 4 * n, "flops": f + N * c["taps"] * (8.0 + 4.0 * mean)}
        return {"bytes": 16.0 * N + 4 * n, "flops": f}
    if k == "instances":
        N = c["count"] * c["median"] * math.exp(0.5)
        return {"bytes": 16.0 * N, "flops": N * per_sample((1 + c["branches"]) / 2, c["taps"])}
    if k == "motion":
        px = c["frames"] * c["width"] * c["height"]
        return {"bytes": 1.9 * px, "flops": 12.0 * px}
    if k == "pipeline":
        px = c["firings"] * c["rate"] * c["width"] * c["height"]
        return {"bytes": 2.0 * px, "flops": 40.0 * px}
    N = c["streams"] * c["length"]
    return {"bytes": 8.0 * N,
            "flops": N * (2 * per_sample(c["branches"], c["taps"]) + per_sample(4, 4) + 5 + 4 * 48.0)}
