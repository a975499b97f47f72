"""The work that programs have this framework do, as cases to be timed.

A case is one pass over a stack of camera frames through the public entry
points (Plan, structure_function, Batch): what a program does once per stack
with a plan that it keeps. Sizes follow the workloads of this repository
(gen/configs.py, bench.py, tests) and the range that the reference paper
processed, 32 to 2048 frames of 32x32 up to 4k x 4k pixels.

Fields of a case:
  kind     "analyse"   reset, push, D(q, tau)
           "spectra"   the same, with the 2D power spectra of every delay
           "gradient"  the same, with the gradient of a loss of D (Plan.backward)
           "train"     structure_function() and autograd's backward, which plan on each call
           "ingest"    frames in pinned host memory, uploaded by the push
           "batch"     several stacks together (Batch); sequences as "n x frames" pairs
  n, frames, dtype            frame side, number of frames, pixel type
  lags, lag_max, lag_count    "all": 1..lag_max; "log": lag_count log-spaced up to lag_max;
                              "pow2": 1, 2, 4, ... up to lag_max
  bins                        rings of |q|
  spec, accum                 storage type of the spectra, kind of the sums
  window                      frames multiplied by a Hann window
  capacity, chunk             ring slots (0: all frames) and frames per push (0: all at once)
"""
import math

import torch

import paper_1209_3362_amd as nfs

_BASE = dict(kind="analyse", n=0, frames=0, dtype="u16", lags="log", lag_max=1, lag_count=0,
             bins=1, spec="f32", accum="plain", window=False, capacity=0, chunk=0)


def _case(**kw):
    c = dict(_BASE)
    c.update(kw)
    if "bins" not in kw:
        c["bins"] = c["n"] // 2
    return c


def listed():
    return [
        # The smallest stacks of the paper's timing grid (32 frames of 32x32, every delay):
        # launches and latency are all of it.
        _case(name="tiny_32x32", n=32, frames=32, lags="all", lag_max=31),
        # A short preview stack: 64 float frames of 128x128, five delays (workload c1).
        _case(name="preview_64x128", n=128, frames=64, dtype="f32", lags="pow2", lag_max=16),
        # Live view of a running measurement: a long stream of small frames arriving in odd
        # chunks, in a ring shorter than the stream.
        _case(name="live_1201x256", n=256, frames=1201, lags="log", lag_max=300, lag_count=32,
              capacity=420, chunk=37),
        # The standard analysis (workload c2): 1000 camera frames, 50 log-spaced delays.
        _case(name="standard_1000x1024", n=1024, frames=1000, lags="log", lag_max=500,
              lag_count=50),
        # The paper's own headline run: 2048 images of 512x512, all 2047 delays.
        _case(name="paper_2048x512_all", n=512, frames=2048, lags="all", lag_max=2047),
        # Precision form (workload c3, first part of its stack): dense delays, 16-bit spectra,
        # compensated sums.
        _case(name="dense_900x1024_bf16", n=1024, frames=900, lags="all", lag_max=400,
              spec="bf16", accum="kahan"),
        # The other 16-bit storage type, an ordinary frame size, an odd number of frames, few rings.
        _case(name="ordinary_701x512_f16", n=512, frames=701, dtype="f32", lags="log",
              lag_max=350, lag_count=32, bins=100, spec="f16", window=True),
        # Large sensor, short stack.
        _case(name="sensor_96x2048", n=2048, frames=96, lags="log", lag_max=48, lag_count=16),
        # Differentiation form (workload c5): gradient with respect to frames and window.
        _case(name="gradient_256x512", kind="gradient", n=512, frames=256, dtype="f32",
              lags="pow2", lag_max=64, window=True),
        # A training step on small patches, through autograd.
        _case(name="train_64x128", kind="train", n=128, frames=64, dtype="f32", lags="pow2",
              lag_max=16, window=True),
        # Frames that come from the acquisition's host memory.
        _case(name="ingest_400x512", kind="ingest", n=512, frames=400, lags="log", lag_max=200,
              lag_count=32),
        # Batching form (workload c4, a smaller draw of it): stacks of uneven size together.
        _case(name="batch_6_stacks", kind="batch", n=1024, frames=233, lags="log", lag_max=0,
              lag_count=32, stacks="1024x233,512x480,256x1000,512x211,256x350,256x640"),
    ]


def _stacks(case):
    """(n, frames, lags, bins) of every stack of a case."""
    if case["kind"] != "batch":
        return [(case["n"], case["frames"], _lags(case), case["bins"])]
    out = []
    for part in case["stacks"].split(","):
        n, N = (int(v) for v in part.split("x"))
        out.append((n, N, _log_lags(N // 2, min(case["lag_count"], N // 2)), n // 2))
    return out


def _log_lags(tau_max, count):
    out = []
    for j in range(count):
        t = tau_max if count == 1 else int(math.floor(tau_max ** (j / (count - 1)) + 0.5))
        out.append(max(t, out[-1] + 1) if out else t)
    return [t for t in out if t <= tau_max]


def _lags(case):
    top = case["lag_max"]
    if case["lags"] == "all":
        return list(range(1, top + 1))
    if case["lags"] == "pow2":
        return [1 << j for j in range(top.bit_length()) if 1 << j <= top]
    return _log_lags(top, case["lag_count"])


def _modes(n):
    return math.pi * n * n / 8  # modes of the half plane with |k| < n/2


def _terms(case):
    """(frame, delay) pairs times modes, and pixels, over the stacks of a case."""
    terms = pixels = 0
    for n, N, lags, _ in _stacks(case):
        terms += sum(max(0, N - t) for t in lags) * _modes(n)
        pixels += N * n * n
    return terms, pixels


def draw(rng):
    top_terms = max(_terms(c)[0] for c in listed())
    top_pixels = max(_terms(c)[1] for c in listed())

    def log_int(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    while True:
        kind = rng.choice(["analyse"] * 6 + ["spectra", "gradient", "gradient", "train",
                                             "ingest", "batch"])
        n = 1 << rng.randint(5, 11)
        N = log_int(16, 2048)
        if kind == "batch":
            stacks = ["%dx%d" % (1 << rng.randint(7, 10), log_int(100, 1000))
                      for _ in range(rng.randint(2, 6))]
            c = _case(kind=kind, n=1024, frames=int(stacks[0].split("x")[1]), lags="log",
                      lag_max=0, lag_count=rng.randint(8, 40), stacks=",".join(stacks))
        else:
            lags = rng.choice(["log", "log", "all", "pow2"])
            top = max(1, min(N - 1, log_int(4, 2048)))
            if kind in ("gradient", "train"):
                n, N = min(n, 512), min(N, 300)
                top, lags = min(top, 64, N - 1), rng.choice(["log", "pow2"])
            c = _case(kind=kind, n=n, frames=N, dtype=rng.choice(["u16", "u16", "f32"]),
                      lags=lags, lag_max=top, lag_count=min(top, rng.randint(4, 64)),
                      bins=rng.choice([n // 2, n // 2, rng.randint(1, n // 2)]),
                      window=rng.random() < 0.3)
            if kind in ("gradient", "train"):
                c["dtype"] = "f32"
            elif kind != "spectra":
                c["spec"] = rng.choice(["f32", "f32", "bf16", "f16"])
                c["accum"] = rng.choice(["plain", "plain", "kahan"])
            if kind == "analyse" and rng.random() < 0.3:
                # A stream in chunks; the ring holds the delays and some frames more.
                c["capacity"] = min(N, top + rng.randint(20, 400))
                c["chunk"] = rng.randint(max(1, N // 40), N)
            if kind == "spectra" and len(_lags(c)) * n * n > 1 << 28:
                continue
        terms, pixels = _terms(c)
        if terms <= top_terms and pixels <= (top_pixels if kind not in ("gradient", "train")
                                             else top_pixels // 4):
            return c


# ---------------------------------------------------------------------------
# Inputs: a static Gaussian beam modulated by a small field whose Fourier modes
# are independent Ornstein-Uhlenbeck processes, with camera noise (the model of
# gen/frames.py, drawn in blocks): 12-bit Poisson counts, or float counts with
# Gaussian noise.


def _frames(n, N, dtype, seed):
    dev = "cuda"
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed) * 1000003 + n * 4099 + N)
    ky = torch.fft.fftfreq(n, 1.0 / n, device=dev)[:, None]
    kx = torch.arange(n // 2 + 1, device=dev)[None, :]
    q = 2 * math.pi * torch.sqrt(ky * ky + kx * kx) / n
    amp = torch.clamp(q, min=2 * math.pi / 64) ** -2
    amp[0, 0] = 0.0
    full = torch.full((n // 2 + 1,), 2.0, device=dev)
    full[0] = full[-1] = 1.0
    amp = amp / torch.sqrt((amp * amp * full).sum())
    u16 = dtype == "u16"
    gamma = (0.002 + 0.5 * q * q) if u16 else (0.05 + 2.0 * q * q)
    peak, eps = (3000.0, 0.005) if u16 else (1000.0, 0.01)
    rho = torch.exp(-gamma)
    drive = torch.sqrt(1 - rho * rho) * amp
    y = torch.arange(n, device=dev) - (n - 1) / 2.0
    beam = peak * torch.exp(-(y[:, None] ** 2 + y[None, :] ** 2) / (2 * (40.0 * n / 128) ** 2))
    out = torch.empty((N, n, n), dtype=torch.uint16 if u16 else torch.float32, device=dev)
    block = max(1, min(64, (1 << 24) // (n * n)))
    z = None
    for t0 in range(0, N, block):
        b = min(block, N - t0)
        xi = torch.view_as_complex(torch.randn((b, n, n // 2 + 1, 2), generator=g, device=dev))
        zs = torch.empty_like(xi)
        for j in range(b):
            z = amp * xi[j] if z is None else rho * z + drive * xi[j]
            zs[j] = z
        s = torch.fft.irfft2(zs, s=(n, n), norm="forward")
        lam = beam * (1 + eps * s)
        if u16:
            lam = torch.poisson(lam.clamp_(min=0), generator=g).clamp_(max=4095)
            out[t0:t0 + b] = lam.to(torch.int32).to(torch.uint16)
        else:
            out[t0:t0 + b] = lam + 2.0 * torch.randn(lam.shape, generator=g, device=dev)
    return out


def _window(case):
    if not case["window"]:
        return None
    w = torch.hann_window(case["n"], periodic=False, device="cuda") + 0.01
    return w[:, None] * w[None, :]


def _upstream(case, seed):
    """Gradient of the loss with respect to D."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) + 77)
    return torch.randn((len(_lags(case)), case["bins"]), generator=g, device="cuda",
                       dtype=torch.float64)


def prepare(case, seed):
    s = dict(case=case)
    kind = case["kind"]
    if kind == "batch":
        stacks = _stacks(case)
        s["frames"] = [_frames(n, N, case["dtype"], seed) for n, N, _, _ in stacks]
        s["batch"] = nfs.Batch([dict(n=n, lags=lags, n_bins=nb, in_dtype=case["dtype"], capacity=N)
                                for n, N, lags, nb in stacks], streams=4)
        return s
    frames = _frames(case["n"], case["frames"], case["dtype"], seed)
    w = _window(case)
    if kind in ("gradient", "train"):
        s["upstream"] = _upstream(case, seed)
    if kind == "train":
        s["frames"], s["window"] = frames, w if w is not None else torch.ones_like(frames[0])
        return s
    if kind == "ingest":
        host = torch.empty(frames.shape, dtype=frames.dtype, pin_memory=True)
        host.copy_(frames)
        frames = host
    s["frames"] = frames
    s["plan"] = nfs.Plan(case["n"], _lags(case), case["bins"], in_dtype=case["dtype"],
                         capacity=case["capacity"] or max(case["frames"], case["lag_max"] + 1),
                         window=w, spec=case["spec"], accum=case["accum"],
                         host_staging=kind == "ingest", backward=kind == "gradient",
                         full_spectra=kind == "spectra")
    return s


def _kept(out):
    """D, modes per ring, pairs per delay, status. The per-mode spectra and sums behind D are
    float32, so a program that keeps D for its fits and files keeps it as float32."""
    D, counts, pairs, status = out
    return D.to(torch.float32), counts, pairs, status


def run(state):
    case = state["case"]
    kind = case["kind"]
    frames = state["frames"]
    if kind == "batch":
        return [_kept(o) for o in state["batch"].run(frames, sync=False)]
    if kind == "train":
        f = frames.detach().requires_grad_(True)
        w = state["window"].detach().requires_grad_(True)
        D = nfs.structure_function(f, _lags(case), case["bins"], window=w)
        (D * state["upstream"]).sum().backward()
        return D.detach().to(torch.float32), f.grad, w.grad
    plan = state["plan"]
    plan.reset()
    chunk = case["chunk"] or case["frames"]
    for t in range(0, case["frames"], chunk):
        plan.push(frames[t:t + chunk])
    # An ingesting program waits for its uploads before it reuses their buffers.
    out = _kept(plan.structure_function(sync=kind == "ingest"))
    if kind == "spectra":
        out += (plan.power_spectra(sync=False),)
    if kind == "gradient":
        out += plan.backward(state["upstream"], frames, sync=False)
    return out


def work(case):
    """Frames read once, D and the other outputs written once; the 2D transforms of real
    frames and two subtractions and two multiply-adds per pair of coefficients."""
    b = fl = 0.0
    px = 2 if case["dtype"] == "u16" else 4
    for n, N, lags, bins in _stacks(case):
        pixels = float(N) * n * n
        pairs = sum(max(0, N - t) for t in lags)
        b += pixels * px + len(lags) * bins * 8.0
        fl += 2.5 * pixels * 2 * math.log2(n) + 6.0 * pairs * _modes(n)
        if case["kind"] == "spectra":
            b += len(lags) * n * (n // 2 + 1) * 4.0
        if case["kind"] in ("gradient", "train"):
            b += pixels * 4 + n * n * 4.0
            fl += 2.5 * pixels * 2 * math.log2(n) + 12.0 * pairs * _modes(n)
    return {"bytes": b, "flops": fl}


# ---------------------------------------------------------------------------
# The definition in 64 bits with plain torch.


def _spectra64(frames, w):
    """Half-plane transforms of the mean-normalised frames minus the first frame's (every
    difference of two of them is that of the transforms), [frames][n][n/2 + 1]."""
    N, n = frames.shape[0], frames.shape[-1]
    out = torch.empty((N, n, n // 2 + 1), dtype=torch.complex128, device=frames.device)
    ref = None
    block = max(1, (1 << 25) // (n * n))
    for t in range(0, N, block):
        u = frames[t:t + block]
        u = (u.to(torch.int32) if u.dtype == torch.uint16 else u).to(torch.float64)
        if w is not None:
            u = u * w.to(torch.float64)
        u = u / u.mean(dim=(1, 2), keepdim=True)
        ref = u[:1].clone() if ref is None else ref
        out[t:t + block] = torch.fft.rfft2(u - ref)
    out[:, 0, 0] = 0
    return out


def _power64(spec, lags):
    """Mean over the pairs of every delay of |difference|^2, [lags][n][n/2 + 1]. Many delays at
    once come from the autocorrelation in time, few from the differences themselves."""
    N, n, h = spec.shape
    P = torch.full((len(lags), n, h), float("nan"), dtype=torch.float64, device=spec.device)
    rows = max(1, min(n, (1 << 27) // (N * h)))
    for r in range(0, n, rows):
        a = spec[:, r:r + rows]
        if len(lags) > 64:
            size = 1 << (N + max(lags)).bit_length()
            f = torch.fft.fft(a, n=size, dim=0)
            corr = torch.fft.ifft(f.real ** 2 + f.imag ** 2, dim=0).real
            del f
            e = torch.zeros((N + 1,) + a.shape[1:], dtype=torch.float64, device=a.device)
            torch.cumsum(a.real ** 2 + a.imag ** 2, dim=0, out=e[1:])
        for i, t in enumerate(lags):
            if N - t <= 0:
                continue
            if len(lags) > 64:
                S = (e[N] - e[t]) + e[N - t] - 2 * corr[t]
            else:
                d = a[t:] - a[:N - t]
                S = (d.real ** 2 + d.imag ** 2).sum(dim=0)
            P[i, r:r + rows] = S / (N - t)
    return P


def _rings(n, bins):
    """Ring of every half-plane mode (-1: none) and its weight in the full plane."""
    k = torch.arange(n, device="cuda", dtype=torch.int64)
    ky = torch.where(k < n // 2, k, k - n)[:, None]
    kx = torch.arange(n // 2 + 1, device="cuda", dtype=torch.int64)[None, :]
    v = (ky * ky + kx * kx) * bins * bins
    s = torch.sqrt(v.to(torch.float64)).to(torch.int64)
    s = torch.where(s * s > v, s - 1, s)
    s = torch.where((s + 1) * (s + 1) <= v, s + 1, s)
    b = s // (n // 2)
    ring = torch.where(b < bins, b, torch.full_like(b, -1))
    weight = torch.where((kx > 0) & (kx < n // 2), 2.0, 1.0).to(torch.float64).expand(n, -1)
    return ring, weight


def _average64(P, n, bins):
    ring, weight = _rings(n, bins)
    inside = ring >= 0
    at, wt = ring[inside], weight[inside]
    C = torch.zeros(bins, dtype=torch.float64, device=P.device).index_add_(0, at, wt)
    D = torch.stack([torch.zeros(bins, dtype=torch.float64, device=P.device)
                     .index_add_(0, at, wt * p[inside]) / C for p in P])
    return D, C


def _results64(frames, lags, bins, w):
    N, n = frames.shape[0], frames.shape[-1]
    P = _power64(_spectra64(frames, w), lags)
    D, C = _average64(P, n, bins)
    pairs = torch.tensor([max(0, N - t) for t in lags], dtype=torch.int64)
    return P, (D, C.round().to(torch.int64), pairs, torch.zeros(1, dtype=torch.int32))


def _gradient64(frames, lags, bins, w, upstream):
    """dL/dframes and dL/dw for L = sum(upstream * D), by autograd in 64 bits."""
    N, n = frames.shape[0], frames.shape[-1]
    ring, weight = _rings(n, bins)
    inside = ring >= 0
    C = torch.zeros(bins, dtype=torch.float64, device="cuda").index_add_(0, ring[inside],
                                                                        weight[inside])
    f = frames.to(torch.float64).requires_grad_(True)
    ww = (torch.ones((n, n), dtype=torch.float64, device="cuda") if w is None
          else w.to(torch.float64)).requires_grad_(True)
    u = f * ww
    u = u / u.mean(dim=(1, 2), keepdim=True)
    a = torch.fft.rfft2(u - u[:1].detach())
    mask = inside.to(torch.float64)
    mask[0, 0] = 0.0
    loss = 0.0
    for i, t in enumerate(lags):
        if N - t <= 0:
            continue
        g = torch.where(inside, upstream[i][ring.clamp(min=0)] * weight / C[ring.clamp(min=0)],
                        torch.zeros_like(weight)) * mask / (N - t)
        d = a[t:] - a[:N - t]
        loss = loss + ((d.real ** 2 + d.imag ** 2) * g).sum()
    return torch.autograd.grad(loss, (f, ww))


def exact(case, seed):
    kind = case["kind"]
    w = _window(case)
    if kind == "batch":
        return [_results64(_frames(n, N, case["dtype"], seed), lags, nb, w)[1]
                for n, N, lags, nb in _stacks(case)]
    frames = _frames(case["n"], case["frames"], case["dtype"], seed)
    if case["n"] ** 2 * len(_lags(case)) > 1 << 31 and kind == "spectra":
        return None
    P, out = _results64(frames, _lags(case), case["bins"], w)
    if kind == "spectra":
        out += (P,)
    if kind in ("gradient", "train"):
        grads = _gradient64(frames, _lags(case), case["bins"], w, _upstream(case, seed))
        out = (out[0],) + grads if kind == "train" else out + grads
    return out
