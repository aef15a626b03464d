"""The calls whose speed this repository answers for.

Each case is one pass through the public entry points (Tracker.track,
Tracker.track_update, track of the autograd module, iterate_reference) as a
program that tracks particles makes it.  listed() names the cases, draw()
gives more of the same ranges, prepare() makes what such a program holds
before the call (frames, references, a tracker), run() is the call, work()
what it cannot do without, exact() its results in 64 bits from plain torch.

Results handed back are the fields of a result record that are determined by
the inputs: d, peak, the Hessian, the integer peak and the status bits.  The
grid estimate d_grid is the seed of the refinement: near a smooth maximum
neighbouring grid values differ by less than their rounding, and either is
then right, so it is no quantity that two builds have in common.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2310_08770_amd import Tracker
from paper_2310_08770_amd.autograd import track as track_with_grad
from paper_2310_08770_amd.reference import iterate_reference

EPS = 200.0  # CC-SN offset for photon counts of gain 1 (the default)

#: square sizes the tracker takes
SIZES = (16, 18, 24, 32, 36, 48, 54, 64, 72, 96, 108, 128, 144, 162, 192, 216, 256, 288, 324, 384,
         432, 486, 512)
#: rectangles of the paper's Table I, both orientations
RECTS = ((128, 256), (256, 128), (256, 512), (512, 256), (128, 1024), (1024, 128))


def _case(name, kind, ny, nx, n, u, **kw):
    c = dict(kind=kind, ny=ny, nx=nx, n=n, u=u, mode="ccu", precision="fp32", dtype="u16", streams=1,
             pad=0, spot="gauss", sigma=3.0, peak=2000.0, bg=20.0, spread=2.0, passes=1)
    if name:
        c["name"] = name
    c.update(kw)
    return c


def listed():
    return [
        # one camera frame per call at the default precision: the per-frame
        # latency of a live display or feedback loop
        _case("plain_256", "track", 256, 256, 1, 100, spot="airy", peak=4000.0, bg=50.0),
        # the real-time run of the paper: one frame tracked and folded into
        # the reference, frame after frame
        _case("realtime_256x128", "update", 256, 128, 16, 256, mode="ccsn", spot="airy", peak=4000.0, bg=50.0),
        # a short clip of a small region
        _case("clip_64", "track", 64, 64, 100, 20, peak=1000.0, bg=10.0),
        # a long recording in one call, split precision, two streams: the
        # throughput workload of bench.py
        _case("stream_256_split", "track", 256, 256, 10000, 100, precision="bf16x2", streams=2, spot="airy",
              peak=4000.0, bg=50.0, spread=8.0),
        # a recording at the default precision
        _case("stream_256", "track", 256, 256, 2048, 100, spot="airy", peak=4000.0, bg=50.0, spread=8.0),
        # many particles in one call: regions of seven sizes, each with its
        # own reference
        _case("rois_mixed", "rois", 32, 256, 2048, 100, spread=4.0),
        # the precision workload: large frames, fine grid
        _case("large_512_split", "track", 512, 512, 512, 200, precision="bf16x2", sigma=4.0, peak=500.0, spread=3.0),
        # Table I: a wide frame, CC-SN, the paper's u
        _case("table1_128x256", "track", 128, 256, 512, 256, mode="ccsn", precision="bf16x2", spot="airy",
              peak=4000.0, bg=50.0),
        # regions of an odd size cut out of camera frames (odd pitch), CC-SN
        _case("crop_162", "track", 162, 162, 300, 64, mode="ccsn", pad=43, sigma=2.5),
        # differentiation: forward and backward on photon counts
        _case("train_128", "train", 128, 128, 1024, 100, dtype="f32", bg=0.0),
        # the offline reference: two passes of tracking and averaging
        _case("refine_192", "refine", 192, 192, 256, 100, dtype="f32", passes=2),
        # the accuracy mode
        _case("accuracy_128", "track", 128, 128, 64, 100, precision="fp64", dtype="f64"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 50.0)


def draw(rng):
    """One more case: the kinds of call above over the sizes, grid factors,
    pixel types, modes and precisions the tracker takes."""
    top = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["track", "track", "track", "update", "rois", "train", "refine"])
        precision = rng.choice(["fp32", "fp32", "bf16x2", "bf16x2", "fp16x2", "fp64"])
        mode = rng.choice(["ccu", "ccsn"])
        dtype = rng.choice(["u16", "u16", "f32"])
        pad, streams, passes = 0, 1, 1
        sigma = round(rng.uniform(1.8, 4.5), 3)
        u = _log_int(rng, 16, 384)
        if kind == "rois":
            precision = rng.choice(["fp32", "bf16x2"])
            ny, nx = rng.choice([16, 24, 32, 48]), rng.choice([96, 128, 192, 256])
            n, u = _log_int(rng, 100, 2048), _log_int(rng, 20, 128)
        elif kind in ("train", "refine") or precision == "fp64":
            ny = nx = rng.choice([s for s in SIZES if 32 <= s <= 256])
            if kind != "track" and precision in ("fp64", "fp16x2"):
                precision = "fp32"
            n = _log_int(rng, 4, 600) if precision != "fp64" else _log_int(rng, 1, 64)
            if kind == "train":  # photon counts; row blocks of 8 throughout
                dtype = "f32"
                ny = nx = rng.choice([s for s in SIZES if 32 <= s <= 256 and s % 8 == 0])
            if kind == "refine":
                passes = rng.choice([1, 2, 3])
            if kind == "update":
                precision, n = "fp32", 16
        else:
            ny, nx = rng.choice(RECTS) if rng.random() < 0.25 else (lambda s: (s, s))(rng.choice(SIZES))
            if precision == "fp16x2":
                ny = nx = 256
            n = 16 if kind == "update" else _log_int(rng, 1, 3000)
            if kind == "track" and precision != "fp16x2":
                pad = rng.choice([0, 0, 0, 16, 37])
                streams = rng.choice([1, 2])
        if min(ny, nx) < 32:
            sigma = min(sigma, 2.2)
        c = _case(None, kind, ny, nx, n, u, precision=precision, mode=mode, dtype=dtype, pad=pad,
                  streams=streams, sigma=sigma, peak=float(_log_int(rng, 500, 8000)),
                  bg=float(rng.choice([5, 20, 50])), spread=2.0, passes=passes)
        # frames of one call in memory, and the cost of the largest listed case
        if c["n"] * c["ny"] * c["nx"] <= 2 ** 30 and _cost(c) <= top:
            return c


# --------------------------------------------------------------------- inputs
def _profile(n, center, sigma, dev):
    r = torch.arange(n, dtype=torch.float64, device=dev)
    s = math.sqrt(2.0) * sigma
    g = torch.special.erf((r + 0.5 - center) / s) - torch.special.erf((r - 0.5 - center) / s)
    return g / (2.0 * math.erf(0.5 / s))


def _spot(case, ny, nx, dev, sigma=None, peak=None):
    """The noiseless spot without its Nyquist row and column, float64."""
    sigma = case["sigma"] if sigma is None else sigma
    peak = case["peak"] if peak is None else peak
    if case["spot"] == "airy":  # [2 J1(v)/v]^2, first zero at 8 px
        y = torch.arange(ny, dtype=torch.float64, device=dev) - ny / 2
        x = torch.arange(nx, dtype=torch.float64, device=dev) - nx / 2
        v = torch.hypot(y[:, None], x[None, :]) * (3.8317059702075125 / 8.0)
        img = torch.where(v > 0, 2.0 * torch.special.bessel_j1(v) / torch.where(v > 0, v, 1.0), 1.0) ** 2
    else:
        img = _profile(ny, ny / 2, sigma, dev)[:, None] * _profile(nx, nx / 2, sigma, dev)[None, :]
    f = torch.fft.fft2(img * peak)
    f[ny // 2, :] = 0
    f[:, nx // 2] = 0
    return torch.fft.ifft2(f).real


def _shifted(spot, d, bg, gen):
    """Photon counts of the spot displaced by each row of d (band-limited
    shift) on a background, float32 [len(d), ny, nx], clipped to 16 bits."""
    ny, nx = spot.shape[-2:]
    dev = spot.device
    f = torch.fft.rfft2(spot).to(torch.complex64)
    ky = torch.fft.fftfreq(ny, device=dev, dtype=torch.float64)
    kx = torch.fft.rfftfreq(nx, device=dev, dtype=torch.float64)
    ry = torch.exp(-2j * math.pi * ky[None, :] * d[:, 0:1]).to(torch.complex64)
    rx = torch.exp(-2j * math.pi * kx[None, :] * d[:, 1:2]).to(torch.complex64)
    mu = torch.fft.irfft2(f * ry[:, :, None] * rx[:, None, :], s=(ny, nx))
    mu = mu + (bg if not torch.is_tensor(bg) else bg[:, None, None].to(torch.float32))
    return torch.poisson(mu.clamp_(min=0.0), generator=gen).clamp_(max=65535.0)


_DTYPES = {"u16": torch.uint16, "f32": torch.float32, "f64": torch.float64}


def _gen(seed, dev):
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed) * 7919 + 13)
    return g


def _inputs(case, seed):
    """Frames and reference(s) of a case from the seed: (frames, refs, ids).
    A [n, ny, nx] tensor (possibly a view with a row pitch) and one reference,
    or for mixed regions two lists and an id list."""
    dev = torch.device("cuda", torch.cuda.current_device())
    gen = _gen(seed, dev)
    dt = _DTYPES[case["dtype"]]
    if case["kind"] == "rois":
        frames, refs = [], []
        sizes = [s for s in (16, 24, 32, 48, 64, 96, 128, 192, 256) if case["ny"] <= s <= case["nx"]]
        pick = np.random.RandomState(int(seed) % (1 << 31)).choice(len(sizes), size=case["n"])
        for k, s in enumerate(sizes):
            m = int((pick == k).sum())
            if not m:
                continue
            r = torch.rand((m, 5), dtype=torch.float64, device=dev, generator=gen)
            sig = 1.5 + (4.5 if s >= 32 else 0.7) * r[:, 0]
            pk = torch.exp(math.log(200.0) + math.log(100.0) * r[:, 1])
            bg = 100.0 * r[:, 2]
            d = case["spread"] * (2.0 * r[:, 3:5] - 1.0)
            one = _profiles(s, sig, dev)
            spots = pk[:, None, None] * one[:, :, None] * one[:, None, :]
            f = torch.fft.fft2(spots)
            f[:, s // 2, :] = 0
            f[:, :, s // 2] = 0
            spots = torch.fft.ifft2(f).real
            fr = _shifted(spots, d, bg, gen).to(dt)
            rf = (spots + bg[:, None, None]).to(torch.float32)
            frames += list(fr.unbind(0))
            refs += list(rf.unbind(0))
        order = np.random.RandomState(int(seed) % (1 << 31) + 1).permutation(len(frames))
        return [frames[i] for i in order], [refs[i] for i in order], list(range(len(frames)))
    ny, nx, n, pad = case["ny"], case["nx"], case["n"], case["pad"]
    spot = _spot(case, ny, nx, dev)
    d = case["spread"] * (2.0 * torch.rand((n, 2), dtype=torch.float64, device=dev, generator=gen) - 1.0)
    if case["kind"] == "refine":
        d[0] = 0.0
    buf = torch.empty((n, ny, nx + pad), dtype=dt, device=dev)
    step = max(1, (1 << 26) // (ny * nx))
    for i in range(0, n, step):
        buf[i:i + step, :, :nx] = _shifted(spot, d[i:i + step], case["bg"], gen).to(dt)
    ref = (spot + case["bg"]).to(torch.float32)
    return buf[:, :, :nx], ref, [0] * n


def _profiles(n, sig, dev):
    r = torch.arange(n, dtype=torch.float64, device=dev)[None, :]
    s = (math.sqrt(2.0) * sig)[:, None]
    g = torch.special.erf((r + 0.5 - n / 2) / s) - torch.special.erf((r - 0.5 - n / 2) / s)
    return g / (2.0 * torch.special.erf(0.5 / s))


def _cotangents(case, seed, dev):
    g = _gen(seed + 500009, dev)
    return (torch.randn((case["n"], 2), dtype=torch.float64, device=dev, generator=g),
            torch.randn((case["n"],), dtype=torch.float64, device=dev, generator=g) * 1e-9)


def prepare(case, seed):
    frames, refs, ids = _inputs(case, seed)
    tr = Tracker(mode=case["mode"], eps=EPS, upsample=case["u"], precision=case["precision"],
                 streams=case["streams"])
    s = dict(case=case, tr=tr, frames=frames)
    if case["kind"] == "rois":
        tr.set_reference(refs)
        s["rois"] = tr.rois(frames, ids)
    elif case["kind"] == "train":
        s["frames"] = frames.contiguous().requires_grad_(True)
        s["ref"] = refs.requires_grad_(True)
        s["g"] = _cotangents(case, seed, frames.device)
    elif case["kind"] == "refine":
        pass  # the reference starts as the first frame
    else:
        tr.set_reference(refs)
    if case["kind"] == "update":
        s["next"] = 0
    return s


# ----------------------------------------------------------------------- runs
def _fields(res):
    """Device views of a result buffer's fields."""
    n = res.shape[0]
    flat = res.reshape(-1)
    f64 = flat.view(torch.float64).reshape(n, 9)
    i32 = flat.view(torch.int32).reshape(n, 18)
    return dict(d=f64[:, 0:2], peak=f64[:, 2], hess=f64[:, 3:6], p=i32[:, 14:16], status=i32[:, 16])


def run(state):
    case, tr = state["case"], state["tr"]
    if case["kind"] == "track":
        return _fields(tr.track(state["frames"]))
    if case["kind"] == "rois":
        return _fields(tr.track(None, rois=state["rois"]))
    if case["kind"] == "update":
        k = state["next"]
        state["next"] = (k + 1) % case["n"]
        return _fields(tr.track_update(state["frames"][k], 0.1))
    if case["kind"] == "train":
        d, peak, status = track_with_grad(state["frames"], state["ref"], tr)
        gf, gr = torch.autograd.grad((d, peak), (state["frames"], state["ref"]), state["g"])
        return dict(d=d.detach(), peak=peak.detach(), status=status, grad_frames=gf, grad_ref=gr)
    E, res = iterate_reference(tr, state["frames"], passes=case["passes"])
    return dict(E=E, last=_fields(res))


# ----------------------------------------------------------------------- work
def work(case):
    """Bytes and operations of one pass: every frame and reference read once
    and every output written once; the r2c and c2r FFTs of the frames, the
    upsampled grid as two real contractions over each axis's conjugate pairs
    and mirrored offsets, one FP64 evaluation of the spectrum for the
    refinement."""
    px = {"u16": 2, "f32": 4, "f64": 8}[case["dtype"]]
    M = math.ceil(1.5 * case["u"])

    def one(ny, nx):
        h = nx // 2 + 1
        fft = 2 * 2.5 * ny * nx * math.log2(ny * nx)
        return fft + 6 * ny * h + 2.0 * M * ny * h + 2.0 * M * M * h + 20.0 * ny * h

    n = 1 if case["kind"] == "update" else case["n"]
    if case["kind"] == "rois":
        sizes = [s for s in (16, 24, 32, 48, 64, 96, 128, 192, 256) if case["ny"] <= s <= case["nx"]]
        frames = n * sum(s * s for s in sizes) / len(sizes)
        return {"bytes": frames * (px + 4) + 72.0 * n, "flops": n * sum(one(s, s) for s in sizes) / len(sizes)}
    ny, nx = case["ny"], case["nx"]
    by, fl = n * (ny * nx * px + 72.0) + 4.0 * ny * nx, n * one(ny, nx)
    fft = 2.5 * ny * nx * math.log2(ny * nx)
    if case["kind"] == "update":  # the reference is read and written
        by += 4.0 * ny * nx
        fl += (2 if case["mode"] == "ccsn" else 0) * fft + 10.0 * ny * nx
    if case["kind"] == "train":  # frame gradients and the reference's
        by += 4.0 * (n + 1) * ny * nx
        fl += n * (fft + 20.0 * ny * nx) + fft
    if case["kind"] == "refine":
        fl = (fl + n * 10.0 * ny * nx) * case["passes"]
        by += n * (case["passes"] - 1) * ny * nx * px + 4.0 * ny * nx
    return {"bytes": by, "flops": fl}


# ---------------------------------------------------------------- 64-bit values
def _phi(n, s, order):
    """d^order/ds^order of exp(2 pi i k s / n) over signed k, cos(pi s) at the
    Nyquist bin: [len(s), n] complex128."""
    k = torch.fft.fftfreq(n, device=s.device, dtype=torch.float64) * n
    w = 2.0 * math.pi / n * k
    v = torch.exp(1j * w[None, :] * s[:, None]) * (1j * w[None, :]) ** order
    v[:, n // 2] = math.pi ** order * torch.cos(math.pi * s + 0.5 * math.pi * order).to(v.dtype)
    return v


def _weights(case, frames, refs):
    if case["mode"] == "ccu":
        return frames, refs
    return (frames + EPS) ** 2, -1.0 / (refs + EPS)


def _moments(X, s):
    """C, gradient and Hessian of the band-limited correlation at s [n, 2]."""
    ny, nx = X.shape[-2:]
    vy = torch.stack([_phi(ny, s[:, 0], o) for o in range(3)], 1)
    vx = torch.stack([_phi(nx, s[:, 1], o) for o in range(3)], 2)
    a = torch.bmm(torch.bmm(vy.contiguous(), X), vx.contiguous()).real / (ny * nx)
    return a[:, 0, 0], torch.stack([a[:, 1, 0], a[:, 0, 1]], 1), torch.stack([a[:, 2, 0], a[:, 1, 1], a[:, 0, 2]], 1)


def _solve(h, g):
    det = h[:, 0] * h[:, 2] - h[:, 1] ** 2
    return torch.stack([h[:, 2] * g[:, 0] - h[:, 1] * g[:, 1], h[:, 0] * g[:, 1] - h[:, 1] * g[:, 0]], 1) / det[:, None]


def _exact_track(case, frames, ref, own_refs=False):
    """Displacements, peak values and Hessians of frames [n, ny, nx] against a
    reference (one, or one each) in float64, with the spectra F[A], F[B]."""
    d, c, h, p = [], [], [], []
    ny, nx = frames.shape[-2:]
    step = max(1, (1 << 25) // (ny * nx))
    for i in range(0, frames.shape[0], step):
        fr = frames[i:i + step].to(torch.float64)
        A, B = _weights(case, fr, (ref[i:i + step] if own_refs else ref).to(torch.float64))
        X = torch.fft.fft2(A) * torch.fft.fft2(B).conj()
        cc = torch.fft.ifft2(X).real.reshape(fr.shape[0], -1)
        at = cc.argmax(1)
        py, px = at // nx, at % nx
        pk = torch.stack([torch.where(2 * py >= ny, py - ny, py), torch.where(2 * px >= nx, px - nx, px)], 1)
        s = pk.to(torch.float64)
        # the best point of a 13 x 13 grid over the 1.5-px window, then Newton
        o = torch.linspace(-0.72, 0.72, 13, dtype=torch.float64, device=fr.device)
        Xp = X * _phi(ny, s[:, 0], 0)[:, :, None] * _phi(nx, s[:, 1], 0)[:, None, :]
        gy, gx = _phi(ny, o, 0), _phi(nx, o, 0)
        g = torch.matmul(torch.matmul(gy, Xp), gx.t().contiguous()).real.reshape(fr.shape[0], -1)
        k = g.argmax(1)
        s = s + torch.stack([o[k // 13], o[k % 13]], 1)
        for _ in range(9):
            _, gr, he = _moments(X, s)
            s = s - _solve(he, gr)
        v, _, he = _moments(X, s)
        d.append(s)
        c.append(v)
        h.append(he)
        p.append(pk)
    return torch.cat(d), torch.cat(c), torch.cat(h), torch.cat(p)


def _exact_align(frames, d):
    """The mean of the frames shifted back by d, float64."""
    ny, nx = frames.shape[-2:]
    acc = torch.zeros((ny, nx), dtype=torch.complex128, device=frames.device)
    step = max(1, (1 << 25) // (ny * nx))
    for i in range(0, frames.shape[0], step):
        F = torch.fft.fft2(frames[i:i + step].to(torch.float64))
        e = d[i:i + step]
        acc += (F * _phi(ny, e[:, 0], 0)[:, :, None] * _phi(nx, e[:, 1], 0)[:, None, :]).sum(0)
    return torch.fft.ifft2(acc / frames.shape[0]).real


def _exact_grad(case, frames, ref, d, h, g_d, g_c):
    """Gradients of sum(g_d . d + g_c C) by the implicit function theorem."""
    ny, nx = frames.shape[-2:]
    lam = -_solve(h, g_d)
    gf = torch.empty(frames.shape, dtype=torch.float64, device=frames.device)
    gB = torch.zeros((ny, nx), dtype=torch.float64, device=frames.device)
    E = ref.to(torch.float64)
    step = max(1, (1 << 25) // (ny * nx))
    for i in range(0, frames.shape[0], step):
        k = slice(i, i + step)
        fr = frames[k].to(torch.float64)
        A, B = _weights(case, fr, E)
        y0, y1 = _phi(ny, d[k, 0], 0), _phi(ny, d[k, 0], 1)
        x0, x1 = _phi(nx, d[k, 1], 0), _phi(nx, d[k, 1], 1)
        psi = ((lam[k, 0:1] * y1 + g_c[k, None] * y0)[:, :, None] * x0[:, None, :]
               + (lam[k, 1:2] * y0)[:, :, None] * x1[:, None, :]) / (ny * nx)
        gA = torch.fft.fft2(torch.fft.fft2(B).conj() * psi).real
        gf[k] = gA if case["mode"] == "ccu" else gA * 2.0 * (fr + EPS)
        gB += (torch.fft.ifft2(torch.fft.fft2(A) * psi).real * (ny * nx)).sum(0)
    return gf, gB if case["mode"] == "ccu" else gB / (E + EPS) ** 2


def exact(case, seed):
    frames, ref, _ = _inputs(case, seed)
    if case["kind"] == "rois":
        n = len(frames)
        dev = frames[0].device
        d = torch.empty((n, 2), dtype=torch.float64, device=dev)
        c, h = torch.empty(n, dtype=torch.float64, device=dev), torch.empty((n, 3), dtype=torch.float64, device=dev)
        for s in sorted({f.shape[0] for f in frames}):
            ids = [i for i in range(n) if frames[i].shape[0] == s]
            at = torch.tensor(ids, device=dev)
            d[at], c[at], h[at], _ = _exact_track(
                case, torch.stack([frames[i].to(torch.float64) for i in ids]), torch.stack([ref[i] for i in ids]), True)
        return dict(d=d, peak=c, hess=h, p=None, status=None)
    if case["kind"] == "update":  # the first frame, against the reference as set
        d, c, h, _ = _exact_track(case, frames[:1], ref)
        return dict(d=d, peak=c, hess=h, p=None, status=None)
    if case["kind"] == "refine":
        E = frames[0].to(torch.float64)
        for _ in range(case["passes"]):
            d, c, h, _ = _exact_track(case, frames, E)
            E = _exact_align(frames, d)
        return dict(E=E, last=dict(d=d, peak=c, hess=h, p=None, status=None))
    d, c, h, _ = _exact_track(case, frames, ref)
    if case["kind"] == "train":
        gf, gr = _exact_grad(case, frames, ref, d, h, *_cotangents(case, seed, frames.device))
        return dict(d=d, peak=c, status=None, grad_frames=gf, grad_ref=gr)
    return dict(d=d, peak=c, hess=h, p=None, status=None)
