"""Timed cases of the speckle-masking library: what a user's program has it do.

``listed()`` names the fixed cases, ``draw(rng)`` gives another one of the same
ranges, ``prepare`` makes what the program holds before a call (frames or
intermediate arrays on the GPU, made from the seed, and the session with its
buffers), ``run`` is one pass through the public entry points, ``work`` the
bytes and operations the pass cannot do without, and ``exact`` the same
outputs in 64-bit torch arithmetic (no code of the package).

Kinds: ``burst`` frames to image (``Session.reconstruct``); ``accumulate``,
``solve`` and ``synth`` the three stages on their own; ``batch`` several uneven
bursts in one call; ``stream`` a burst arriving in groups of frames;
``seeing`` the D/r0 estimate with its model transfer functions.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1701_00581_amd as nv

DEV = "cuda"
# bispectrum terms (samples x patches x frames) above which exact() would
# take longer than is reasonable
EXACT_TERMS = 6e10
# bispectrum terms of the largest listed case: no drawn case exceeds it
MOST_TERMS = 1.61e11


# ---------------------------------------------------------------------------
# Cases.
# ---------------------------------------------------------------------------
def _burst(name, kind, N, H, W, F, dtype, R, window=1, noise_bias=1, **kw):
    c = dict(kind=kind, N=N, H=H, W=W, F=F, dtype=dtype, R=R, window=window, noise_bias=noise_bias, **kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one isoplanatic subimage of photon counts, no taper: the smallest
        # call, where launches and the serial phase recursion count
        _burst("single64", "burst", 64, 64, 64, 100, "f32", 8, window=0),
        # a ragged crop with an odd frame count (12 patches, the last row and
        # column clamped): a quick look at a region
        _burst("crop250x300", "burst", 128, 250, 300, 101, "u16", 10),
        # the smaller camera's whole burst
        _burst("burst1024", "burst", 128, 1024, 1024, 100, "u16", 10),
        # the large camera's whole burst: the throughput case
        _burst("burst2560", "burst", 128, 2160, 2560, 100, "u16", 12),
        # the accumulation stage alone on float frames of odd shape, for
        # programs that keep the bispectrum
        _burst("accumulate_f32", "accumulate", 128, 611, 517, 73, "f32", 12, noise_bias=0),
        # the accumulation with the photon-noise model (low light)
        _burst("accumulate_photon", "accumulate", 128, 512, 512, 100, "u16", 10, noise_bias=2),
        # modulus and phase recursion of a 1024 x 1024 burst's 225 patches
        dict(name="solve1024", kind="solve", N=128, H=1024, W=1024, R=10, iters=0),
        # the same with ten least-squares steps
        dict(name="solve_lsq", kind="solve", N=128, H=640, W=640, R=10, iters=10),
        # subimages and mosaic of the large camera's field
        dict(name="synth2560", kind="synth", N=128, H=2160, W=2560, R=12),
        # eight small bursts of uneven shape and frame count in one call
        dict(name="batch8", kind="batch", N=128, R=10, bursts=8, side=512, F=120, dtype="u16"),
        # a 1024 x 1024 burst arriving in groups of 20 frames, then finished
        dict(name="stream1024", kind="stream", N=128, H=1024, W=1024, F=100, group=20, dtype="u16", R=10),
        # seeing estimate of a 1024 x 1024 burst at the default settings
        dict(name="seeing1024", kind="seeing", N=128, H=1024, W=1024, F=100, dtype="u16", screens=1000, points=40),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _terms(c):
    """Bispectrum terms of a case with frames (the batch: of its bursts)."""
    if c["kind"] == "batch":
        return sum(_n_samples(c["N"] // 2 - 1, c["R"]) * _n_patches(c["N"], h, w) * f
                   for f, h, w in _batch_shapes(c))
    return _n_samples(c["N"] // 2 - 1, c["R"]) * _n_patches(c["N"], c["H"], c["W"]) * c.get("F", 1)


def draw(rng):
    kind = rng.choice(["burst", "burst", "burst", "accumulate", "accumulate", "solve", "solve", "synth", "batch",
                       "stream", "seeing"])
    while True:
        N = 64 if rng.random() < 0.3 else 128
        R = rng.randint(5, 8) if N == 64 else rng.randint(8, 12)
        H, W = _log_int(rng, N, 2200), _log_int(rng, N, 2600)
        # images come from bursts of about 100 exposures (with far fewer, single
        # frequencies whose samples cancel make an image unstable in any
        # arithmetic); the accumulation and the seeing take short ones too
        F = rng.randint(24, 130) if kind in ("accumulate", "seeing") else rng.randint(88, 130)
        dtype = rng.choice(["u16", "u16", "f32"])
        if kind == "burst":
            c = _burst(None, kind, N, H, W, F, dtype, R)
        elif kind == "accumulate":
            c = _burst(None, kind, N, min(H, 900), min(W, 900), F, dtype, R, noise_bias=rng.choice([0, 2]))
        elif kind == "solve":
            c = dict(kind=kind, N=N, H=min(H, 1100), W=min(W, 1100), R=R, iters=rng.choice([0, 0, rng.randint(1, 10)]))
        elif kind == "synth":
            c = dict(kind=kind, N=N, H=H, W=W, R=R)
        elif kind == "batch":
            c = dict(kind=kind, N=N, R=R, bursts=rng.randint(2, 10), side=_log_int(rng, 2 * N, 700), F=F, dtype=dtype)
        elif kind == "stream":
            c = dict(kind=kind, N=N, H=min(H, 1100), W=min(W, 1100), F=F, group=rng.randint(8, 40), dtype=dtype, R=R)
        else:
            c = dict(kind=kind, N=N, H=min(H, 1500), W=min(W, 1500), F=F, dtype=dtype,
                     screens=2 * rng.randint(100, 500), points=rng.randint(16, 40))
        if kind in ("synth", "seeing") or _terms(c) <= (MOST_TERMS if kind == "burst" else 2.5e10):
            return c


# ---------------------------------------------------------------------------
# Index sets (numpy, in the library's documented orders).
# ---------------------------------------------------------------------------
def _tiles(L, N):
    n = -(-(L - N) // (N // 2)) + 1
    return [min(k * (N // 2), L - N) for k in range(n)]


def _n_patches(N, H, W):
    return len(_tiles(H, N)) * len(_tiles(W, N))


def _sets(uc, R):
    """W [n][2] by |w|^2, wy, wx; per sample the index of its w, and v."""
    y, x = np.mgrid[0:uc + 1, -uc:uc + 1]
    x, y = x.ravel(), y.ravel()
    r2 = x * x + y * y
    ok = (r2 > 0) & (r2 <= uc * uc) & ((y > 0) | (x > 0))
    x, y, r2 = x[ok], y[ok], r2[ok]
    o = np.lexsort((x, y, r2))
    w = np.stack([x[o], y[o]], 1)
    vy, vx = np.mgrid[-R:R + 1, -R:R + 1]
    v = np.stack([vx.ravel(), vy.ravel()], 1)
    v2 = (v * v).sum(1)
    v, v2 = v[(v2 > 0) & (v2 <= R * R)], v2[(v2 > 0) & (v2 <= R * R)]
    n2 = (w * w).sum(1)[:, None]
    d2 = ((w[:, None, :] - v[None]) ** 2).sum(2)
    wi, vi = np.nonzero((v2[None] < n2) & (d2 > 0) & (d2 < n2))
    return w, wi, v[vi], v, vi


_SIZES = {}


def _n_samples(uc, R):
    if (uc, R) not in _SIZES:
        w, wi, _, _, _ = _sets(uc, R)
        _SIZES[uc, R] = (len(w), len(wi))
    return _SIZES[uc, R][1]


def _n_freqs(uc, R):
    _n_samples(uc, R)
    return _SIZES[uc, R][0]


def _flat(a, N):
    return torch.from_numpy((a[:, 1] % N) * N + a[:, 0] % N).to(DEV)


# ---------------------------------------------------------------------------
# Synthetic inputs: turbulent short exposures of a granulation-like object.
# ---------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _freqs(H, W, half=False):
    fy = torch.fft.fftfreq(H, device=DEV)[:, None]
    fx = (torch.fft.rfftfreq if half else torch.fft.fftfreq)(W, device=DEV)[None, :]
    return torch.sqrt(fx * fx + fy * fy)


def _otfs(M, n, d_over_r0, g):
    """PSFs [n][M][M] of unit sum through Kolmogorov screens (FFT method with
    three subharmonic levels), pupil of diameter M/2."""
    r0 = (M / 2) / d_over_r0
    psd = lambda f: math.sqrt(0.023) * r0 ** (-5 / 6) * f ** (-11 / 6)  # noqa: E731
    f = _freqs(M, M)
    sig = torch.where(f > 0, psd(f.clamp_min(1e-9)), torch.zeros_like(f)) / M
    c = torch.randn(n, M, M, dtype=torch.complex64, generator=g, device=DEV) * (sig * math.sqrt(2))
    scr = torch.fft.fft2(c).real
    t = torch.arange(M, device=DEV, dtype=torch.float32)
    for p in (1, 2, 3):
        for iy, ix in ((0, 1), (1, 0), (1, 1), (1, -1)):
            fr = math.hypot(ix, iy) / M / 3 ** p
            amp = psd(fr) / M / 3 ** p * math.sqrt(2)
            k = torch.randn(n, 2, 1, 1, generator=g, device=DEV) * amp
            a = (2 * math.pi / M / 3 ** p) * (iy * t[:, None] + ix * t[None, :])
            scr += k[:, 0] * torch.cos(a) + k[:, 1] * torch.sin(a)
    d = t - (M - 1) / 2
    pupil = (d[:, None] ** 2 + d[None, :] ** 2 <= (M / 4) ** 2).float()
    psf = torch.fft.fft2(pupil * torch.polar(torch.ones_like(scr), scr)).abs() ** 2
    return psf / psf.sum((1, 2), keepdim=True)


def _turbulence(N):
    return (256, 15.0) if N == 128 else (64, 10.0)      # PSF grid, D/r0


def _frames(N, H, W, F, dtype, seed, photons=1e4):
    """Frames [F][H][W]: 12-bit camera units (int16 bits) or photon counts."""
    M, x = _turbulence(N)
    g = _gen(seed)
    Hs, Ws = (-(-max(L, M) // 32) * 32 for L in (H, W))
    k = _freqs(Hs, Ws, half=True)
    obj = torch.fft.rfft2(torch.randn(Hs, Ws, generator=g, device=DEV))
    obj = torch.fft.irfft2(obj * torch.where(k > 0, k.clamp_min(1e-9) ** -1.5, torch.zeros_like(k)), s=(Hs, Ws))
    obj = torch.fft.rfft2(1 + 0.1 * (obj - obj.mean()) / obj.std())
    out = torch.empty(F, H, W, dtype=torch.int16 if dtype == "u16" else torch.float32, device=DEV)
    h, step = M // 2, max(1, min(F, (1 << 25) // (Hs * Ws)))
    for f in range(0, F, step):
        n = min(step, F - f)
        psf = _otfs(M, n, x, g)
        big = torch.zeros(n, Hs, Ws, device=DEV)
        for ys, yd in ((slice(0, h), slice(0, h)), (slice(h, M), slice(Hs - h, Hs))):
            for xs, xd in ((slice(0, h), slice(0, h)), (slice(h, M), slice(Ws - h, Ws))):
                big[:, yd, xd] = psf[:, ys, xs]
        img = torch.fft.irfft2(torch.fft.rfft2(big) * obj, s=(Hs, Ws))[:, :H, :W].clamp_min(0)
        ph = torch.poisson((img * photons).contiguous(), generator=g)
        out[f:f + n] = (ph * (2048 / photons)).round().clamp(0, 4095).to(torch.int16) if dtype == "u16" else ph
    return out


def _stf(N):
    """Speckle transfer function [N][N]: the mean of 200 screens."""
    M, x = _turbulence(N)
    o = torch.fft.fft2(_otfs(M, 200, x, _gen(7)).double()).abs().square().mean(0)
    k = (torch.fft.fftfreq(N, device=DEV) * N).round().long() * (M // N) % M
    return (o / o[0, 0])[k][:, k].contiguous()


def _spectra_like(c, seed):
    """Inputs of the solve (power, mean spectrum, bispectrum) of an object of
    random phases seen through a falling transfer, with noise growing towards
    the cut-off; and the modulus and phasors a solve would return."""
    N, uc, R = c["N"], c["N"] // 2 - 1, c["R"]
    P = _n_patches(N, c["H"], c["W"])
    g = _gen(seed)
    w, wi, sv, _, _ = _sets(uc, R)
    f = (_freqs(N, N) * N).float()
    amp = 1e5 * (1 + f) ** -1.5 * (1 - f / N).clamp_min(0.05)
    phi = (torch.rand(P, N * N, generator=g, device=DEV) - 0.5) * 2 * math.pi
    iw, iv, idd = _flat(w, N), _flat(sv, N), _flat(w[wi] - sv, N)
    neg = _flat(-w, N)
    phi[:, neg] = -phi[:, iw]
    power = (amp * amp)[None] * (0.5 + torch.rand(P, N, N, generator=g, device=DEV))
    a = amp.reshape(-1)
    noise = 0.2 + 2.0 * (f.reshape(-1)[iw][wi] / uc)
    bis = torch.empty(P, len(wi), 2, device=DEV)
    for k in range(P):
        ph = phi[k]
        b = torch.polar(a[idd] * a[iv] * a[iw][wi], ph[idd] + ph[iv] - ph[iw][wi])
        n = torch.randn(len(wi), dtype=torch.complex64, generator=g, device=DEV) * noise
        bis[k] = torch.view_as_real(b * (1 + n))
    seeds = torch.stack([phi[:, 1], phi[:, N]], 1)                  # (1, 0) and (0, 1)
    mean = torch.view_as_real(torch.polar(torch.full_like(seeds, 3e4), seeds)).contiguous()
    return power, mean, bis, phi[:, iw], a[iw]


# ---------------------------------------------------------------------------
# prepare / run
# ---------------------------------------------------------------------------
def _params(c):
    kw = dict(v_radius=c["R"], window=c.get("window", 1), noise_bias=c.get("noise_bias", 1), filter=1)
    if kw["noise_bias"] == 2:
        kw["photons_per_adu"] = 1e4 / 2048 if c["dtype"] == "u16" else 1.0
    if c.get("iters"):
        kw.update(phase_method=1, lsq_iters=c["iters"])
    return nv.default_params(c["N"], **kw)


def _batch_shapes(c):
    """(F, H, W) of each burst: sides from the class's down to half of it."""
    N, n = c["N"], c["bursts"]
    return [(max(8, c["F"] - 3 * i), max(N, c["side"] - i * c["side"] // (2 * n)),
             max(N, c["side"] - ((3 * i + 1) % n) * c["side"] // (2 * n))) for i in range(n)]


class _State:
    """What the program keeps: a library context and its buffers."""

    def __init__(self):
        self.ctx = nv.nvsm_create(0)

    def __del__(self):
        nv.nvsm_destroy(self.ctx)


def _bytes(n):
    return torch.empty(int(n), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    kind, N = case["kind"], case["N"]
    if kind in ("burst", "accumulate"):
        st = nv.Session(_params(case), case["H"], case["W"], case["F"])
        st.frames = _frames(N, case["H"], case["W"], case["F"], case["dtype"], seed)
        st.stf = _stf(N)
    elif kind == "solve":
        st = nv.Session(_params(case), case["H"], case["W"], 1)
        power, mean, bis, _, _ = _spectra_like(case, seed)
        st.power.copy_(power), st.mean_spec.copy_(mean), st.bispec.copy_(bis)
        st.stf = _stf(N)
    elif kind == "synth":
        st = nv.Session(_params(case), case["H"], case["W"], 1)
        amp, phasor, mu = _synth_inputs(case, seed)
        st.amp.copy_(amp), st.phasor.copy_(phasor), st.mu.copy_(mu)
    elif kind == "batch":
        st = _State()
        st.p = _params(case)
        stf = _stf(N)
        st.bursts = [(_frames(N, h, w, f, case["dtype"], seed * 100 + i), stf, torch.empty(h, w, device=DEV))
                     for i, (f, h, w) in enumerate(_batch_shapes(case))]
        st.ws = _bytes(nv.nvsm_batch_plan(st.p, _batch_shapes(case))[1])
        nv.nvsm_prepare(st.ctx, st.p)
    elif kind == "stream":
        st = _State()
        st.p = _params(case)
        st.frames = _frames(N, case["H"], case["W"], case["F"], case["dtype"], seed)
        st.stf = _stf(N)
        st.out = torch.empty(case["H"], case["W"], device=DEV)
        st.state, st.ws = (_bytes(n) for n in nv.nvsm_stream_plan(st.p, case["H"], case["W"],
                                                                  min(case["group"], case["F"])))
        nv.nvsm_prepare(st.ctx, st.p)
    else:
        st = _State()
        st.p = nv.default_params(N)
        st.sp = nv.seeing_default_params(screens=case["screens"], points=case["points"], seed=seed + 1)
        st.frames = _frames(N, case["H"], case["W"], case["F"], case["dtype"], seed)
        n, cubes = nv.nvsm_seeing_plan(st.p, st.sp, case["H"], case["W"], case["F"])
        st.ws = _bytes(n)
        st.x = torch.empty(1 + cubes, dtype=torch.float64, device=DEV)
        st.stf = torch.empty(N, N, dtype=torch.float64, device=DEV)
        st.curves = torch.empty(cubes, st.sp.bins, dtype=torch.float64, device=DEV)
        nv.nvsm_prepare(st.ctx, st.p)
    st.case = case
    return st


def run(st):
    kind = st.case["kind"]
    if kind == "burst":
        return st.reconstruct(st.frames, st.stf)
    if kind == "accumulate":
        st.accumulate(st.frames)
        return {"power": st.power, "mean_spec": st.mean_spec, "mu": st.mu, "bispec": st.bispec}
    if kind == "solve":
        st.solve(st.stf)
        return {"amp": st.amp, "phasor": st.phasor}
    if kind == "synth":
        st.synthesize()
        return {"patches": st.patches, "image": st.image}
    if kind == "batch":
        nv.nvsm_reconstruct_batch(st.ctx, st.p, st.bursts, st.ws)
        return [out for _, _, out in st.bursts]
    if kind == "stream":
        F, G = st.case["F"], st.case["group"]
        for f in range(0, F, G):
            n = min(G, F - f)
            nv.nvsm_stream_add(st.ctx, st.p, st.frames[f:f + n], f, F if f + n == F else 0, st.state, st.ws)
        nv.nvsm_stream_finish(st.ctx, st.p, st.case["H"], st.case["W"], st.stf, st.out, st.ws)
        return st.out
    nv.nvsm_seeing(st.ctx, st.p, st.sp, st.frames, st.x, st.stf, st.ws, st.curves)
    return {"d_over_r0": st.x, "stf": st.stf, "curves": st.curves}


def _synth_inputs(c, seed):
    _, _, P = c["H"], c["W"], _n_patches(c["N"], c["H"], c["W"])
    g = _gen(seed)
    w, _, _, _, _ = _sets(c["N"] // 2 - 1, c["R"])
    r = torch.from_numpy(np.hypot(w[:, 0], w[:, 1])).to(DEV)
    amp = 1e5 * (1 + r) ** -1.5 * (0.5 + torch.rand(P, len(w), dtype=torch.float64, generator=g, device=DEV))
    t = 2 * math.pi * torch.rand(P, len(w), dtype=torch.float64, generator=g, device=DEV)
    return amp, torch.stack([torch.cos(t), torch.sin(t)], 2), 1000 * (1 + 0.1 * torch.rand(P, generator=g, device=DEV))


# ---------------------------------------------------------------------------
# work: bytes in and out once, operations of the method
# ---------------------------------------------------------------------------
def work(case):
    kind, N = case["kind"], case["N"]
    nW, S = (_n_freqs(N // 2 - 1, case["R"]), _n_samples(N // 2 - 1, case["R"])) if "R" in case else (0, 0)
    fft = 5 * N * N * math.log2(N * N)
    px = 2 if case.get("dtype") == "u16" else 4
    shapes = _batch_shapes(case) if kind == "batch" else [(case.get("F", 1), case["H"], case["W"])]
    frames = sum(f * h * w for f, h, w in shapes) * px
    pixels = sum(h * w for _, h, w in shapes)
    P = sum(_n_patches(N, h, w) for _, h, w in shapes)
    PF = sum(_n_patches(N, h, w) * f for f, h, w in shapes)
    acc = PF * (fft / 2 + 3 * N * N) + 14 * S * PF          # two real frames per transform
    solve = P * 16 * S
    if kind in ("burst", "batch", "stream"):
        return dict(bytes=frames + 8 * N * N + 4 * pixels, flops=acc + solve + P * fft)
    if kind == "accumulate":
        extra = PF * (fft / 2 + 8 * N * N) if case["noise_bias"] == 2 else 0
        return dict(bytes=frames + P * (4 * N * N + 8 * S), flops=acc + extra)
    if kind == "solve":
        return dict(bytes=P * (8 * S + 4 * N * N + 24 * nW), flops=solve + case["iters"] * P * 48 * S)
    if kind == "synth":
        return dict(bytes=P * (24 * nW + 4 * N * N) + 4 * pixels, flops=P * fft)
    cubes = (case["H"] // N) * (case["W"] // N)
    return dict(bytes=frames + 8 * N * N, flops=(case["points"] + 1) * case["screens"] * 2.5 * fft + cubes * case["F"] * fft / 2)


# ---------------------------------------------------------------------------
# exact: the same outputs in 64 bits
# ---------------------------------------------------------------------------
def _hann(N):
    return 0.5 - 0.5 * torch.cos(2 * math.pi * torch.arange(N, dtype=torch.float64, device=DEV) / N)


def _taper(N, window):
    return torch.outer(_hann(N), _hann(N)) if window else torch.ones(N, N, dtype=torch.float64, device=DEV)


def _accumulate64(frames, N, R, window, noise_bias, gain, y, x, sets, bispec=True):
    """power, (I(1,0), I(0,1)), level and bispectrum of the patch at (y, x)."""
    w, wi, sv, _, _ = sets
    t = _taper(N, window)
    p = frames[:, y:y + N, x:x + N]
    p = (p.int() & 0xffff).double() if p.dtype == torch.int16 else p.double()
    mu = (t * p).sum((1, 2)) / t.sum()
    spec = torch.fft.fft2((p - mu[:, None, None]) * t)
    power = spec.abs().square().mean(0)
    mean = torch.stack([spec[:, 0, 1].mean(), spec[:, 1, 0].mean()])
    bis = None
    if bispec:
        rows = spec.reshape(len(spec), N * N).t().contiguous()       # a frequency's frames side by side
        iw, iv, idd = _flat(w, N)[torch.from_numpy(wi).to(DEV)], _flat(sv, N), _flat(w[wi] - sv, N)
        bis = torch.empty(len(wi), dtype=torch.complex128, device=DEV)
        for a in range(0, len(wi), 1 << 18):
            s = slice(a, a + (1 << 18))
            bis[s] = (rows[idd[s]] * rows[iv[s]] * rows[iw[s]].conj()).mean(1)
    if noise_bias == 2:
        q = torch.fft.fft2(p * t * t) / gain
        cc = (spec.conj() * q).mean(0).reshape(-1)
        power = power - (p * t * t).sum((1, 2)).mean() / gain
        if bispec:
            third = (p * t ** 3).sum((1, 2)).mean() / gain ** 2
            bis = bis - (cc[iw] + cc[iv].conj() + cc[idd].conj()) + 2 * third
    return power, mean, mu.mean(), bis


def _modulus64(power, stf, w, N, noise_bias, floor=1e-6):
    k = torch.fft.fftfreq(N, dtype=torch.float64, device=DEV) * N
    corner = k[:, None] ** 2 + k[None, :] ** 2 > (N / 2 + 2) ** 2
    nb = power[:, corner].mean(1, keepdim=True) if noise_bias == 1 else 0.0
    i = _flat(w, N)
    s = stf.reshape(-1)[i]
    a = ((power.reshape(len(power), -1)[:, i] - nb).clamp_min(0) / s).sqrt()
    return torch.where(s >= floor, a, torch.zeros_like(a))


def _unit(z):
    m = z.abs()
    return torch.where(m > 0, z / m.clamp_min(1e-300), torch.ones_like(z))


def _phases64(mean, bis, sets, N):
    """Phase recursion of all patches: mean [P][2], bis [P][S] complex."""
    w, wi, sv, _, _ = sets
    P = len(mean)
    E = torch.zeros(P, N * N, dtype=torch.complex128, device=DEV)
    iw, neg, iv, idd = _flat(w, N), _flat(-w, N), _flat(sv, N), _flat(w[wi] - sv, N)
    out = torch.empty(P, len(w), dtype=torch.complex128, device=DEV)
    first = np.searchsorted(wi, np.arange(len(w) + 1))
    r2 = (w * w).sum(1)
    shells = np.flatnonzero(np.diff(r2, prepend=-1, append=-1))
    for a, b in zip(shells[:-1], shells[1:]):
        if a == 0:
            z = mean
        else:
            lo, hi = first[a], first[b]
            t = E[:, idd[lo:hi]] * E[:, iv[lo:hi]] * bis[:, lo:hi].conj()
            n = int(np.max(np.diff(first[a:b + 1])))
            pad = torch.zeros(P, (b - a) * n, dtype=torch.complex128, device=DEV)
            k = wi[lo:hi]
            pad[:, torch.from_numpy((k - a) * n + np.arange(lo, hi) - first[k]).to(DEV)] = t
            z = pad.reshape(P, b - a, n).sum(2)
        e = _unit(z)
        out[:, a:b] = e
        E[:, iw[a:b]] = e
        E[:, neg[a:b]] = e.conj()
    return out


def _least_squares64(e, bis, sets, N, iters):
    """The refinement steps for one patch (e [W], bis [S]): samples laid out
    as a grid [v][u of the plane], so every sum is over one axis."""
    w, wi, sv, v, vi = sets
    iw, neg, iv = _flat(w, N), _flat(-w, N), _flat(v, N)
    wpos = iw[torch.from_numpy(wi).to(DEV)]
    B = torch.zeros(len(v), N * N, dtype=torch.complex128, device=DEV)
    B[torch.from_numpy(vi).to(DEV), wpos] = bis
    y, x = (torch.arange(N * N, device=DEV) // N), torch.arange(N * N, device=DEV) % N
    vt = torch.from_numpy(v).to(DEV)
    minus = ((y[None] - vt[:, 1:2]) % N) * N + (x[None] - vt[:, 0:1]) % N       # u - v
    plus = ((y[None] + vt[:, 1:2]) % N) * N + (x[None] + vt[:, 0:1]) % N        # u + v
    Bp = torch.gather(B, 1, plus)
    for _ in range(iters):
        E = torch.zeros(N * N, dtype=torch.complex128, device=DEV)
        E[iw], E[neg] = e, e.conj()
        Em, Ev = E[minus], E[iv][:, None]
        g = (Em * Ev * B.conj()).sum(0) + (Ev.conj() * E[plus] * Bp).sum(0)
        g.index_add_(0, iv, (Em.conj() * E[None] * B).sum(1))
        g = g[iw] + g[neg].conj()
        new = torch.where(g.abs() > 0, _unit(_unit(g) + e), e)
        new[:2] = e[:2]
        e = new
    return e


def _subimages64(amp, e, mu, w, N, window):
    rho = torch.from_numpy(np.hypot(w[:, 0], w[:, 1])).to(DEV) / (N / 2)
    val = amp * e * (2 / math.pi) * (torch.acos(rho) - rho * (1 - rho * rho).sqrt())
    spec = torch.zeros(len(amp), N * N, dtype=torch.complex128, device=DEV)
    spec[:, _flat(w, N)], spec[:, _flat(-w, N)] = val, val.conj()
    return torch.fft.ifft2(spec.reshape(-1, N, N)).real + mu[:, None, None] * _taper(N, window)


def _mosaic64(patches, N, H, W, window):
    num = torch.zeros(H, W, dtype=torch.float64, device=DEV)
    den = torch.zeros_like(num)
    t, k = _taper(N, window), 0
    for y in _tiles(H, N):
        for x in _tiles(W, N):
            num[y:y + N, x:x + N] += patches[k]
            den[y:y + N, x:x + N] += t
            k += 1
    return torch.where(den >= 1e-3, num / den.clamp_min(1e-3), torch.zeros_like(num))


def _stages64(c, frames, solve=True):
    """Accumulation of every patch of a burst; with solve: the image."""
    N, H, W = c["N"], c["H"], c["W"]
    nb, window = c.get("noise_bias", 1), c.get("window", 1)
    gain = 1e4 / 2048 if c["dtype"] == "u16" else 1.0
    sets = _sets(N // 2 - 1, c["R"])
    acc = [_accumulate64(frames, N, c["R"], window, nb, gain, y, x, sets) for y in _tiles(H, N) for x in _tiles(W, N)]
    power, mean, mu = (torch.stack([a[i] for a in acc]) for i in range(3))
    if not solve:
        bis = torch.view_as_real(torch.stack([a[3] for a in acc]))
        return {"power": power, "mean_spec": torch.view_as_real(mean), "mu": mu, "bispec": bis}
    e = _phases64(mean, torch.stack([a.pop() for a in map(list, acc)]), sets, N)
    amp = _modulus64(power, _stf(N), sets[0], N, nb)
    return _mosaic64(_subimages64(amp, e, mu, sets[0], N, window), N, H, W, window)


def _philox(c0, c1, c2, k0, k1):
    """Philox4x32-10 (Salmon et al. 2011) on int64 tensors holding 32 bits."""
    m = 0xffffffff
    c = [c0, c1, c2, torch.zeros_like(c1)]
    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
        # 32 x 32 bits in 64: the wrapped product has the right low 64 bits
        a, b = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((b >> 32) & m) ^ c[1] ^ k0, b & m, ((a >> 32) & m) ^ c[3] ^ k1, a & m]
    return c


def _model64(N, x, screens, seed, m):
    """<OTF> and <|OTF|^2> over the Kolmogorov screens of one model point."""
    pairs, nw = screens // 2, N * N // 2 + 12
    j = torch.arange(pairs, device=DEV)[:, None].expand(pairs, nw)
    word = torch.arange(nw, device=DEV)[None].expand(pairs, nw)
    r = _philox(j, word, torch.full_like(word, m), seed & 0xffffffff, seed >> 32)
    u = [(v.double() + 0.5) * 2.0 ** -32 for v in r]
    g = torch.stack([torch.polar((-2 * u[a].log()).sqrt(), 2 * math.pi * u[a + 1]) for a in (0, 2)], 2).reshape(pairs, -1)
    r0 = (N / 2) / x
    psd = lambda f: math.sqrt(0.023) * r0 ** (-5 / 6) * f ** (-11 / 6)  # noqa: E731
    k = torch.fft.fftfreq(N, dtype=torch.float64, device=DEV)
    f = torch.hypot(k[:, None], k[None, :])
    sig = torch.where(f > 0, psd(f.clamp_min(1e-9)), torch.zeros_like(f)) / N
    z = torch.fft.fft2(g[:, :N * N].reshape(-1, N, N) * sig)
    t, s = torch.arange(N, dtype=torch.float64, device=DEV), 0
    for p in (1, 2, 3):
        for iy in (-1, 0, 1):
            for ix in (-1, 0, 1):
                if ix or iy:
                    fr = 1 / (N * 3 ** p)
                    a = 2 * math.pi * fr * (iy * t[:, None] + ix * t[None, :])
                    amp = psd(math.hypot(ix, iy) * fr) * fr
                    z += (g[:, N * N + s] * amp)[:, None, None] * torch.polar(torch.ones_like(a), a)
                    s += 1
    d = t - (N - 1) / 2
    pupil = (d[:, None] ** 2 + d[None, :] ** 2 <= (N / 4) ** 2).double()
    A, S = torch.zeros(N, N, dtype=torch.complex128, device=DEV), torch.zeros(N, N, dtype=torch.float64, device=DEV)
    for phi in (z.real, z.imag):
        o = torch.fft.fft2(torch.fft.fft2(pupil * torch.polar(torch.ones_like(phi), phi)).abs() ** 2)
        o = o / o[:, :1, :1].real
        A += o.sum(0)
        S += o.abs().square().sum(0)
    return A / screens, S / screens


def _seeing64(c, frames, seed):
    N, J, Q, lo, hi = c["N"], c["points"], 12, 2.0, 50.0
    t = _taper(N, 1)
    grid = [lo * (hi / lo) ** (j / (J - 1)) for j in range(J)]
    rho = []
    for m, x in enumerate(grid):
        A, S = _model64(N, x, c["screens"], seed + 1, m)
        rho.append(A.abs() ** 2 / S)
    rho = torch.stack(rho)
    members = [[] for _ in range(Q)]
    for uy in range(Q + 1):
        for ux in range(-Q, Q + 1):
            q = math.floor(math.hypot(ux, uy) + 0.5)
            if (uy > 0 or ux > 0) and 1 <= q <= Q:
                members[q - 1].append(uy * N + ux % N)
    members = [torch.tensor(m, device=DEV) for m in members]
    annuli = lambda a: torch.stack([a.reshape(len(a), -1)[:, m].mean(1) for m in members], 1)  # noqa: E731
    curves, xs = [], []
    for i in range(c["H"] // N):
        for k in range(c["W"] // N):
            p = frames[:, i * N:i * N + N, k * N:k * N + N]
            p = (p.int() & 0xffff).double() if p.dtype == torch.int16 else p.double()
            F = len(p)
            spec = torch.fft.fft2((p - ((t * p).sum((1, 2)) / t.sum())[:, None, None]) * t)
            P, m2 = spec.abs().square().mean(0), spec.mean(0).abs() ** 2
            eps = annuli(((m2 - P / F) / (P * (1 - 1 / F)))[None])[0]
            P = P.clone()
            P[0, 0] = 0
            num, den = torch.zeros_like(rho), torch.zeros_like(P)
            for ky in (-1, 0, 1):
                for kx in (-1, 0, 1):
                    wt = (1 / 16 if ky else 1 / 4) * (1 / 16 if kx else 1 / 4)
                    num += wt * torch.roll(P * rho, (ky, kx), (1, 2))
                    den += wt * torch.roll(P, (ky, kx), (0, 1))
            err = ((annuli(num / den) - eps) ** 2).sum(1).tolist()
            j = min(range(J), key=lambda n: err[n])
            s = float(j)
            if 0 < j < J - 1 and (d := err[j - 1] - 2 * err[j] + err[j + 1]) > 0:
                s += 0.5 * (err[j - 1] - err[j + 1]) / d
            curves.append(eps)
            xs.append(lo * (hi / lo) ** (s / (J - 1)))
    x = len(xs) / sum(1 / v for v in xs)
    return {"d_over_r0": torch.tensor([x] + xs, dtype=torch.float64), "stf": _model64(N, x, c["screens"], seed + 1, J)[1],
            "curves": torch.stack(curves)}


def exact(case, seed):
    kind, N = case["kind"], case["N"]
    if kind in ("burst", "accumulate", "batch", "stream") and _terms(case) > EXACT_TERMS:
        return None
    if kind == "batch":
        return [_stages64(dict(case, H=h, W=w), _frames(N, h, w, f, case["dtype"], seed * 100 + i))
                for i, (f, h, w) in enumerate(_batch_shapes(case))]
    if kind == "synth":
        amp, phasor, mu = _synth_inputs(case, seed)
        w = _sets(N // 2 - 1, case["R"])[0]
        sub = _subimages64(amp, torch.view_as_complex(phasor), mu.double(), w, N, 1)
        return {"patches": sub, "image": _mosaic64(sub, N, case["H"], case["W"], 1)}
    if kind == "solve":
        power, mean, bis, _, _ = _spectra_like(case, seed)
        sets = _sets(N // 2 - 1, case["R"])
        bis = torch.view_as_complex(bis.double())
        e = _phases64(torch.view_as_complex(mean.double()), bis, sets, N)
        if case["iters"]:
            e = torch.stack([_least_squares64(e[k], bis[k], sets, N, case["iters"]) for k in range(len(e))])
        return {"amp": _modulus64(power.double(), _stf(N), sets[0], N, 1), "phasor": torch.view_as_real(e)}
    frames = _frames(N, case["H"], case["W"], case["F"], case["dtype"], seed)
    if kind == "seeing":
        return _seeing64(case, frames, seed)
    return _stages64(case, frames, solve=kind != "accumulate")
