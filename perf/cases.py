"""Workloads the library is timed on, through its public Python entry points.

A case is a dict of plain values.  ``prepare`` makes what a program holds
before the call (inputs, plans, loaded networks) on the GPU, ``run`` makes one
pass and returns its outputs, ``work`` gives the bytes and operations of one
pass, and ``exact`` the same outputs in 64-bit torch arithmetic written from
the definitions, with no code of the library.  ``draw`` makes further cases of
the same ranges.

Sizes are those of the repository's own workloads (the 64 px and 160 px
pyramids, six heterogeneous polychromatic sensors, the SOUL chain with its
detector, the Shack-Hartmann shapes, the closed loop, the surrogate network),
from one frame to full batches.
"""

from __future__ import annotations

import math
from types import SimpleNamespace

import torch

from paper_2602_06688_amd import pwfs as P
from paper_2602_06688_amd.loop import ClosedLoop

REF, FULL, LOCAL, ROOF = P.F_REF_SLOPES, P.F_FULL_PLANE, P.F_LOCAL_NORM, P.F_DOUBLE_ROOF
DEV = "cuda"
TWO_PI = 2.0 * math.pi


# ------------------------------------------------------------------ cases --
def _pwfs(name, **kw):
    c = dict(name=name, kind="pwfs", D=160, N=512, sub=40, mod=48, S=192, r=3.0, obs=0.12, nl=1, prec=P.FP32,
             flags=REF, rings=0, rho=0.0, fov=0.0, frames=1)
    c.update(kw)
    return c


def listed():
    return [
        # one frame of the 160 px sensor per call: a real-time timestep, where launches and latency count
        _pwfs("pyramid_160_one_frame"),
        # the small sensor's batch: many short transforms
        _pwfs("pyramid_64_batch", D=64, N=128, sub=16, mod=16, S=64, obs=0.0, frames=100),
        # the headline batch of the 160 px sensor: Monte-Carlo frames
        _pwfs("pyramid_160_batch", frames=1000),
        # the same sensor in the float32-accurate matrix-core precision a user may select
        _pwfs("pyramid_160_fp16x3", prec=P.FP16X3, frames=200),
        # six different three-wavelength sensors in one plan, one call per timestep batch
        dict(name="hetero_six", kind="hetero", frames=10),
        # the SOUL chain: 220 px pyramid behind a field stop, non-integer pixels, noisy detector, detector slopes
        dict(name="soul_chain", kind="soul", frames=100, photon=True, excess=True, readout=True),
        # Shack-Hartmann single-conjugate sensor, slopes and detector pixels
        dict(name="sh_scao", kind="sh", D=160, n=20, M=56, rebin=7, obs=0.12, nl=1, frames=500, pixels=True),
        # Shack-Hartmann for laser guide stars: many subapertures, fine focal sampling, slopes only
        dict(name="sh_lgs", kind="sh", D=476, n=68, M=240, rebin=15, obs=0.28, nl=1, frames=10, pixels=False),
        # one timestep of the closed loop (atmosphere, mirror, sensor, reconstructor, integrator) as a graph replay
        dict(name="closed_loop_step", kind="loop", modes=500, layers=4, screen=1024),
        # one training step of the surrogate network
        dict(name="surrogate_train", kind="train", inputs=500, hidden=1024, outputs=3200, batch=1024,
             prec=P.BF16),
        # a prediction of 20k samples by the network with its linear term
        dict(name="surrogate_predict", kind="predict", inputs=500, hidden=1024, outputs=3200, batch=20000,
             prec=P.BF16),
        # modal commands to wavefronts for a thousand samples (training data, interaction matrices)
        dict(name="modes_to_opd", kind="gemm", m=1000, n=25600, k=500, prec=P.BF16X3),
    ]


def _log_int(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def draw(rng):
    kind = rng.choice(["pwfs"] * 6 + ["hetero", "soul", "sh", "sh", "loop", "train", "predict", "gemm"])
    if kind == "pwfs":
        N = rng.choice([64, 128, 256, 384, 512, 768])
        D = 2 * _log_int(rng, 10, N // 4 if N <= 128 else int(N * 0.16))
        S = min(N - D, 2 * int(round(D * rng.choice([1.0, 1.2, 1.3]) / 2)))
        S = max(S, D)
        sub = rng.choice([b for b in range(4, 65) if D % b == 0 and D // b <= 8] or [min(40, D // 2)])
        if rng.random() < 0.2:
            sub = max(2, min(40, D // 5))          # subapertures that need not be whole pixels
        prec = rng.choice([P.FP32] * 5 + [P.FP16X3, P.BF16X3, P.FP16, P.BF16])
        c = _pwfs("", D=D, N=N, sub=sub, S=S, mod=rng.choice([1, 8, 15, 16, 24, 32, 48, 64, 96]),
                  r=rng.choice([2.0, 3.0, 5.0]), obs=rng.choice([0.0, 0.12, 0.28]), nl=rng.choice([1, 1, 1, 2, 3]),
                  prec=prec, flags=rng.choice([REF, REF, REF, 0, REF | LOCAL]))
        if prec == P.FP32:
            u = rng.random()
            if u < 0.12:
                c["flags"] |= ROOF
            elif u < 0.24:
                c["flags"] |= FULL
            elif u < 0.32:
                c["rings"], c["rho"], c["mod"] = 1, 1.0, min(c["mod"], 16)
            if rng.random() < 0.12:
                c["fov"] = 30.0
        per = _pwfs_flops(c, 1)
        c["frames"] = _log_int(rng, 1, max(1, min(1000, int(3e11 / per))))
    elif kind == "hetero":
        c = dict(kind=kind, frames=_log_int(rng, 1, 16))
    elif kind == "soul":
        photon = rng.random() < 0.8
        c = dict(kind=kind, frames=_log_int(rng, 1, 200), photon=photon, excess=photon and rng.random() < 0.5,
                 readout=rng.random() < 0.8)
    elif kind == "sh":
        b = rng.choice([4, 5, 7, 8, 10, 16])
        n = _log_int(rng, 4, 68 if b <= 8 else 30)
        rebin, px = rng.choice([(7, 8), (4, 8), (5, 10), (15, 16), (6, 6), (10, 12)])
        c = dict(kind=kind, D=n * b, n=n, M=rebin * px, rebin=rebin, obs=rng.choice([0.0, 0.12, 0.28]),
                 nl=rng.choice([1, 1, 1, 3]), frames=1, pixels=rng.random() < 0.5)
        c["frames"] = _log_int(rng, 1, max(1, min(1000, int(4e10 / _sh_flops(c)))))
    elif kind == "loop":
        c = dict(kind=kind, modes=_log_int(rng, 50, 600), layers=rng.randint(1, 6), screen=rng.choice([512, 1024]))
    elif kind in ("train", "predict"):
        c = dict(kind=kind, inputs=_log_int(rng, 50, 600), hidden=rng.choice([256, 512, 1000, 1024, 2048]),
                 outputs=rng.choice([512, 800, 2048, 3200]),
                 batch=32 * _log_int(rng, 1, 64) if kind == "train" else _log_int(rng, 1, 32768),
                 prec=rng.choice([P.BF16, P.BF16, P.BF16, P.BF16X3]))
    else:
        c = dict(kind=kind, m=_log_int(rng, 1, 3000), n=_log_int(rng, 64, 25600), k=_log_int(rng, 16, 1000),
                 prec=rng.choice([P.BF16X3, P.BF16X3, P.BF16]))
    c.pop("name", None)
    return c


# ---------------------------------------------------------------- sensors --
def _lambdas(nl):
    if nl == 1:
        return (750.0,), (1.0,)
    return tuple(600.0 + 300.0 * i / (nl - 1) for i in range(nl)), (1.0 / nl,) * nl


def _sensor(c):
    lams, w = _lambdas(c["nl"])
    return SimpleNamespace(n_pupil=c["D"], n_fft=c["N"], n_subap=c["sub"], n_mod=c["mod"],
                           pupil_sep_px=float(c["S"]), mod_radius_lod=c["r"], obstruction=c["obs"],
                           diameter_m=c.get("diameter", 8.0), lambda_ref_nm=750.0, lambdas_nm=lams,
                           lambda_weights=w, precision=c["prec"], flags=c["flags"], src_rings=c["rings"],
                           src_radius_lod=c["rho"], fov_lod=c["fov"])


def _hetero_cases():
    spec = [(80, 256, 2.0, 16), (120, 384, 3.0, 32), (160, 512, 3.0, 48), (160, 512, 4.0, 64), (240, 768, 5.0, 80),
            (240, 768, 5.0, 96)]
    return [_pwfs("", D=D, N=N, sub=D // 4, mod=m, S=int(1.2 * D), r=r, obs=0.28, nl=3, diameter=38.5)
            for D, N, r, m in spec]


def _soul_case():
    # 220 px, 40 x 40 subapertures of 5.5 px, 24 points at 3 lambda/D, 2 arcsec stop on 8.222 m at 750 nm
    fov = 2.0 / 206264.806 * 8.222 / 750e-9
    return _pwfs("", D=220, N=768, sub=40, mod=24, S=264, r=3.0, obs=0.0, fov=fov, diameter=8.222)


def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 17)


def _screens(frames, D, g, rms_nm=250.0):
    """Turbulence-like wavefronts [frames, D, D] float32 nm: a von Karman power spectrum on a 2D grid, cropped."""
    M = 2 * D
    f = torch.fft.fftfreq(M, device=DEV, dtype=torch.float64)
    f2 = f[:, None] ** 2 + f[None, :] ** 2
    amp = (f2 + (0.3 / M) ** 2) ** (-11.0 / 12.0)
    amp[0, 0] = 0.0
    amp = (amp * (M / amp.square().sum().sqrt())).float()
    out = torch.empty((frames, D, D), dtype=torch.float32, device=DEV)
    for i in range(0, frames, 128):
        n = min(128, frames - i)
        w = torch.randn((n, M, M, 2), generator=g, device=DEV)
        out[i:i + n] = torch.fft.ifft2(torch.view_as_complex(w) * amp).real[:, :D, :D] * (rms_nm * M)
    return out


# ---------------------------------------------------------------- prepare --
def prepare(case, seed):
    k, g = case["kind"], _generator(seed)
    if k == "pwfs":
        plan = P.Plan([_sensor(case)], max_frames=case["frames"])
        F = case["frames"]
        return dict(kind=k, plan=plan, opd=_screens(F, case["D"], g), I=plan.new_intensity(F),
                    s=plan.new_slopes(F), f=torch.zeros((F, 1), device=DEV))
    if k == "hetero":
        cs = _hetero_cases()
        F = case["frames"]
        plan = P.Plan([_sensor(c) for c in cs], max_frames=F)
        opd = torch.cat([_screens(F, c["D"], g).reshape(F, -1) for c in cs], dim=1).contiguous()
        return dict(kind=k, plan=plan, opd=opd, I=plan.new_intensity(F), s=plan.new_slopes(F),
                    f=torch.zeros((F, len(cs)), device=DEV))
    if k == "soul":
        c, F = _soul_case(), case["frames"]
        plan = P.Plan([_sensor(c)], max_frames=F)
        flags = (P.CCD_PHOTON * case["photon"] | P.CCD_EXCESS * case["excess"] | P.CCD_READOUT * case["readout"])
        from fractions import Fraction
        ccd = P.ccd_desc(120, Fraction(11, 2), 9.5e4, flags=int(flags), readout_e=0.4, seed=int(seed))
        return dict(kind=k, plan=plan, ccd=ccd, opd=_screens(F, c["D"], g), I=plan.new_intensity(F),
                    pix=torch.empty((F, 120, 120), device=DEV), s=plan.new_slopes(F), f=torch.zeros(F, device=DEV))
    if k == "sh":
        lams, w = _lambdas(case["nl"])
        d = P.sh_desc(case["D"], case["n"], case["M"], case["rebin"], case["obs"], lams[0],
                      lams if case["nl"] > 1 else None, w if case["nl"] > 1 else None)
        sh = P.SH(d, max_frames=case["frames"])
        F, n, px = case["frames"], case["n"], case["M"] // case["rebin"]
        return dict(kind=k, sh=sh, opd=_screens(F, case["D"], g), s=torch.empty((F, 2, n, n), device=DEV),
                    pix=torch.empty((F, n, n, px, px), device=DEV) if case["pixels"] else None)
    if k == "loop":
        i = _loop_inputs(case, g)
        loop = ClosedLoop(_sensor(_pwfs("")), i["B"].cpu().numpy(), i["screens"].cpu().numpy(), i["layers"],
                          i["gain"].cpu().numpy(), i["ff"].cpu().numpy(), 2, R=i["R"].cpu().numpy())
        loop.capture()
        loop.reset(i["t0"])
        loop.hist.copy_(i["hist"])
        loop.applied.copy_(i["applied"])
        return dict(kind=k, loop=loop)
    if k in ("train", "predict"):
        i = _net_inputs(case, g)
        mlp = P.MLP(_net_sizes(case), max_batch=32 * -(-case["batch"] // 32), precision=case["prec"])
        mlp.set_params(i["params"])
        if k == "train":
            mlp.set_state(i["moments"], 1000)     # a run that goes on from a checkpoint
            return dict(kind=k, mlp=mlp, x=i["x"], t=i["t"], grads=torch.empty(mlp.n_params, device=DEV))
        mlp.set_linear(i["C"])
        return dict(kind=k, mlp=mlp, x=i["x"], y=torch.empty((case["batch"], case["outputs"]), device=DEV))
    A, B = _gemm_inputs(case, g)
    return dict(kind=k, A=A, B=B, out=torch.empty((case["m"], case["n"]), device=DEV), prec=case["prec"])


def run(state):
    k = state["kind"]
    if k in ("pwfs", "hetero"):
        I, s, f = state["plan"].step(state["opd"], state["I"], state["s"], state["f"])
        return dict(intensity=I, slopes=s, flux=f)
    if k == "soul":
        plan = state["plan"]
        I = plan.forward(state["opd"], state["I"])
        pix = plan.ccd(I, state["ccd"], 0, state["pix"])
        s, f = plan.ccd_slopes(pix, state["ccd"], state["s"], state["f"])
        return dict(intensity=I, pixels=pix, slopes=s, flux=f)
    if k == "sh":
        s, pix = state["sh"].forward(state["opd"], state["s"], state["pix"])
        return dict(slopes=s, pixels=pix)
    if k == "loop":
        loop = state["loop"]
        loop.run(1)
        return dict(opd=loop.opd, slopes=loop.slopes, modes=loop.modes, applied=loop.applied)
    if k == "train":
        mlp = state["mlp"]
        loss = mlp.grad(state["x"], state["t"], 1.0, state["grads"])
        mlp.adam(1e-4)
        return dict(loss=loss, grads=state["grads"])
    if k == "predict":
        return state["mlp"].forward(state["x"], state["y"], _OUT_SCALE)
    return P.gemm(state["A"], state["B"], state["out"], precision=state["prec"])


# ------------------------------------------------------- inputs of a kind --
_OUT_SCALE = 0.05


def _net_sizes(case):
    return [case["inputs"], case["hidden"], case["hidden"], case["outputs"]]


def _net_inputs(case, g):
    sizes, B = _net_sizes(case), case["batch"]
    parts, C = [], None
    for i, o in zip(sizes[:-1], sizes[1:]):
        parts += [torch.randn(o * i, generator=g, device=DEV) / math.sqrt(i),
                  0.01 * torch.randn(o, generator=g, device=DEV)]
    params = torch.cat(parts)
    x = torch.randn((B, sizes[0]), generator=g, device=DEV)
    out = dict(params=params, x=x)
    if case["kind"] == "train":
        out["t"] = torch.randn((B, sizes[-1]), generator=g, device=DEV)
        m = 1e-4 * torch.randn(params.numel(), generator=g, device=DEV)
        out["moments"] = torch.cat([m, torch.full_like(m, 1e-6)])
    else:
        out["C"] = torch.randn((sizes[-1], sizes[0]), generator=g, device=DEV) * 0.005
    return out


def _gemm_inputs(case, g):
    A = torch.randn((case["m"], case["k"]), generator=g, device=DEV)
    decay = 100.0 / torch.arange(1, case["k"] + 1, device=DEV) ** 0.9      # wavefront modes of falling strength
    return A, (torch.randn((case["n"], case["k"]), generator=g, device=DEV) * decay).contiguous()


def _loop_inputs(case, g):
    D, n, L, px = 160, case["modes"], case["layers"], case["screen"]
    y = (torch.arange(D, device=DEV, dtype=torch.float32) + 0.5) / D
    fx = torch.randint(0, 12, (n,), generator=g, device=DEV)
    fy = torch.randint(0, 12, (n,), generator=g, device=DEV)
    cx, cy = torch.cos(math.pi * y[:, None] * fx), torch.cos(math.pi * y[:, None] * fy)
    B = (cy[:, None, :] * cx[None, :, :]).reshape(D * D, n).contiguous()
    layers = [(1.0 / math.sqrt(L), 37.0 * i + 0.25, 111.0 * i + 0.5, 0.05 + 0.1 * i, 0.02 * i) for i in range(L)]
    rnd = lambda *s: torch.randn(s, generator=g, device=DEV)                # noqa: E731
    return dict(B=B, layers=layers, screens=_screens(L, px, g), R=rnd(n, 3200), gain=torch.full((n,), 0.45, device=DEV),
                ff=torch.full((n,), 0.9994, device=DEV), t0=101, hist=rnd(3, n), applied=rnd(n))


# ------------------------------------------------------------------- work --
def _fft(N):
    return 5.0 * N * math.log2(N)


def _tilts(c):
    points = c["mod"] * (1 + 3 * c["rings"] * (c["rings"] + 1))
    keys = (c["mod"] // 2 + 1) * (1 + 3 * c["rings"] * (c["rings"] + 1))
    return points, keys


def _pwfs_flops(c, frames):
    """A transform pair per (row, distinct x-tilt) and per (kept column, point), and the |e|^2 sums."""
    points, keys = _tilts(c)
    Nc = c["N"] if c["flags"] & FULL else 2 * c["D"]
    pair = 2 * _fft(c["N"])
    arms = 0.5 if c["flags"] & ROOF else 1.0
    return frames * c["nl"] * (arms * (keys * c["D"] + points * Nc) * pair + 3.0 * points * Nc * Nc)


def _pwfs_bytes(c, frames):
    Nc = c["N"] if c["flags"] & FULL else 2 * c["D"]
    planes = 2 if c["flags"] & ROOF else 1
    return frames * 4.0 * (c["D"] ** 2 + planes * Nc * (Nc if planes == 1 else c["D"]) + 2 * c["sub"] ** 2)


def _sh_flops(c):
    b = c["D"] // c["n"]
    return c["nl"] * 0.78 * c["n"] ** 2 * (8.0 * b * c["M"] * (b + c["M"]) + 3.0 * c["M"] ** 2)


def work(case):
    k = case["kind"]
    if k == "pwfs":
        return dict(bytes=_pwfs_bytes(case, case["frames"]), flops=_pwfs_flops(case, case["frames"]))
    if k == "hetero":
        cs = _hetero_cases()
        return dict(bytes=sum(_pwfs_bytes(c, case["frames"]) for c in cs),
                    flops=sum(_pwfs_flops(c, case["frames"]) for c in cs))
    if k == "soul":
        c, F = _soul_case(), case["frames"]
        return dict(bytes=_pwfs_bytes(c, F) + F * 4.0 * 120 * 120, flops=_pwfs_flops(c, F))
    if k == "sh":
        F, px = case["frames"], case["M"] // case["rebin"]
        out = 2 * case["n"] ** 2 + (case["n"] ** 2 * px * px if case["pixels"] else 0)
        return dict(bytes=F * 4.0 * (case["D"] ** 2 + out), flops=F * _sh_flops(case))
    if k == "loop":
        c = _pwfs("")
        return dict(bytes=4.0 * (160 * 160 * (case["modes"] + case["layers"] + 1) + 3200 * case["modes"]),
                    flops=_pwfs_flops(c, 1) + 2.0 * case["modes"] * (25600 + 3200))
    if k in ("train", "predict"):
        s, B = _net_sizes(case), case["batch"]
        w = sum(a * b + b for a, b in zip(s[:-1], s[1:]))
        if k == "train":      # weights and two moments read and written, gradients written
            return dict(bytes=4.0 * (7 * w + B * (s[0] + s[-1])), flops=6.0 * w * B - 2.0 * s[0] * s[1] * B)
        w += s[0] * s[-1]
        return dict(bytes=4.0 * (w + B * (s[0] + s[-1])), flops=2.0 * w * B)
    m, n, kk = case["m"], case["n"], case["k"]
    return dict(bytes=4.0 * (m * kk + n * kk + m * n), flops=2.0 * m * n * kk)


# ------------------------------------------------------------------ exact --
def _centred(n):
    return torch.arange(n, dtype=torch.float64, device=DEV) - (n - 1) / 2.0


def _pupil(D, obs):
    r2 = _centred(D)[:, None] ** 2 + _centred(D)[None, :] ** 2
    return ((r2 <= (D / 2.0) ** 2) & (r2 >= (obs * D / 2.0) ** 2)).double()


def _cis(a):
    return torch.polar(torch.ones_like(a), a)


def _axis_operator(c, lam, sep, rows):
    """One axis of pad, half-pixel tilt, DFT, mask (faces `sep` apart, field stop), inverse DFT, at output `rows`."""
    N, D = c["N"], c["D"]
    j = torch.arange(N, dtype=torch.float64, device=DEV)
    ub = torch.where(j < N // 2, j + 0.5, j - N + 0.5)
    mask = _cis(math.pi * sep * ub.abs() / N)
    if c["fov"] > 0.0:
        side = ((c["fov"] * (750.0 / lam)) * N) / D
        mask = mask * (2.0 * ub.abs() <= side).double()
    o = (N - D) // 2
    x = torch.arange(o, o + D, dtype=torch.float64, device=DEV)
    fwd = _cis(-TWO_PI * torch.remainder(j[:, None] * x[None, :], N) / N) * _cis(-math.pi * x / N)[None, :]
    y = torch.as_tensor(rows, dtype=torch.float64, device=DEV)
    inv = _cis(TWO_PI * torch.remainder(y[:, None] * j[None, :], N) / N) / N
    return (inv * mask[None, :]) @ fwd                                       # [rows, D]


def _points(c):
    src = [(0.0, 0.0)]
    for q in range(1, c["rings"] + 1):
        for j in range(6 * q):
            a = TWO_PI * j / (6 * q)
            src.append((c["rho"] * q / c["rings"] * math.cos(a), c["rho"] * q / c["rings"] * math.sin(a)))
    return [(c["r"] * math.cos(TWO_PI * k / c["mod"]) + dx, c["r"] * math.sin(TWO_PI * k / c["mod"]) + dy)
            for k in range(c["mod"]) for dx, dy in src]


def _plane(c, opd, sep_x, sep_y, share):
    """Normalised intensity [F, N, N] of one set of faces, only its image windows unless the full plane is kept."""
    D, N = c["D"], c["N"]
    F = opd.shape[0]
    A = _pupil(D, c["obs"])
    pts = _points(c)

    def kept(sep):
        if c["flags"] & FULL:
            return list(range(N))
        starts = sorted({N // 2 + s * sep // 2 - D // 2 for s in (-1, 1)})
        return [o + i for o in starts for i in range(D)]

    X, Y = kept(sep_x), kept(sep_y)
    acc = torch.zeros((F, len(Y), len(X)), dtype=torch.float64, device=DEV)
    xc = _centred(D)
    for lam, w in zip(*_lambdas(c["nl"])):
        Px, Py = _axis_operator(c, lam, sep_x, X), _axis_operator(c, lam, sep_y, Y)
        sc = 750.0 / lam
        tx = torch.tensor([p[0] for p in pts], dtype=torch.float64, device=DEV)
        ty = torch.tensor([p[1] for p in pts], dtype=torch.float64, device=DEV)
        rx = _cis(TWO_PI * sc / D * tx[:, None] * xc[None, :])               # [points, D]
        ry = _cis(TWO_PI * sc / D * ty[:, None] * xc[None, :])
        step = max(1, int(3e8 / (16.0 * len(X) * max(D, len(Y)))))
        for f in range(F):
            E0 = A * _cis(TWO_PI / lam * opd[f].double())
            for k0 in range(0, len(pts), step):
                Ek = E0[None] * rx[k0:k0 + step, None, :] * ry[k0:k0 + step, :, None]
                n = Ek.shape[0]
                T = (Ek.reshape(n * D, D) @ Px.T).reshape(n, D, len(X)).transpose(1, 2).reshape(n * len(X), D)
                e = torch.view_as_real(T @ Py.T).square().sum(-1).reshape(n, len(X), len(Y)).sum(0)
                acc[f] += e.T * (w * share / len(pts))
    acc /= A.square().sum()
    out = torch.zeros((F, N, N), dtype=torch.float64, device=DEV)
    out[:, torch.tensor(Y, device=DEV)[:, None], torch.tensor(X, device=DEV)[None, :]] = acc
    return out


def _valid(c):
    W = _overlap(c["D"], c["sub"])
    return 2.0 * (W @ _pupil(c["D"], c["obs"]) @ W.T) >= float(c["D"]) ** 2


def _overlap(D, n):
    """Length of pixel y's overlap with subaperture i in units of 1/n pixel, [n, D]."""
    i = torch.arange(n, dtype=torch.float64, device=DEV)[:, None] * D
    y = torch.arange(D, dtype=torch.float64, device=DEV)[None, :] * n
    return (torch.minimum(y + n, i + D) - torch.maximum(y, i)).clamp(min=0.0)


def _raw_slopes(c, I):
    N, D, S = c["N"], c["D"], c["S"]
    lo, hi, mid = N // 2 - S // 2 - D // 2, N // 2 + S // 2 - D // 2, N // 2 - D // 2
    W = _overlap(D, c["sub"]) / c["sub"]
    v = _valid(c)

    def image(plane, r, col):
        return W @ plane[:, r:r + D, col:col + D] @ W.T

    if c["flags"] & ROOF:
        a, b = image(I[:, 0], mid, lo), image(I[:, 0], mid, hi)
        d, e = image(I[:, 1], lo, mid), image(I[:, 1], hi, mid)
        tx, ty, dx, dy = a + b, d + e, a - b, d - e
    else:
        q = [image(I, r, col) for r in (lo, hi) for col in (lo, hi)]
        tx = ty = q[0] + q[1] + q[2] + q[3]
        dx, dy = (q[0] + q[2]) - (q[1] + q[3]), (q[0] + q[1]) - (q[2] + q[3])
    total = tx + ty if c["flags"] & ROOF else tx
    flux = total[:, v].sum(1)
    if not c["flags"] & LOCAL:
        tx, ty = (t[:, v].mean(1)[:, None, None] for t in (tx, ty))
    s = torch.stack([dx / tx, dy / ty], 1)
    return torch.where(v[None, None], s, torch.zeros_like(s)), flux


def _sensor_exact(c, opd):
    def planes(o):
        if c["flags"] & ROOF:
            return torch.stack([_plane(c, o, c["S"], 0, 0.5), _plane(c, o, 0, c["S"], 0.5)], 1)
        return _plane(c, o, c["S"], c["S"], 1.0)

    I = planes(opd)
    s, flux = _raw_slopes(c, I)
    if c["flags"] & REF:
        s = s - _raw_slopes(c, planes(torch.zeros_like(opd[:1])))[0]
    return I, s, flux


def _exact_sh(case, opd):
    D, n, M, r = case["D"], case["n"], case["M"], case["rebin"]
    b, px, F = D // n, M // r, opd.shape[0]
    A = _pupil(D, case["obs"])
    lit = A.reshape(n, b, n, b).sum((1, 3))
    valid = 2.0 * lit >= b * b
    u = torch.arange(M, dtype=torch.float64, device=DEV) - M / 2.0 + 0.5
    lams, w = _lambdas(case["nl"])
    pix = torch.zeros((F, n, n, px, px), dtype=torch.float64, device=DEV)
    for f in range(F):
        for lam, wl in zip(lams, w):
            sc = lams[0] / lam
            W = _cis(-TWO_PI / M * sc * u[:, None] * _centred(b)[None, :])   # [M, b]
            E = (A * _cis(TWO_PI / lam * opd[f].double())).reshape(n, b, n, b).transpose(1, 2).reshape(-1, b, b)
            for i in range(0, n * n, 512):
                e = E[i:i + 512]
                k = e.shape[0]
                T = (e.reshape(-1, b) @ W.T).reshape(k, b, M).transpose(1, 2).reshape(-1, b)     # [k M(u), b(y)]
                G = torch.view_as_real(T @ W.T).square().sum(-1).reshape(k, M, M)                # [k, u, v]
                G = G.reshape(k, px, r, px, r).sum((2, 4)).transpose(1, 2)
                pix[f].view(-1, px, px)[i:i + 512] += G * (wl * sc * sc / (M * M * A.sum()))
    pix = torch.where(valid[None, :, :, None, None], pix, torch.zeros_like(pix))
    t = pix.sum((3, 4))
    x = _centred(px)
    t = torch.where(t > 0, t, torch.ones_like(t))
    s = torch.stack([(pix * x[None, None, None, None, :]).sum((3, 4)) / t,
                     (pix * x[None, None, None, :, None]).sum((3, 4)) / t], 1)
    return dict(slopes=s, pixels=pix if case["pixels"] else None)


def _exact_net(case, i):
    sizes, p, at = _net_sizes(case), i["params"].double(), 0
    layers = []
    for a, b in zip(sizes[:-1], sizes[1:]):
        layers.append((p[at:at + a * b].reshape(b, a).clone(), p[at + a * b:at + a * b + b].clone()))
        at += a * b + b
    train = case["kind"] == "train"
    flat = [t.requires_grad_(train) for layer in layers for t in layer]
    h = i["x"].double()
    for k, (W, b) in enumerate(layers):
        h = h @ W.T + b
        if k + 1 < len(layers):
            h = 0.5 * h * (1.0 + torch.erf(h / math.sqrt(2.0)))
    if not train:
        return _OUT_SCALE * h + i["x"].double() @ i["C"].double().T
    loss = (h - i["t"].double()).square().mean()
    grads = torch.autograd.grad(loss, flat)
    return dict(loss=loss.detach().reshape(1), grads=torch.cat([q.reshape(-1) for q in grads]))


def _exact_loop(case, i):
    c, D, t = _pwfs(""), 160, float(i["t0"])
    px = case["screen"]
    x = torch.arange(D, dtype=torch.float64, device=DEV)
    opd = torch.zeros((D, D), dtype=torch.float64, device=DEV)
    for S, (w, ox, oy, vx, vy) in zip(i["screens"].double(), i["layers"]):
        X, Y = x + ox + vx * t, x + oy + vy * t
        fx, fy = X - X.floor(), Y - Y.floor()
        i0, j0 = torch.remainder(X.floor(), px).long(), torch.remainder(Y.floor(), px).long()
        rows = (1.0 - fy)[:, None] * S[j0] + fy[:, None] * S[(j0 + 1) % px]
        opd += w * ((1.0 - fx) * rows[:, i0] + fx * rows[:, (i0 + 1) % px])
    opd -= (i["B"].double() @ i["applied"].double()).reshape(D, D)
    _, s, _ = _sensor_exact(c, opd[None])
    m = i["R"].double() @ s.reshape(-1)
    slots = i["hist"].double()
    # c(t) goes to slot t mod 3; the mirror next applies c(t - 1) (total delay of two steps)
    applied = slots[(int(t) - 1) % 3]
    return dict(opd=opd, slopes=s, modes=m, applied=applied)


def exact(case, seed):
    k, g = case["kind"], _generator(seed)
    if k == "pwfs":
        I, s, f = _sensor_exact(case, _screens(case["frames"], case["D"], g))
        return dict(intensity=I, slopes=s, flux=f[:, None])
    if k == "hetero":
        cs, F = _hetero_cases(), case["frames"]
        parts = [_sensor_exact(c, o) for c, o in zip(cs, [_screens(F, c["D"], g) for c in cs])]
        return dict(intensity=torch.cat([p[0].reshape(F, -1) for p in parts], 1),
                    slopes=torch.cat([p[1].reshape(F, -1) for p in parts], 1),
                    flux=torch.stack([p[2] for p in parts], 1))
    if k == "soul":
        I, _, _ = _sensor_exact(_soul_case(), _screens(case["frames"], 220, g))
        return dict(intensity=I, pixels=None, slopes=None, flux=None)      # the detector's noise is drawn
    if k == "sh":
        return _exact_sh(case, _screens(case["frames"], case["D"], g))
    if k == "loop":
        return _exact_loop(case, _loop_inputs(case, g))
    if k in ("train", "predict"):
        return _exact_net(case, _net_inputs(case, g))
    A, B = _gemm_inputs(case, g)
    return A.double() @ B.double().T
