"""The work that a program using this framework has it do, as cases that can be
timed and checked: one call (or one step of a loop) each, through the public
entry points of paper_2604_07248_amd.

    listed()            the named cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) what a program holds before the call: plan, source, masks
    run(state)          one pass, with its outputs whole
    work(case)          bytes and operations the pass cannot do without
    exact(case, seed)   the outputs of prepare + run in 64 bits, in plain torch

Every case is a path geometry (grid, wavelength, distances, turbulence) and a
kind of use:
    forward   a batch of realizations through fresh screens (Plan.propagate)
    adjoint   the same with checkpoints, and the gradients back
    given     screens generated once, looked at, and propagated through by
              autograd with gradients to the sources and to the screens
    ar        one time step of an autoregressive sequence
    serving   an uneven batch of requests in one call (Batch), with or without
              gradients
    train     forward and backward of a training step of the two-mask receiver
    stats     ensemble moments of received fields and their summary
"""

import math
import random

import torch

from paper_2604_07248_amd import api, binding, d2nn, workloads

WAVELENGTHS = (532e-9, 1064e-9, 1550e-9)


def _case(name, kind, n, side, wavelength, length, m, cn2, r, **more):
    c = {"kind": kind, "n": n, "side": side, "wavelength": wavelength, "length": length, "m": m, "cn2": cn2,
         "l0": 0.005, "L0": 20.0, "sh": 0, "angular": False, "r": r, "source": "gaussian", "w0": side / 16}
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the first thing a new user runs: the plain forward workload, 16
        # realizations on a small grid, where launches and latency count
        _case("example_128", "forward", 128, 0.5, 1550e-9, 1000.0, 5, 1e-14, 16, l0=0.01, L0=10.0, w0=0.02),
        # one beam at a time, as an interactive program or a request handler
        # asks for it: a single realization with subharmonics
        _case("one_beam_256", "forward", 256, 0.5, 1064e-9, 1200.0, 10, 3e-15, 1, sh=3, w0=0.04),
        # one batch of a point of the weak-to-strong sweep: tapered plane wave,
        # subharmonics, moments taken inside the pass
        _case("sweep_512", "forward", 512, 1.0, 1550e-9, 2000.0, 10, 1e-15, 256, sh=3, source="flat_top",
              moments=True),
        # the headline propagation workload: 64 realizations x 8 fresh screens
        _case("headline_1024", "forward", 1024, 1.0, 1064e-9, 1500.0, 8, 2e-14, 64, w0=0.05, moments=True),
        # a few fields on the largest grid, angular spectrum, an odd count
        _case("angular_2048", "forward", 2048, 1.6, 1064e-9, 4000.0, 12, 1e-15, 3, angular=True, sh=3, w0=0.1),
        # end-to-end gradients of the headline workload: dL/du of the shared
        # source and dL/dphi of every screen
        _case("adjoint_1024", "adjoint", 1024, 1.0, 1064e-9, 1500.0, 8, 2e-14, 64, w0=0.05),
        # screens made once and held by the caller, gradients to fields and
        # screens through autograd; a ragged count on a small grid
        _case("given_256", "given", 256, 0.5, 1550e-9, 900.0, 6, 5e-15, 5, w0=0.03),
        # one time step of the autoregressive workload, 32 sequences
        _case("ar_1024", "ar", 1024, 1.0, 1064e-9, 1500.0, 8, 2e-14, 32, w0=0.05, alpha=0.99, shift_x=0.5,
              shift_y=0.0),
        # a wave of the serving mix (uneven grids, screen counts, wavelengths)
        {"name": "serving_96", "kind": "serving", "count": 96, "grad": False, "mix": 5},
        # requests that ask for gradients too
        {"name": "serving_grad_24", "kind": "serving", "count": 24, "grad": True, "mix": 7},
        # a step of training the receiver's masks through turbulence
        _case("train_512", "train", 512, 1.0, 1550e-9, 1000.0, 6, 5e-15, 64, w0=0.02),
        # the end of an ensemble: the last batch joins the moments, then the
        # scintillation map, the power-cutoff region and the beam radii
        _case("stats_1024", "stats", 1024, 1.0, 1064e-9, 1500.0, 0, 0.0, 64, w0=0.12, power=0.999),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the ranges above: grids 128..2048, 1..20 screens, counts from
    one realization to what the listed cases hold, both transfer functions, 0
    to 3 subharmonic levels."""
    kind = rng.choice(["forward", "forward", "forward", "adjoint", "adjoint", "given", "ar", "ar", "serving", "train",
                       "stats"])
    if kind == "serving":
        grad = rng.random() < 0.5
        return {"kind": kind, "count": _log(rng, 3, 24 if grad else 96), "grad": grad, "mix": rng.randrange(1000)}
    n = rng.choice([256, 512, 1024] if kind == "train" else [128, 256, 512, 1024, 2048])
    if kind == "stats":
        r = _log(rng, 4, min(512, 64 * 2 ** 20 // n ** 2))
        side = rng.uniform(0.5, 1.5)
        return _case("", kind, n, side, rng.choice(WAVELENGTHS), 1000.0, 0, 0.0, r, w0=side * rng.uniform(0.08, 0.15),
                     power=rng.choice([0.0, 0.9, 0.999]))
    m = rng.randint(1, 20)
    most = 2 ** 29 if kind in ("forward", "ar") else 2 ** 28  # R N^2 M
    if kind == "train":
        m = rng.randint(2, 8)
    r = _log(rng, 1, max(1, min(256, most // (m * n * n))))
    wavelength = rng.choice(WAVELENGTHS)
    length = rng.uniform(500.0, 4000.0)
    dx = math.sqrt(2 * wavelength * (length / m) / n)  # twice the sampling limit of a step
    side = n * dx
    c = _case("", kind, n, side, wavelength, length, m, 10.0 ** rng.uniform(-16, -14), r, sh=rng.choice([0, 0, 3, 2]),
              w0=side * rng.uniform(0.05, 0.12))
    if kind in ("forward", "adjoint"):
        c["angular"] = rng.random() < 0.25
    if kind == "forward":
        c["moments"] = rng.random() < 0.5
        c["source"] = rng.choice(["gaussian", "flat_top", "own"])
    if kind == "ar":
        c.update(alpha=rng.choice([0.9, 0.99, 0.999]), shift_x=rng.uniform(-1, 1), shift_y=rng.uniform(-1, 1))
    if kind == "train":
        c["r"] = max(2, c["r"])
    return c


# -- inputs -------------------------------------------------------------------

def _geometry(c):
    """dx, the distances (screens in the middle of M equal steps) and the
    integrated strength of each step."""
    m, step = c["m"], c["length"] / max(1, c["m"])
    dz = (0.5 * step,) + (step,) * (m - 1) + (0.5 * step,) if m else (c["length"],)
    return c["side"] / c["n"], dz, (c["cn2"] * step,) * m


def _path(c):
    dx, dz, cn2dz = _geometry(c)
    return workloads.Path(n=c["n"], dx=dx, wavelength=c["wavelength"], dz=dz, cn2dz=cn2dz, l0=c["l0"], L0=c["L0"],
                          sh_levels=c["sh"], tf_kind=workloads.TF_ANGULAR_SPECTRUM if c["angular"] else
                          workloads.TF_FRESNEL, realizations=c["r"])


def _mix(c):
    """The requests of a serving case: the mix's sizes, distances and strengths
    (grids 256..2048, 5 to 20 screens, dx at the sampling limit)."""
    rng, out = random.Random(c["mix"]), []
    for _ in range(c["count"]):
        n, wavelength = rng.choice([256, 512, 1024, 2048]), rng.choice(WAVELENGTHS)
        m, cn2, length = rng.randint(5, 20), 10.0 ** rng.uniform(-16, -13), rng.uniform(500.0, 5000.0)
        side = n * math.sqrt(2 * wavelength * (length / m) / n)
        out.append(_case("", "forward", n, side, wavelength, length, m, cn2, 1, sh=3, w0=side / 8))
    return out


def _grid(n, dx, device="cuda"):
    return (torch.arange(n, dtype=torch.float64, device=device) - n // 2) * dx


def _source(c, seed, count=0):
    """The source field(s): a Gaussian beam or a tapered plane wave, its centre,
    width and tilt a little different with each seed; count > 0: one per
    realization."""
    rng = random.Random(1000003 * seed + 17)
    x = _grid(c["n"], c["side"] / c["n"])
    out = []
    for _ in range(max(1, count)):
        cx, cy = (rng.uniform(-0.03, 0.03) * c["side"] for _ in range(2))
        r2 = (x[None, :] - cx) ** 2 + (x[:, None] - cy) ** 2
        w = rng.uniform(0.95, 1.05)
        if c["source"] == "flat_top":
            amp = torch.exp(-(r2 / (0.4 * w * c["side"]) ** 2) ** 10)
        else:
            amp = torch.exp(-r2 / (w * c["w0"]) ** 2)
        tilt = [rng.uniform(-3, 3) / c["side"] for _ in range(2)]
        ph = 2 * math.pi * (tilt[0] * x[None, :] + tilt[1] * x[:, None])
        out.append(torch.polar(amp, ph).to(torch.complex64))
    return torch.stack(out) if count else out[0]


def _random(shape, seed, dtype=torch.complex64):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda", dtype=dtype)


def _cotangent(c, seed, shape=None):
    """dL/du_out of a loss over the received intensity's neighbourhood."""
    n = c["n"]
    x = _grid(n, c["side"] / n)
    bump = torch.exp(-(x[None, :] ** 2 + x[:, None] ** 2) / (0.25 * c["side"]) ** 2).to(torch.float32)
    return _random(shape or (c["r"], n, n), 7919 * seed + 3) * bump


def _masks(n, seed):
    """Two phase masks as they are part of the way through training: smooth."""
    out = []
    for k in range(2):
        coarse = _random((1, 1, n // 16, n // 16), 31 * seed + k, torch.float32)
        out.append(torch.nn.functional.interpolate(coarse, size=(n, n), mode="bilinear")[0, 0].contiguous())
    return out


def _received(c, seed):
    """Fields as they arrive at the end of a turbulent path: a Gaussian envelope
    under smooth log-normal amplitude and phase fluctuations, and a faint
    speckle of light scattered wide over the whole grid."""
    n, r = c["n"], c["r"]
    x = _grid(n, c["side"] / n)
    env = torch.exp(-(x[None, :] ** 2 + x[:, None] ** 2) / c["w0"] ** 2).to(torch.float32)
    u = torch.empty((r, n, n), dtype=torch.complex64, device="cuda")
    for i in range(0, r, 16):
        k = min(16, r - i)
        f = torch.nn.functional.interpolate(_random((k, 2, n // 16, n // 16), 101 * seed + i, torch.float32),
                                            size=(n, n), mode="bicubic")
        u[i:i + k] = torch.polar(env * torch.exp(0.3 * f[:, 0]), 2.0 * f[:, 1])
        u[i:i + k] += 1e-3 * _random((k, n, n), 211 * seed + i)
    return u


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = {"case": c, "seed": seed, "t": 0}
    if kind == "serving":
        mix = _mix(c)
        s["batch"] = api.Batch([_path(p) for p in mix])
        s["u"] = torch.cat([_source(p, seed + i).reshape(-1) for i, p in enumerate(mix)])
        if c["grad"]:
            s["g"] = torch.cat([_cotangent(p, seed + i).reshape(-1) for i, p in enumerate(mix)])
        return s
    if kind == "stats":
        s["moments"] = api.Moments(c["n"], c["side"] / c["n"])
        s["u"] = _received(c, seed)
        x = _grid(c["n"], c["side"] / c["n"])
        s["weight"] = ((x[None, :] ** 2 + x[:, None] ** 2) <= (0.4 * c["side"]) ** 2).to(torch.float32)
        return s
    if kind == "train":
        w = workloads.Workload("train", _path(c), seed=seed, source="gaussian", w0=c["w0"])
        s["trainer"] = d2nn.D2NNTrainer(w, diameter=0.3 * c["side"])
        with torch.no_grad():
            for theta, value in zip((s["trainer"].theta1, s["trainer"].theta2), _masks(c["n"], seed)):
                theta.copy_(value)
        return s
    s["plan"] = api.Plan(_path(c), flags=binding.SCREEN_CHECKPOINTS if kind == "adjoint" else 0)
    s["u"] = _source(c, seed, c["r"] if kind == "given" or c["source"] == "own" else 0)
    if c.get("moments"):
        s["moments"] = api.Moments(c["n"], c["side"] / c["n"])
        s["plan"].bind_moments(s["moments"])
    if kind in ("adjoint", "given"):
        s["g"] = _cotangent(c, seed)
    if kind == "ar":
        s["state"] = s["plan"].init_spectra(seed)
        s["t"] = 1
    return s


def run(state):
    s = state
    c, kind, seed, t = s["case"], s["case"]["kind"], s["seed"], s["t"]
    s["t"] = t + 1  # fresh screens at every call
    if kind == "forward":
        u = s["plan"].propagate(s["u"], seed=seed, t=t)
        return {"u": u, "moments": s["moments"].buf} if c.get("moments") else {"u": u}
    if kind == "adjoint":
        u, ck = s["plan"].propagate(s["u"], seed=seed, t=t, checkpoints=True)
        g_in, g_phi = s["plan"].propagate_backward(s["g"], ck, seed=seed, t=t, shared_source=True)
        return {"u": u, "g_in": g_in, "g_phi": g_phi}
    if kind == "given":
        phi = s["plan"].screens(seed, t).requires_grad_()
        u_in = s["u"].detach().requires_grad_()
        u = api.Propagate.apply(u_in, phi, s["plan"], seed, t)
        g_in, g_phi = torch.autograd.grad(u, [u_in, phi], grad_outputs=s["g"])
        return {"screens": phi.detach(), "u": u.detach(), "g_in": g_in, "g_phi": g_phi}
    if kind == "ar":
        u = s["plan"].evolve_propagate(s["state"], seed, t, c["alpha"], c["shift_x"], c["shift_y"], u_in=s["u"])
        return {"u": u, "state": s["state"]}
    if kind == "serving":
        if not c["grad"]:
            return {"u": s["batch"].propagate(s["u"], seed=seed, t=t)}
        u, ck = s["batch"].propagate(s["u"], seed=seed, t=t, checkpoints=True)
        g_in, g_phi = s["batch"].propagate_backward(s["g"], ck, seed=seed, t=t)
        return {"u": u, "g_in": g_in, "g_phi": g_phi}
    if kind == "train":
        # the step without the optimizer, whose sign-like update would carry
        # the rounding of the smallest gradients into the next step's masks
        tr = s["trainer"]
        u = tr.forward(t)
        loss = d2nn.loss_fn(u, tr.i_vac, tr.aperture)
        g1, g2 = torch.autograd.grad(loss, [tr.theta1, tr.theta2])
        return {"loss": loss.detach(), "g1": g1, "g2": g2, "u": u.detach()}
    if kind == "stats":
        s["moments"].add(s["u"])
        si, summary = s["moments"].finalize(weight=s["weight"], power_fraction=c["power"])
        return {"si": si, "summary": summary, "moments": s["moments"].buf}
    raise ValueError(kind)


# -- work ---------------------------------------------------------------------

def work(case):
    c, kind = case, case["kind"]
    if kind == "serving":
        parts = [work(dict(p, kind="served", grad=c["grad"])) for p in _mix(c)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    n, m, r = c["n"], c["m"], c["r"]
    px = n * n
    fft = 10.0 * px * math.log2(n)  # one 2-D transform of one plane
    if kind == "stats":  # fields in, moments in and out, the map out
        return {"bytes": 8 * r * px + 2 * 16 * px + 4 * px, "flops": 8.0 * r * px}
    screens = 0.5 * r * m * (fft + 60 * px)  # one synthesis for two realizations
    steps = r * (m + 1) * (2 * fft + 6 * px) + 10.0 * r * m * px
    own = c["source"] == "own" or kind in ("given", "served")
    nbytes = 8 * px * (r if own else 1) + 8 * r * px  # sources in, fields out
    flops = screens + steps
    if c.get("moments"):
        nbytes += 2 * 16 * px
    if kind in ("adjoint", "given") or c.get("grad"):  # cotangents in, both gradients out
        nbytes += 8 * r * px + 8 * px * (r if own else 1) + 4 * r * m * px
        flops += steps
    if kind == "given":
        nbytes += 4 * r * m * px  # the screens themselves
    if kind == "ar":  # the state in and out
        nbytes += 2 * 8 * ((r + 1) // 2) * m * px
    if kind == "train":  # masks, their gradients, the vacuum beam, the aperture
        nbytes += 6 * 4 * px
        flops += r * (5 * fft + 60 * px)
    return {"bytes": nbytes, "flops": flops}


# -- the same in 64 bits ------------------------------------------------------

_OFFSETS = [(a, b) for a in (-1, 0, 1) for b in (-1, 0, 1) if (a, b) != (0, 0)]
_LO = 0xFFFFFFFF


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 over int64 tensors holding 32-bit words (products wrap
    modulo 2^64; the masks keep each half)."""
    c0, c1, c2, c3 = torch.broadcast_tensors(c0, c1, c2, c3)
    k0, k1 = seed & _LO, (seed >> 32) & _LO
    for i in range(10):
        if i:
            k0, k1 = (k0 + 0x9E3779B9) & _LO, (k1 + 0xBB67AE85) & _LO
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = (((p1 >> 32) & _LO) ^ c1 ^ k0, p1 & _LO, ((p0 >> 32) & _LO) ^ c3 ^ k1, p0 & _LO)
    return c0, c1, c2, c3


def _normal(va, vb):
    ua, ub = (((v >> 9).double() + 0.5) * 2.0 ** -23 for v in (va, vb))
    return torch.polar(torch.sqrt(-2 * torch.log(ua)), 2 * math.pi * ub)


def _word(v):
    return torch.as_tensor(v, dtype=torch.int64, device="cuda")


def _spectral_noise(n, seed, t, pairs, tag, screen):
    """[pairs][n][n] unit normals, bins (k0, k1) and (k0 + n/2, k1) of a block."""
    e = torch.arange(n // 2 * n, dtype=torch.int64, device="cuda")
    v = _philox(e[None, :], _word(t), pairs[:, None], _word((tag << 28) | screen), seed)
    return torch.cat([_normal(v[0], v[1]), _normal(v[2], v[3])], 1).view(len(pairs), n, n)


def _bins(n):
    k = torch.arange(n, dtype=torch.float64, device="cuda")
    return torch.where(k < n // 2, k, k - n)


def _psd(c, f2, cn2dz):
    k = 2 * math.pi / c["wavelength"]
    return 0.023 * 0.423 * k * k * cn2dz * torch.exp(-f2 * c["l0"] ** 2) / (f2 + 1.0 / c["L0"] ** 2) ** (11.0 / 6.0)


def _amplitude(c, cn2dz):
    n, df = c["n"], 1.0 / c["side"]
    k = _bins(n)
    a = torch.sqrt(_psd(c, (k[:, None] ** 2 + k[None, :] ** 2) * df * df, cn2dz)) * df
    a[0, 0] = 0
    return a


def _sh_coefficients(c, seed, t, pairs, screen, cn2dz, tag):
    """[pairs][levels][8] subharmonic coefficients."""
    df, out = 1.0 / c["side"], []
    for p in range(1, c["sh"] + 1):
        dfp = df / 3.0 ** p
        e = torch.arange(4 * (p - 1), 4 * p, dtype=torch.int64, device="cuda")
        v = _philox(e[None, :], _word(t), pairs[:, None], _word((tag << 28) | screen), seed)
        z = torch.stack([_normal(v[0], v[1]), _normal(v[2], v[3])], 2).reshape(len(pairs), 8)
        f2 = torch.tensor([(a * a + b * b) * dfp * dfp for a, b in _OFFSETS], dtype=torch.float64, device="cuda")
        out.append(z * torch.sqrt(_psd(c, f2, cn2dz)) * dfp)
    return torch.stack(out, 1)


def _screens(c, spectra, coefs):
    """Real screens [2 pairs][n][n] of pair spectra and subharmonic coefficients."""
    n = c["n"]
    z = torch.fft.ifft2(spectra, norm="forward")
    if coefs is not None:
        x = _grid(n, 1.0)
        for p in range(coefs.shape[1]):
            for q, (a, b) in enumerate(_OFFSETS):
                ph = 2 * math.pi * (b * x[None, :] + a * x[:, None]) / (n * 3.0 ** (p + 1))
                z = z + coefs[:, p, q, None, None] * torch.polar(torch.ones_like(ph), ph)
        z = z - z.mean((1, 2), keepdim=True)
    return torch.view_as_real(z).permute(0, 3, 1, 2).reshape(-1, n, n)


def _synthesised(c, seed, t, pairs, screen, cn2dz):
    spec = _spectral_noise(c["n"], seed, t, pairs, 1, screen) * _amplitude(c, cn2dz)
    return _screens(c, spec, _sh_coefficients(c, seed, t, pairs, screen, cn2dz, 2) if c["sh"] else None)


def _transfer(c, dz):
    k = _bins(c["n"]) / c["side"]
    f2 = k[:, None] ** 2 + k[None, :] ** 2
    if c["angular"]:  # every bin propagates on these grids
        kk, kap2 = 2 * math.pi / c["wavelength"], 4 * math.pi ** 2 * f2
        ph = -dz * kap2 / (torch.sqrt(kk * kk - kap2) + kk)
    else:
        ph = -math.pi * c["wavelength"] * dz * f2
    return torch.polar(torch.ones_like(ph), ph)


def _chunks(c):
    """Realization ranges, whole pairs, of about 2^26 pixels."""
    per = max(2, 2 * (2 ** 25 // c["n"] ** 2))
    return [(lo, min(c["r"], lo + per)) for lo in range(0, c["r"], per)]


def _exact_path(c, source, screen_of, g_out=None, want_phi=True):
    """Fields at the end of the path and, with g_out, the gradients; screen_of
    (lo, hi, s): screens of realizations lo..hi - 1."""
    _, dz, cn2dz = _geometry(c)
    m, outs, g_ins, g_phis = c["m"], [], [], []
    for lo, hi in _chunks(c):
        u = (source if source.dim() == 2 else source[lo:hi]).to(torch.complex128)
        u = u.expand(hi - lo, -1, -1)
        kept, phis = [], []
        for s in range(m):
            u = torch.fft.ifft2(torch.fft.fft2(u) * _transfer(c, dz[s]))
            phi = screen_of(lo, hi, s)
            u = u * torch.polar(torch.ones_like(phi), phi)
            if g_out is not None:
                kept.append(u)
                phis.append(phi)
        u = torch.fft.ifft2(torch.fft.fft2(u) * _transfer(c, dz[m]))
        outs.append(u)
        if g_out is not None:
            g = g_out[lo:hi].to(torch.complex128)
            g = torch.fft.ifft2(torch.fft.fft2(g) * _transfer(c, dz[m]).conj())
            back = [None] * m
            for s in range(m - 1, -1, -1):
                w = kept.pop()
                back[s] = w.real * g.imag - w.imag * g.real
                phi = phis.pop()
                g = g * torch.polar(torch.ones_like(phi), -phi)
                g = torch.fft.ifft2(torch.fft.fft2(g) * _transfer(c, dz[s]).conj())
            g_ins.append(g)
            g_phis.append(torch.stack(back, 1))
    u = torch.cat(outs)
    if g_out is None:
        return u
    g_in = torch.cat(g_ins)
    return u, (g_in.sum(0) if source.dim() == 2 else g_in), torch.cat(g_phis)


def _moments64(u):
    i = u.real ** 2 + u.imag ** 2
    zero = torch.zeros_like(i[0])
    return torch.stack([i.sum(0), zero, (i * i).sum(0), zero])


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "serving":
        parts = [[], [], []]
        for i, p in enumerate(_mix(c)):
            key = (seed + i * 0x9E3779B97F4A7C15) % (1 << 64)
            got = _exact_fields(p, key, 0, _source(p, seed + i).unsqueeze(0),
                                _cotangent(p, seed + i) if c["grad"] else None)
            for k, x in enumerate(got if c["grad"] else (got,)):
                parts[k].append(x.reshape(-1))
        return dict(zip(("u", "g_in", "g_phi") if c["grad"] else ("u",), (torch.cat(x) for x in parts if x)))
    if kind == "stats":
        return _exact_stats(c, seed)
    if kind == "train":
        return _exact_train(c, seed)
    source = _source(c, seed, c["r"] if kind == "given" or c["source"] == "own" else 0)
    if kind == "forward":
        u = _exact_fields(c, seed, 0, source)
        return {"u": u, "moments": _moments64(u)} if c.get("moments") else {"u": u}
    if kind == "adjoint":
        return dict(zip(("u", "g_in", "g_phi"), _exact_fields(c, seed, 0, source, _cotangent(c, seed))))
    if kind == "given":
        _, _, cn2dz = _geometry(c)
        pairs = torch.arange((c["r"] + 1) // 2, device="cuda")
        phi = torch.stack([_synthesised(c, seed, 0, pairs, s, cn2dz[s])[:c["r"]] for s in range(c["m"])], 1)
        # the gradients are those at the screens that the caller holds, in 32 bits
        held = phi.float().double()
        u, g_in, g_phi = _exact_path(c, source, lambda lo, hi, s: held[lo:hi, s], _cotangent(c, seed))
        return {"screens": phi, "u": u, "g_in": g_in, "g_phi": g_phi}
    if kind == "ar":
        return _exact_ar(c, seed, source)
    return None


def _exact_fields(c, key, t, source, g_out=None):
    _, _, cn2dz = _geometry(c)

    def screen_of(lo, hi, s):
        pairs = torch.arange(lo // 2, (hi + 1) // 2, device="cuda")
        return _synthesised(c, key, t, pairs, s, cn2dz[s])[:hi - lo]
    return _exact_path(c, source, screen_of, g_out)


def _exact_ar(c, seed, source):
    """One step (t = 1) from the static spectra: the translation by (shift_x,
    shift_y) pixels, then the blend with fresh innovations."""
    n, alpha = c["n"], c["alpha"]
    _, _, cn2dz = _geometry(c)
    pairs = torch.arange((c["r"] + 1) // 2, device="cuda")
    k = _bins(n)
    ph = -2 * math.pi * (k[None, :] * c["shift_x"] + k[:, None] * c["shift_y"]) / n
    move = alpha * torch.polar(torch.ones_like(ph), ph)
    blend = math.sqrt(1 - alpha * alpha)
    spectra = torch.empty((len(pairs), c["m"], n, n), dtype=torch.complex128, device="cuda")
    coefs = []
    for s in range(c["m"]):
        amp = _amplitude(c, cn2dz[s])
        spectra[:, s] = (_spectral_noise(n, seed, 0, pairs, 1, s) * move +
                         blend * _spectral_noise(n, seed, 1, pairs, 3, s)) * amp
        if c["sh"]:
            d = _sh_coefficients(c, seed, 0, pairs, s, cn2dz[s], 2)
            ph = torch.tensor([[-2 * math.pi * (b * c["shift_x"] + a * c["shift_y"]) / (3.0 ** p * n)
                                for a, b in _OFFSETS] for p in range(1, c["sh"] + 1)], dtype=torch.float64,
                              device="cuda")
            coefs.append(alpha * d * torch.polar(torch.ones_like(ph), ph) +
                         blend * _sh_coefficients(c, seed, 1, pairs, s, cn2dz[s], 4))
    u = _exact_path(c, source, lambda lo, hi, s: _screens(
        c, spectra[lo // 2:(hi + 1) // 2, s], coefs[s][lo // 2:(hi + 1) // 2] if coefs else None)[:hi - lo])
    return {"u": u, "state": spectra}


def _receive(c, u, theta1, theta2):
    n, dx = c["n"], c["side"] / c["n"]
    x = _grid(n, dx)
    disc = ((x[None, :] ** 2 + x[:, None] ** 2) <= (0.5 * 0.3 * c["side"]) ** 2).double()
    z = torch.fft.fft2(disc * u * torch.polar(torch.ones_like(theta1), theta1))
    m2 = torch.fft.ifftshift(theta2)
    return torch.fft.ifft2(z * torch.polar(torch.ones_like(m2), m2)), disc


def _exact_train(c, seed):
    x = _grid(c["n"], c["side"] / c["n"])
    source = torch.exp(-(x[None, :] ** 2 + x[:, None] ** 2) / c["w0"] ** 2).to(torch.complex64)
    u_rx = _exact_fields(c, seed, 0, source)
    theta1, theta2 = (t.double().requires_grad_() for t in _masks(c["n"], seed))
    still = dict(c, r=1)
    vac = _exact_path(still, source, lambda lo, hi, s: torch.zeros((1, c["n"], c["n"]), dtype=torch.float64,
                                                                   device="cuda"))
    i_vac = _receive(c, vac, torch.zeros_like(theta1), torch.zeros_like(theta2))[0].abs()[0].detach() ** 2
    u, disc = _receive(c, u_rx, theta1, theta2)
    i = u.real ** 2 + u.imag ** 2
    m1 = i.mean(0)
    loss = (((i - m1) ** 2).mean(0) * disc).sum() / (m1 * m1 * disc).sum() + ((m1 - i_vac) ** 2).sum() / \
        (i_vac * i_vac).sum()
    g1, g2 = torch.autograd.grad(loss, [theta1, theta2])
    return {"loss": loss.detach(), "g1": g1, "g2": g2, "u": u.detach()}


def _exact_stats(c, seed):
    n, r, dx = c["n"], c["r"], c["side"] / c["n"]
    mom = torch.zeros((4, n, n), dtype=torch.float64, device="cuda")
    u = _received(c, seed)
    for i in range(0, r, 16):
        mom += _moments64(u[i:i + 16].to(torch.complex128))
    m1, m2 = mom[0] / r, mom[2] / r
    si = m2 / (m1 * m1) - 1
    x = _grid(n, dx)
    r2 = x[None, :] ** 2 + x[:, None] ** 2
    weight = (r2 <= (0.4 * c["side"]) ** 2).double()
    if c["power"] > 0:
        v = m1.reshape(-1).sort(descending=True).values
        at = int(torch.searchsorted(v.cumsum(0), c["power"] * v.sum()))
        threshold = float(v[min(at, v.numel() - 1)])
        region = m1 >= threshold
    else:
        threshold = 0.0
        inner = (torch.arange(n, device="cuda") - n // 2).abs() < n // 4
        region = inner[:, None] & inner[None, :]
    total = float(weight[region].sum())
    si_sum = float((weight * si)[region].sum())
    fit = m1 >= math.exp(-2) * m1.max()
    a, b = r2[fit], torch.log(m1[fit])
    slope = float(((a - a.mean()) * (b - b.mean())).sum() / ((a - a.mean()) ** 2).sum())
    summary = {"si_plane": si_sum / total, "w_2nd": math.sqrt(2 * float((r2 * m1).sum() / m1.sum())),
               "w_fit": math.sqrt(-2 / slope), "count": r, "si_sum": si_sum, "region_weight": total,
               "threshold": threshold}
    return {"si": si, "summary": summary, "moments": mom}
