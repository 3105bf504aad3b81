"""Work that a user of this library has it do, through the Python entry points of paper_1609_08146_amd.

Every case is a plain dict with a "kind" and sizes:

  solve    a problem is set up once (mirror, spectrum, beam, points); a pass evaluates the reflected
           spectral field into device tensors (evaluate, or evaluate_noalloc in a tight loop)
  step     a pass is the whole path from the parameters: mirror nodes, spectrum, incident beam, points,
           evaluation, time samples
  scan     the same for a small mesh, results as host arrays: one point of a parameter scan
  fields   a pass hands over the incident field on the mirror nodes (device tensors) and evaluates
  surface  a mirror given by its own quadrature (an off-axis paraboloid segment) and its field
  energy   a pass evaluates a focal volume and sums its field energy at a few times
  batch    several problems of uneven size in one evaluate_batch
  serve    a burst of requests through the serving loop, results on the host

Lengths are in metres with the 800 nm / 10 fs pulse ("si"), or in wavelengths ("unit").  The seed
moves what a user's next problem changes: polarisation, waist, chirp of the spectrum, and the exact
place of the observation grid.  exact() sums the same discrete integrals in 64 bits with torch.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

C_LIGHT = 299_792_458.0
LAMBDA0 = 800e-9
TAU = 10e-15
EXACT_EVALS = 1.2e11      # point x frequency x node sums that exact() does in about ten seconds on the GPU


def listed():
    return [
        # a point or two of a focal spot inside a caller's own loop: the call's latency is all there is
        dict(name="spot_noalloc", kind="solve", scale="unit", f=20.0, a=40.0, n_r=64, n_phi=48, n_k=1, grid=10,
             axial=14, half=2.0, beam="linear", prec="fp32_split", call="noalloc"),
        # the monochromatic reference problem (wavelength 1, f = 20, NA = 1) in double precision
        dict(name="mono_fp64", kind="solve", scale="unit", f=20.0, a=40.0, n_r=200, n_phi=200, n_k=1, grid=32,
             axial=0, half=2.0, beam="linear", prec="fp64", call="out"),
        # one point of a scan over mirrors: everything from the parameters, result on the host
        dict(name="scan_host", kind="scan", scale="si", f=0.0675, a=0.125, n_r=100, n_phi=100, n_k=5, grid=21,
             axial=17, half=2.0, beam="radial", prec="fp32_split"),
        # the broadband pulse of the benchmark, whole path with 256 time samples
        dict(name="broadband_step", kind="step", scale="si", f=0.1, a=0.075, n_r=400, n_phi=400, n_k=128, grid=64,
             axial=64, half=4.0, beam="linear", prec="fp32_split", n_t=256),
        # the same pulse, spectral field alone, in double precision
        dict(name="broadband_fp64", kind="solve", scale="si", f=0.1, a=0.075, n_r=400, n_phi=400, n_k=128, grid=64,
             axial=64, half=4.0, beam="linear", prec="fp64", call="out"),
        # the deep dish with its fine mesh and a 128 x 128 focal plane
        dict(name="deep_dish", kind="solve", scale="si", f=0.05, a=0.15, n_r=800, n_phi=800, n_k=11, grid=128,
             axial=0, half=2.0, beam="linear", prec="fp32_split", call="out"),
        # a circularly polarised Laguerre-Gauss set: the current of a node does not keep one direction
        dict(name="lg_circular", kind="solve", scale="si", f=0.0675, a=0.125, n_r=300, n_phi=280, n_k=32, grid=41,
             axial=33, half=2.0, beam="lg", prec="fp32_split", call="out"),
        # an aberrated field that the caller computed on the nodes
        dict(name="user_fields", kind="fields", scale="unit", f=20.0, a=30.0, n_r=160, n_phi=144, n_k=12, grid=33,
             axial=25, half=2.5, prec="fp32_split"),
        # an off-axis segment handed over as its own quadrature, double precision
        dict(name="off_axis_fp64", kind="surface", scale="unit", f=20.0, a=8.0, n_r=90, n_phi=96, n_k=4, grid=17,
             axial=11, half=2.0, prec="fp64"),
        # energy in a focal volume, double precision
        dict(name="volume_energy", kind="energy", scale="si", f=0.0675, a=0.125, n_r=200, n_phi=200, n_k=20, grid=19,
             axial=0, half=3.0, beam="linear", prec="fp64", n_t=5),
        # eight problems of uneven size in one launch
        dict(name="sweep_batch", kind="batch", scale="si", count=8, n_lo=100, n_hi=420, k_hi=64, g_lo=16, g_hi=90,
             prec="fp32_split"),
        # a burst of six requests to the serving loop
        dict(name="serve_burst", kind="serve", scale="si", count=6, n_lo=100, n_hi=300, k_hi=32, g_lo=16, g_hi=48,
             prec="fp32_split", n_t=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "step", "scan", "fields", "surface", "energy", "batch", "serve"])
    prec = rng.choice(["fp32_split", "fp32_split", "fp64"])
    scale = rng.choice(["si", "si", "unit"])
    f = rng.uniform(0.03, 0.15) if scale == "si" else rng.uniform(15.0, 40.0)
    a = f * rng.uniform(0.6, 2.5)
    c = dict(kind=kind, scale=scale, f=f, a=a, prec=prec, half=rng.uniform(1.0, 4.0))
    if kind in ("batch", "serve"):
        return dict(kind=kind, scale="si", count=rng.randint(2, 8), n_lo=rng.randint(40, 120), n_hi=rng.randint(150, 380),
                    k_hi=_log(rng, 4, 64), g_lo=rng.randint(8, 20), g_hi=rng.randint(24, 64), prec="fp32_split",
                    **({"n_t": _log(rng, 8, 128)} if kind == "serve" else {}))
    c.update(n_r=_log(rng, 24, 500), n_phi=_log(rng, 24, 500), n_k=_log(rng, 1, 128), grid=_log(rng, 4, 90),
             axial=rng.randint(0, 40))
    if kind == "surface":
        c.update(scale="unit", f=20.0, a=rng.uniform(4.0, 10.0), n_r=_log(rng, 20, 160), n_phi=_log(rng, 20, 160),
                 n_k=_log(rng, 1, 8), grid=_log(rng, 4, 33))
    elif kind == "fields":
        c.update(scale="unit", f=rng.uniform(15.0, 40.0), n_r=_log(rng, 30, 220), n_phi=_log(rng, 30, 220),
                 n_k=_log(rng, 1, 24))
        c["a"] = c["f"] * rng.uniform(0.6, 2.0)
    elif kind == "energy":
        c.update(prec="fp64", beam="linear", n_r=_log(rng, 40, 240), n_phi=_log(rng, 40, 240), n_k=_log(rng, 2, 24),
                 grid=rng.randint(5, 19), axial=0, n_t=rng.randint(1, 6))
    elif kind == "scan":
        c.update(n_r=_log(rng, 24, 130), n_phi=_log(rng, 24, 130), n_k=_log(rng, 1, 8), grid=_log(rng, 4, 33),
                 beam=rng.choice(["linear", "radial", "azimuthal"]))
    elif kind == "step":
        c.update(beam=rng.choice(["linear", "radial"]), n_k=_log(rng, 2, 128), n_t=_log(rng, 16, 256))
    else:
        c.update(beam=rng.choice(["linear", "linear", "radial", "azimuthal", "lg"]), call="out")
    # no larger than the largest listed case, and in double precision half of it
    most = 8e10 if c["prec"] == "fp32_split" else 3e10
    while _evals(c) > most:
        big = max(("n_r", "n_phi", "n_k", "grid"), key=lambda s: c[s])
        c[big] = max(2, int(c[big] * 0.8))
    return c


# ------------------------------------------------------------------------------------------ inputs

def _spectrum(n_k, scale, rng):
    """Wavenumbers, complex amplitudes (Gaussian pulse with a seeded chirp) and their spacing."""
    if scale == "si":
        k0, sig = 2 * math.pi / LAMBDA0, 2 * math.sqrt(math.log(2.0)) / TAU / C_LIGHT
    else:
        k0, sig = 2 * math.pi, 0.07 * 2 * math.pi
    if n_k == 1:
        return np.array([k0]), np.array([np.exp(1j * rng.uniform(0, 6))]), 6.0 * sig
    k = np.linspace(k0 - 3 * sig, k0 + 3 * sig, n_k)
    x = (k - k0) / sig
    return k, np.exp(-0.5 * x * x + 1j * (rng.uniform(-1, 1) * x * x + rng.uniform(0, 6))), float(k[1] - k[0])


def _points(c, rng, volume=False):
    lam = LAMBDA0 if c["scale"] == "si" else 1.0
    h, n = c["half"] * lam, c["grid"]
    s = np.linspace(-h, h, n) + rng.uniform(-0.05, 0.05) * lam
    if volume:
        z, y, x = np.meshgrid(s, s, s, indexing="ij")
        return np.ascontiguousarray(np.stack([x.ravel(), y.ravel(), z.ravel()], axis=-1))
    y, x = np.meshgrid(s, s, indexing="ij")
    pts = [np.stack([x.ravel(), y.ravel(), np.full(n * n, rng.uniform(-0.05, 0.05) * lam)], axis=-1)]
    if c.get("axial"):
        z = np.linspace(-h, h, c["axial"]) + rng.uniform(-0.05, 0.05) * lam
        pts.append(np.stack([0 * z, 0 * z, z], axis=-1))
    return np.ascontiguousarray(np.concatenate(pts))


def _problem(c, seed):
    """Parameters of one mirror problem (a workload as problem_from_workload takes it)."""
    rng = np.random.default_rng([seed, 11])
    k, amp, dk = _spectrum(c["n_k"], c["scale"], rng)
    obs = _points(c, rng, c["kind"] == "energy")
    t = 2 * c["f"] + (np.arange(c.get("n_t", 0)) - c.get("n_t", 0) // 2) * (2 * math.pi / (max(c.get("n_t", 1), 1) * dk))
    if c["kind"] == "energy":
        t = 2 * c["f"] + np.linspace(-0.4, 0.4, c["n_t"]) * (LAMBDA0 if c["scale"] == "si" else 1.0)
    beam = c.get("beam", "linear")
    return SimpleNamespace(f=c["f"], a=c["a"], n_r=c["n_r"], n_phi=c["n_phi"], k=k, spectrum=amp, dk=dk, obs=obs,
                           w0=c["a"] * rng.uniform(0.45, 0.75), pol=rng.uniform(0, math.pi), consistent=0,
                           beam={"linear": 0, "radial": 1, "azimuthal": 2}.get(beam, 0), t=t,
                           modes=[(0, 1, 1.0, 1j * rng.uniform(0.8, 1.0)), (1, -2, 0.4, -0.5j)] if beam == "lg" else None)


def _uneven(c, seed):
    """Problems of uneven size; the sizes are the case's, the seed moves their contents."""
    sizes = np.random.default_rng([c["count"], c["n_lo"], c["n_hi"], c["k_hi"]])
    out = []
    for i in range(c["count"]):
        f = sizes.uniform(0.02, 0.2)
        n = int(sizes.integers(c["n_lo"], c["n_hi"] + 1))
        q = dict(kind="solve", scale="si", f=f, a=f * sizes.uniform(1.0, 3.0), n_r=n, n_phi=n, beam="linear", half=4.0,
                 n_k=int(round(math.exp(sizes.uniform(0.0, math.log(c["k_hi"]))))),
                 grid=int(sizes.integers(c["g_lo"], c["g_hi"] + 1)), axial=int(sizes.integers(8, 64)),
                 n_t=c.get("n_t", 0))
        out.append((q, _problem(q, seed * 64 + i)))
    return out


def _user_field(pts, k, amp, c, seed, cx=0.0):
    """A collimated beam along -z with a smooth aberration and a little field noise, on any nodes."""
    rng = np.random.default_rng([seed, 23])
    w0, tilt, coma = 0.6 * c["a"], rng.uniform(-0.3, 0.3, 2), rng.uniform(-0.3, 0.3)
    noise = np.random.default_rng([seed, 29]).standard_normal((4, len(pts))) * 1e-3
    x, y = (pts[:, 0] - cx) / c["a"], pts[:, 1] / c["a"]
    ab = tilt[0] * x + tilt[1] * y + coma * (x * x + y * y) * x
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    tt = lambda v: torch.as_tensor(v, dtype=torch.float64, device=dev)  # noqa: E731
    G = tt(np.exp(-((x * c["a"]) ** 2 + (y * c["a"]) ** 2) / w0 ** 2))
    ph = tt(ab)[None, :] - tt(k)[:, None] * tt(pts[:, 2])[None, :]
    psi = torch.polar(G.expand_as(ph).contiguous(), ph) * torch.as_tensor(amp, device=dev)[:, None]
    n = tt(noise)
    ex, ey = psi * (1.0 + n[0]), psi * (0.3j + n[1])
    z = torch.zeros_like(psi)
    E = torch.stack([ex, ey, z], dim=-1).contiguous()
    B = torch.stack([ey * (1.0 + n[2]), -ex * (1.0 + n[3]), z], dim=-1).contiguous()
    return E, B


def _segment(c):
    """Off-axis paraboloid segment (disk of radius a about (f, 0)): nodes, n dS, rim nodes, normals, dl."""
    f, cx, rad = c["f"], c["f"], c["a"]
    xg, wg = np.polynomial.legendre.leggauss(c["n_r"])
    rho, wr = rad * (xg + 1) / 2, rad * wg / 2
    psi = 2 * math.pi * np.arange(c["n_phi"]) / c["n_phi"]

    def lift(R, P):
        x, y = cx + R * np.cos(P), R * np.sin(P)
        return np.stack([x, y, (x * x + y * y) / (4 * f) - f], -1), np.stack([-x / (2 * f), -y / (2 * f), 1 + 0 * x], -1)

    R, P = np.meshgrid(rho, psi, indexing="ij")
    xyz, n = lift(R, P)
    W = (wr * rho)[:, None] * (2 * math.pi / c["n_phi"]) * np.ones_like(P)
    rx, rn = lift(np.full_like(psi, rad), psi)
    dx, dy = -rad * np.sin(psi), rad * np.cos(psi)
    dl = np.stack([dx, dy, (rx[:, 0] * dx + rx[:, 1] * dy) / (2 * f)], -1) * (2 * math.pi / c["n_phi"])
    return xyz.reshape(-1, 3), (n * W[..., None]).reshape(-1, 3), rx, rn, dl


# ------------------------------------------------------------------------------------- the library

def _outputs(n_k, n_obs, prec):
    dt = torch.complex128 if prec == "fp64" else torch.complex64
    return tuple(torch.empty((n_k, n_obs, 3), dtype=dt, device="cuda") for _ in range(2))


def _set_up(p, w):
    p.set_mirror(w.f, w.a, w.n_r, w.n_phi)
    p.set_frequencies(w.k)
    if w.modes:
        p.set_incident_lg(w.modes, w.w0, w.spectrum)
    else:
        p.set_incident_beam(w.beam, w.w0, w.pol, w.spectrum)
    p.set_observation(w.obs)


def prepare(case, seed):
    from paper_1609_08146_amd import Context, Problem, Server
    c, kind = case, case["kind"]
    if kind == "serve":
        ctx = Context(0, use_torch_stream=False)
        s = SimpleNamespace(case=c, ctx=ctx, works=[w for _, w in _uneven(c, seed)],
                            server=Server(ctx, hbm_budget=int(24e9), max_running=16))
        return s
    s = SimpleNamespace(case=c, ctx=Context(0))
    if kind == "batch":
        s.probs = []
        for _, w in _uneven(c, seed):
            p = Problem(s.ctx)
            _set_up(p, w)
            s.probs.append(p)
        return s
    s.p = Problem(s.ctx)
    if kind in ("solve", "step", "scan", "energy"):
        s.w = _problem(c, seed)
        if kind in ("solve", "energy"):
            _set_up(s.p, s.w)
        if kind in ("solve", "step"):
            s.out = _outputs(len(s.w.k), len(s.w.obs), c["prec"])
        if kind == "step":
            s.tout = _outputs(c["n_t"], len(s.w.obs), c["prec"])
        if c.get("call") == "noalloc":
            s.p.evaluate(c["prec"], out=s.out)     # the call without allocation needs one ordinary evaluation first
        return s
    rng = np.random.default_rng([seed, 11])
    k, amp, _ = _spectrum(c["n_k"], c["scale"], rng)
    obs = _points(c, rng)
    if kind == "fields":
        s.p.set_mirror(c["f"], c["a"], c["n_r"], c["n_phi"])
        s.p.set_frequencies(k)
        s.p.set_observation(obs)
        s.E, s.B = _user_field(s.p.get_nodes()[0], k, amp, c, seed)
    else:
        xyz, nds, rx, rn, dl = _segment(c)
        s.p.set_surface(xyz, nds, rx, rn, dl)
        s.p.set_frequencies(k)
        s.p.set_observation(obs)
        E, B = _user_field(np.concatenate([xyz, rx]), k, amp, c, seed, cx=c["f"])
        s.p.set_incident(E, B)
        torch.cuda.synchronize()
    s.out = _outputs(len(k), len(obs), c["prec"])
    return s


def run(s):
    c = s.case
    kind, prec = c["kind"], c.get("prec")
    if kind == "solve":
        if c["call"] == "noalloc":
            return s.p.evaluate_noalloc(s.out, prec)
        return s.p.evaluate(prec, out=s.out)
    if kind == "step":
        _set_up(s.p, s.w)
        s.p.evaluate(prec, out=s.out)
        return s.out + tuple(s.p.to_time_at(s.w.dk, s.w.t, out=s.tout))
    if kind == "scan":
        _set_up(s.p, s.w)
        return s.p.evaluate(prec)
    if kind == "fields":
        s.p.set_incident(s.E, s.B)
        return s.p.evaluate(prec, out=s.out)
    if kind == "surface":
        return s.p.evaluate(prec, out=s.out)
    if kind == "energy":
        s.p.evaluate(prec, keep_on_device=True)
        return s.p.field_energy(s.w.t, s.w.dk, 1.0)
    if kind == "batch":
        s.ctx.evaluate_batch(s.probs, prec)
        return [p.result() for p in s.probs]
    tickets = [s.server.submit(w, prec, t=w.t, dk=w.dk) for w in s.works]
    return [s.server.wait(t)[:4] for t in tickets]


# ------------------------------------------------------------------------------------------- work

def _shapes(c):
    """(frequencies, points, nodes, times) of each problem of a case."""
    if c["kind"] in ("batch", "serve"):
        return [(q["n_k"], q["grid"] ** 2 + q["axial"], (q["n_r"] + 1) * q["n_phi"], q["n_t"]) for q, _ in _uneven(c, 0)]
    n_obs = c["grid"] ** 3 if c["kind"] == "energy" else c["grid"] ** 2 + c["axial"]
    return [(c["n_k"], n_obs, (c["n_r"] + 1) * c["n_phi"], c.get("n_t", 0))]


def _evals(c):
    return sum(k * o * n for k, o, n, _ in _shapes(c))


def work(case):
    """What no method can do without: every node's current and charge at every frequency (four complex
    numbers) enters once, every output is written once (and the time samples read the spectrum once)."""
    real = 8 if case["prec"] == "fp64" else 4
    bytes_ = flops = 0
    for k, o, n, t in _shapes(case):
        bytes_ += 8 * real * k * n + 12 * real * k * o + 24 * o
        flops += 8 * 4 * k * n + 48 * k * o
        if case["kind"] != "energy" and t:
            bytes_ += 12 * real * o * (k + t)
            flops += 8 * 6 * k * t * o
        if case["kind"] == "fields":
            bytes_ += 96 * k * n
    return {"bytes": float(bytes_), "flops": float(flops)}


# ------------------------------------------------------------------------------------------ exact

def _nodes(f, a, n_r, n_phi):
    """Nodes, n~ times weight (surface) and rim data of the paraboloid, Gauss-Legendre x trapezoid."""
    xg, wg = np.polynomial.legendre.leggauss(n_r)
    r, wr = a * (xg + 1) / 2, a * wg / 2
    phi = 2 * math.pi * np.arange(n_phi) / n_phi
    rr = np.append(r, a)
    x, y = np.outer(rr, np.cos(phi)), np.outer(rr, np.sin(phi))
    xyz = np.stack([x, y, (rr ** 2 / (4 * f) - f)[:, None] + 0 * x], -1)
    n = np.stack([-x / (2 * f), -y / (2 * f), 1 + 0 * x], -1)
    W = (wr * r)[:, None] * (2 * math.pi / n_phi) + 0 * x[:-1]
    rim = xyz[-1]
    dl = np.stack([-rim[:, 1], rim[:, 0], 0 * phi], -1) * (2 * math.pi / n_phi)
    return xyz.reshape(-1, 3), (n[:-1] * W[..., None]).reshape(-1, 3), n[-1], dl


def _cross(a, b):
    return torch.stack([a[..., 1] * b[..., 2] - a[..., 2] * b[..., 1], a[..., 2] * b[..., 0] - a[..., 0] * b[..., 2],
                        a[..., 0] * b[..., 1] - a[..., 1] * b[..., 0]], -1)


def _field(k, obs, xyz, nds, rim_n, rim_dl, EB):
    """The discrete sums: EB(n) gives E, B on all nodes at frequency n with the node phase e^{ik|r_s|} in."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    T = lambda v: torch.as_tensor(np.ascontiguousarray(v), dtype=torch.float64, device=dev)  # noqa: E731
    rs, o, nds, rim_n, rim_dl = T(xyz), T(obs), T(nds), T(rim_n), T(rim_dl)
    n_surf, R0, o2 = len(nds), T(xyz).norm(dim=1), (T(obs) ** 2).sum(1)
    E = torch.zeros((len(k), len(obs), 3), dtype=torch.complex128, device=dev)
    B = torch.zeros_like(E)
    tabs = []
    for n, kn in enumerate(k):
        e, b = EB(n)
        J = torch.zeros_like(b)
        J[:n_surf] = (2j * kn / (4 * math.pi)) * _cross(nds.to(b.dtype), b[:n_surf])
        rho = torch.zeros(len(rs), dtype=b.dtype, device=dev)
        rho[:n_surf] = (2 / (4 * math.pi)) * (nds * e[:n_surf]).sum(-1)
        if len(rs) > n_surf:
            br, nh = b[n_surf:], rim_n / rim_n.norm(dim=1, keepdim=True)
            rho[n_surf:] = (2j / (4 * math.pi * kn)) * ((nh * (nh * br).sum(-1, keepdim=True) - br) * rim_dl).sum(-1)
        rc = rs.to(b.dtype)
        tabs.append((J, torch.cat([rho[:, None] * rc, rho[:, None], _cross(J, rc), J], 1)))
    ob = max(1, min(len(obs), 4096))
    step = max(1, int(2.5e7 // ob))
    for o0 in range(0, len(obs), ob):
        op = o[o0:o0 + ob]
        oc = op.to(torch.complex128)
        for q0 in range(0, len(rs), step):
            q = slice(q0, q0 + step)
            d = rs[q][None] - op[:, None]
            R = d.norm(dim=-1)
            delta = (o2[o0:o0 + ob, None] - 2 * (op @ rs[q].T)) / (R + R0[q][None])
            del d
            inv = 1.0 / R
            for n, kn in enumerate(k):
                G = torch.polar(inv, kn * delta)
                H = G * torch.complex(-inv * inv, kn * inv)
                e = G @ tabs[n][0][q]
                h = H @ tabs[n][1][q]
                E[n, o0:o0 + ob] += e + h[:, :3] - h[:, 3:4] * oc
                B[n, o0:o0 + ob] += (h[:, 4:7] - _cross(h[:, 7:], oc)) / (1j * kn)
    return E, B


def _beam_EB(w, xyz):
    """E, B of the built-in beams on the nodes; on the paraboloid k (|r_s| - z) = 2 k f exactly."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    x, y = (torch.as_tensor(xyz[:, i].copy(), device=dev) for i in (0, 1))
    G, z = torch.exp(-(x * x + y * y) / w.w0 ** 2), torch.zeros_like(x)
    turn = [complex(np.exp(1j * float((np.longdouble(k) * 2 * np.longdouble(w.f)) % (8 * np.arctan(np.longdouble(1))))))
            for k in w.k]
    if w.modes:
        t = 2 * (x * x + y * y) / w.w0 ** 2
        ex = ey = 0
        for p, l, ax, ay in w.modes:
            L = torch.ones_like(t) if p == 0 else 1 + abs(l) - t
            C = math.sqrt(2 * math.factorial(p) / (math.pi * math.factorial(p + abs(l)))) / w.w0
            u = C * L * G * (torch.complex(x, y if l >= 0 else -y) * (math.sqrt(2) / w.w0)) ** abs(l)
            ex, ey = ex + ax * u, ey + ay * u
        E, B = torch.stack([ex, ey, 0 * ex], -1), torch.stack([ey, -ex, 0 * ex], -1)
    elif w.beam == 0:
        c, s = math.cos(w.pol), math.sin(w.pol)
        E, B = torch.stack([c * G, s * G, z], -1), torch.stack([s * G, -c * G, z], -1)
    else:
        g = G / w.w0
        E = torch.stack([x * g, y * g, z], -1) if w.beam == 1 else torch.stack([-y * g, x * g, z], -1)
        B = torch.stack([y * g, -x * g, z], -1) if w.beam == 1 else torch.stack([x * g, y * g, z], -1)
    E, B = E.to(torch.complex128), B.to(torch.complex128)
    return lambda n: (E * (w.spectrum[n] * turn[n]), B * (w.spectrum[n] * turn[n]))


def _times(k, dk, t, F):
    """dk sum_n F_n e^{-i k_n t}, phases reduced in extended precision."""
    ph = -np.outer(t.astype(np.longdouble), k.astype(np.longdouble)) % (8 * np.arctan(np.longdouble(1)))
    tw = torch.as_tensor(dk * np.exp(1j * ph.astype(np.float64)), device=F.device)
    return (tw @ F.reshape(len(k), -1)).reshape(len(t), *F.shape[1:])


def _solve(w):
    xyz, nds, rim_n, dl = _nodes(w.f, w.a, w.n_r, w.n_phi)
    return _field(w.k, w.obs, xyz, nds, rim_n, dl, _beam_EB(w, xyz))


def exact(case, seed):
    c, kind = case, case["kind"]
    if _evals(c) > EXACT_EVALS:
        return None
    if kind in ("batch", "serve"):
        out = []
        for _, w in _uneven(c, seed):
            E, B = _solve(w)
            out.append((E, B) + ((_times(w.k, w.dk, w.t, E), _times(w.k, w.dk, w.t, B)) if kind == "serve" else ()))
        return out
    if kind in ("solve", "step", "scan", "energy"):
        w = _problem(c, seed)
        E, B = _solve(w)
        if kind in ("solve", "scan"):
            return E, B
        Et, Bt = _times(w.k, w.dk, w.t, E), _times(w.k, w.dk, w.t, B)
        if kind == "step":
            return E, B, Et, Bt
        return 2.0 * ((Et.real ** 2).sum((1, 2)) + (Bt.real ** 2).sum((1, 2)))
    rng = np.random.default_rng([seed, 11])
    k, amp, _ = _spectrum(c["n_k"], c["scale"], rng)
    obs = _points(c, rng)
    if kind == "fields":
        xyz, nds, rim_n, dl = _nodes(c["f"], c["a"], c["n_r"], c["n_phi"])
        E, B = _user_field(xyz, k, amp, c, seed)
    else:
        xyz, nds, rx, rim_n, dl = _segment(c)
        xyz = np.concatenate([xyz, rx])
        E, B = _user_field(xyz, k, amp, c, seed, cx=c["f"])
    R0 = torch.as_tensor(np.linalg.norm(xyz, axis=1), device=E.device)
    return _field(k, obs, xyz, nds, rim_n, dl, lambda n: (E[n] * torch.exp(1j * k[n] * R0)[:, None],
                                                          B[n] * torch.exp(1j * k[n] * R0)[:, None]))
