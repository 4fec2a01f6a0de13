"""The framework's work at the sizes its users run it at: track finding (one
event to a batch, plain, steered, with a material map, with duplicate seeds, in
the parametrised field), Kalman fits (a handful of tracks to millions, fused
and per layer, every precision, learned start) and the training of the learned
start.

Inputs are synthetic events made on the GPU in 64 bits: charged tracks from a
Gaussian vertex through ten barrels (and 2 x 7 disks) in 3.8 T, hits smeared on
their surfaces, uniform noise hits.
"""
import functools
import math

import numpy as np
import torch

import paper_1906_02253_amd as K
from paper_1906_02253_amd import pipeline

KAPPA = 0.00299792458           # GeV / (T cm)
BZ = 3.8
MASS = 0.13957
BARREL_R = (4.0, 7.0, 11.0, 16.0, 25.0, 34.0, 50.0, 65.0, 80.0, 100.0)
DISK_Z = (30.0, 70.0, 110.0, 150.0, 190.0, 230.0, 270.0)
SIG_U, SIG_V = 0.01, 0.05
FIELD_Z0, FIELD_STEP = 300.0, 2.0
MAP_R, MAP_Z, MAP_N = 120.0, 300.0, 250
PREC = {"mixed": K.PREC_MIXED, "fp32": K.PREC_FP32, "fp64": K.PREC_FP64}

FIND = dict(kind="find", events=1, tracks=800, uneven=False, noise=60, disks=False, graph=True,
            steer=False, map=False, overlap=False, field=False)
FIT = dict(kind="fit", tracks=1000, disks=False, mix=False, shuffled=True, prec="mixed",
           per_layer=False, field=False, learned=False)
TRAIN = dict(kind="train", rows=100_000, batch=4096, steps=48)


def listed():
    return [
        # the shortest call: a region of interest or a test event, eager (seed, fit, find)
        dict(FIND, name="find_region", tracks=60, noise=50, graph=False),
        # one event as an event loop hands it over, through the captured pass
        dict(FIND, name="find_event", tracks=800, noise=62),
        # the throughput workload: events of uneven multiplicity, barrels and disks
        dict(FIND, name="find_batch", events=64, tracks=2100, uneven=True, disks=True),
        # tracking regions with layer plans and the r-z material map with energy loss
        dict(FIND, name="find_steered_map", events=24, tracks=1500, uneven=True, disks=True,
             steer=True, map=True),
        # up to eight seeds per particle: seed cleaning and duplicate removal
        dict(FIND, name="find_overlap", events=16, tracks=2100, uneven=True, disks=True,
             overlap=True),
        # the parametrised field, Runge-Kutta transport
        dict(FIND, name="find_field", events=16, tracks=2100, uneven=True, field=True),
        # the refit of one event's tracks, barrels and disks, hits in event order
        dict(FIT, name="fit_event", tracks=1000, disks=True),
        # the fit throughput set: loopers and stiff tracks, hits step-major
        dict(FIT, name="fit_large", tracks=4_000_000, mix=True, shuffled=False),
        # one launch per layer, the state through memory between layers
        dict(FIT, name="fit_per_layer", tracks=2_000_003, mix=True, shuffled=False,
             per_layer=True),
        # the precision set in 64 bits
        dict(FIT, name="fit_fp64", tracks=200_000, mix=True, prec="fp64"),
        # the learned start of the propagation solve
        dict(FIT, name="fit_learned", tracks=1_000_000, mix=True, shuffled=False, learned=True),
        # training of the learned start's network
        dict(TRAIN, name="train"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["find", "find", "find", "fit", "fit", "train"])
    if kind == "train":
        return dict(TRAIN, rows=_log_int(rng, 20_000, 400_000), batch=_log_int(rng, 64, 8192),
                    steps=rng.randint(4, 48))
    if kind == "fit":
        prec = rng.choice(["mixed", "mixed", "fp32", "fp64"])
        what = rng.choice(["plain", "plain", "per_layer", "field", "learned"])
        top = 4_000_000 if what == "plain" and prec != "fp64" else 500_000
        disks = what in ("plain", "per_layer") and rng.random() < 0.3
        return dict(FIT, tracks=_log_int(rng, 100, top), disks=disks,
                    mix=not disks and what != "field" and rng.random() < 0.6,
                    shuffled=rng.random() < 0.5, prec=prec, per_layer=what == "per_layer",
                    field=what == "field", learned=what == "learned")
    what = rng.choice(["plain", "plain", "steer", "map", "overlap", "field"])
    events = _log_int(rng, 1, 64)
    tracks = _log_int(rng, 40, 2100)
    if what in ("overlap", "field"):
        events = min(events, 24)
    return dict(FIND, events=events, tracks=tracks, uneven=events > 1 and rng.random() < 0.7,
                noise=rng.randint(20, 65), disks=what != "field" and rng.random() < 0.6,
                graph=events > 4 or rng.random() < 0.5, steer=what == "steer",
                map=what == "map" or (what == "steer" and rng.random() < 0.5),
                overlap=what == "overlap", field=what == "field")


# ---------------------------------------------------------------- detector
def _geometry(disks, x0):
    out = []
    for r in BARREL_R:
        half = r * math.sinh(1.0) + 2.0
        out.append(dict(kind=0, r_or_z=r, lo=-half, hi=half))
    for z in (DISK_Z + tuple(-z for z in DISK_Z)) if disks else ():
        out.append(dict(kind=1, r_or_z=z, lo=abs(z) / math.sinh(2.5),
                        hi=min(100.0, abs(z) / math.sinh(1.0))))
    return [dict(L, x0=x0, nbin_phi=128, nbin_2=32, win_su=SIG_U, win_sv=SIG_V) for L in out]


def _plans(geom):
    """Five tracking regions in eta; a plan lists the layers a straight line
    from the origin crosses in the region, by median path length."""
    out = []
    for lo, hi in ((-2.5, -1.6), (-1.6, -0.8), (-0.8, 0.8), (0.8, 1.6), (1.6, 2.5)):
        paths = {}
        for eta in np.linspace(lo, hi, 41)[1:-1]:
            sh, ch = math.sinh(eta), math.cosh(eta)
            for i, L in enumerate(geom):
                if L["kind"] == 0:
                    if L["lo"] <= L["r_or_z"] * sh <= L["hi"]:
                        paths.setdefault(i, []).append(L["r_or_z"] * ch)
                elif L["r_or_z"] * sh > 0 and L["lo"] <= L["r_or_z"] / sh <= L["hi"]:
                    paths.setdefault(i, []).append(abs(L["r_or_z"] / sh) * ch)
        out.append(dict(eta_lo=lo, eta_hi=hi,
                        layers=sorted(paths, key=lambda i: float(np.median(paths[i])))))
    return out


def _material_map(geom, base=0.02):
    """Radiation length fraction and areal density [g/cm^2] per r-z cell,
    varying smoothly along each surface; zero where no surface passes."""
    x0 = np.zeros((MAP_N, MAP_N), np.float32)
    dr, dz = MAP_R / MAP_N, 2 * MAP_Z / MAP_N
    rc, zc = (np.arange(MAP_N) + 0.5) * dr, -MAP_Z + (np.arange(MAP_N) + 0.5) * dz
    for L in geom:
        if L["kind"] == 0:
            u = np.clip(zc / L["hi"], -1, 1)
            x0[int(L["r_or_z"] / dr), :] = base * (1 + 0.6 * u ** 2 + 0.2 * np.sin(3 * u))
        else:
            u = np.clip((rc - L["lo"]) / (L["hi"] - L["lo"]) * 2 - 1, -1, 1)
            x0[:, int((L["r_or_z"] + MAP_Z) / dz)] = base * (1 + 0.6 * u ** 2 + 0.2 * np.sin(3 * u))
    return dict(r_max=MAP_R, z_min=-MAP_Z, z_max=MAP_Z, x0=x0, xi=(x0 * 21.82).astype(np.float32))


# ---------------------------------------------------------------- tracks
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _rand(g, n, lo=0.0, hi=1.0):
    return lo + (hi - lo) * torch.rand(n, dtype=torch.float64, device="cuda", generator=g)


def _randn(g, *n):
    return torch.randn(*n, dtype=torch.float64, device="cuda", generator=g)


def _wrap(a):
    return torch.remainder(a + math.pi, 2 * math.pi) - math.pi


def _vertex(g, n, spectrum, eta_max):
    """Production states [6, n] (x, y, z, c = q/pT, phi, theta)."""
    v = 0.01 * _randn(g, 3, n)
    u = _rand(g, n)
    if spectrum == "power2":
        pt = 1.0 / (1.0 / 0.5 - u * (1.0 / 0.5 - 1.0 / 50.0))
    elif spectrum == "mix":
        pt = torch.where(u < 0.5, 0.3, 100.0)
    else:
        pt = 0.5 + 9.5 * u
    theta = 2.0 * torch.atan(torch.exp(-_rand(g, n, -eta_max, eta_max)))
    q = torch.where(_rand(g, n) < 0.5, -1.0, 1.0).double()
    return torch.stack([v[0], v[1], v[2], q / pt, _rand(g, n, -math.pi, math.pi), theta])


def _sinc(u):
    return torch.where(u.abs() < 1e-6, 1.0 - u * u / 6.0, torch.sin(u) / torch.where(u == 0, 1.0, u))


def _at(x, y, phi, h, s):
    """Transverse position after arc length s."""
    u = 0.5 * h * s
    return x + s * torch.cos(phi + u) * _sinc(u), y + s * torch.sin(phi + u) * _sinc(u)


def _to_radius(x, y, phi, h, r, back=0.01):
    """Arc length to the outward crossing of radius r (circle intersection,
    two Newton steps after it); infinite where there is none.  A start up to
    `back` cm beyond the surface counts as before it."""
    inv = 1.0 / h
    cx, cy = x - torch.sin(phi) * inv, y + torch.cos(phi) * inv
    d = torch.hypot(cx, cy)
    a = (r * r - inv * inv + d * d) / (2.0 * d)
    disc = r * r - a * a
    hh = torch.sqrt(disc.clamp(min=0.0))
    best = torch.full_like(x, math.inf)
    for sgn in (1.0, -1.0):
        px, py = (a * cx - sgn * hh * cy) / d, (a * cy + sgn * hh * cx) / d
        al = torch.atan2((x - cx) * (py - cy) - (y - cy) * (px - cx),
                         (x - cx) * (px - cx) + (y - cy) * (py - cy))
        off = back * h.abs()
        s = (torch.remainder(torch.sign(h) * al + off, 2 * math.pi) - off) / h.abs()
        out = px * torch.cos(phi + h * s) + py * torch.sin(phi + h * s) > 0.0
        best = torch.where((disc >= 0) & out & (s < best), s, best)
    fin = torch.isfinite(best)
    s = torch.where(fin, best, 0.0)
    for _ in range(2):
        X, Y = _at(x, y, phi, h, s)
        rr = torch.hypot(X, Y)
        dr = (X * torch.cos(phi + h * s) + Y * torch.sin(phi + h * s)) / rr
        s = torch.where(dr.abs() > 1e-3, s - (rr - r) / dr, s)
    return torch.where(fin, s, math.inf)


def _cos_incidence(p, kind):
    cosa = torch.where(kind == 0, torch.sin(p[5]) * torch.cos(p[4] - torch.atan2(p[1], p[0])),
                       torch.cos(p[5]))
    return cosa.abs().clamp(min=1e-6)


def _highland(p, t):
    pm = 1.0 / (p[3].abs() * torch.sin(p[5]))
    b2 = pm * pm / (pm * pm + MASS * MASS)
    return 0.0136 / (b2.sqrt() * pm) * t.sqrt() * (1.0 + 0.038 * torch.log(t / b2))


def _simulate(g, geom, st, matmap=None):
    """Walks tracks [6, n] through the layers in the uniform field: the first
    surface reached each time, a scattering kick (and, with a map, the mean
    energy loss) there.  Returns layers [steps, n] (-1: none) and the crossing
    states [steps, 6, n]."""
    n = st.shape[1]
    dev = st.device
    nb = len(BARREL_R)
    b_r = torch.tensor(BARREL_R, dtype=torch.float64, device=dev)
    b_z = torch.tensor([L["hi"] for L in geom[:nb]], dtype=torch.float64, device=dev)
    rz = torch.tensor([L["r_or_z"] for L in geom], dtype=torch.float64, device=dev)
    kinds = torch.tensor([L["kind"] for L in geom], device=dev)
    if matmap is not None:
        mx0 = torch.as_tensor(matmap["x0"], device=dev).double()
        mxi = torch.as_tensor(matmap["xi"], device=dev).double()
    p = st.clone()
    alive = torch.ones(n, dtype=torch.bool, device=dev)
    turned = torch.zeros(n, dtype=torch.float64, device=dev)
    lay, at = [], []
    for _ in range(len(geom)):
        h = -KAPPA * BZ * p[3]
        k = torch.searchsorted(b_r, torch.hypot(p[0], p[1]) + 0.05, right=True)
        kk = k.clamp(max=nb - 1)
        s = _to_radius(p[0], p[1], p[4], h, b_r[kk], back=0.0)
        ok = (k < nb) & torch.isfinite(s) & (s > 1e-9)
        ok &= (p[2] + torch.where(ok, s, 0.0) / torch.tan(p[5])).abs() <= b_z[kk]
        best = torch.where(ok, s, math.inf)
        which = torch.where(ok, kk, -1)
        for i in range(nb, len(geom)):
            L = geom[i]
            s = (L["r_or_z"] - p[2]) * torch.tan(p[5])
            X, Y = _at(p[0], p[1], p[4], h, s)
            r = torch.hypot(X, Y)
            ok = (s > 1e-9) & (r >= L["lo"]) & (r <= L["hi"]) & (s < best)
            best = torch.where(ok, s, best)
            which = torch.where(ok, i, which)
        alive = alive & (which >= 0)
        s = torch.where(alive, best, 0.0)
        turned = turned + h.abs() * s
        alive = alive & (turned <= math.pi)
        if not bool(alive.any()):
            break
        w = which.clamp(min=0)
        X, Y = _at(p[0], p[1], p[4], h, s)
        kind = kinds[w]
        snap = torch.where(kind == 0, rz[w] / torch.hypot(X, Y), 1.0)
        Z = torch.where(kind == 1, rz[w], p[2] + s / torch.tan(p[5]))
        q = torch.stack([X * snap, Y * snap, Z, p[3], _wrap(p[4] + h * s), p[5]])
        lay.append(torch.where(alive, which, -1))
        at.append(q)
        if matmap is not None:
            ir = (torch.hypot(q[0], q[1]) * (MAP_N / MAP_R)).long().clamp(0, MAP_N - 1)
            iz = ((q[2] + MAP_Z) * (MAP_N / (2 * MAP_Z))).long().clamp(0, MAP_N - 1)
            x0, xi = mx0[ir, iz], mxi[ir, iz]
        else:
            x0 = torch.full_like(s, geom[0]["x0"])
            xi = None
        if geom[0]["x0"] > 0 or matmap is not None:
            cosa = _cos_incidence(q, kind)
            th0 = torch.where(x0 > 0, _highland(q, (x0 / cosa).clamp(min=1e-12)), 0.0)
            g1, g2 = _randn(g, n), _randn(g, n)
            pm = 1.0 / (q[3].abs() * torch.sin(q[5]))
            th = q[5] + g1 * th0
            ph = _wrap(q[4] + g2 * th0 / torch.sin(q[5]))
            c = torch.sign(q[3]) / (pm * torch.sin(th))
            if xi is not None:
                E = torch.sqrt(pm * pm + MASS * MASS)
                dE = torch.minimum(_bethe(pm) * xi / cosa * 1e-3, 0.5 * (E - MASS))
                c = c * pm / torch.sqrt((E - dE) ** 2 - MASS * MASS)
            q = torch.stack([q[0], q[1], q[2], c, ph, th])
        p = torch.where(alive, q, p)
    return torch.stack(lay), torch.stack(at)


def _bethe(p):
    """Mean ionisation loss in silicon [MeV cm^2/g] (no density effect)."""
    me, M = 0.51099895, MASS * 1e3
    E = torch.sqrt((p * 1e3) ** 2 + M * M)
    b2 = (p * 1e3 / E) ** 2
    bg2 = b2 * (E / M) ** 2
    tmax = 2 * me * bg2 / (1 + 2 * (E / M) * me / M + (me / M) ** 2)
    return 0.307075 * 0.49848 / b2 * (0.5 * torch.log(2 * me * bg2 * tmax / (173e-6) ** 2) - b2)


# ---------------------------------------------------------------- parametrised field
def _field(x, y, z):
    g = 1.0 / (1.0 + (z / FIELD_Z0) ** 2)
    k = BZ * z / FIELD_Z0 ** 2 * g * g
    return k * x, k * y, BZ * g


def _rk(p, l, step=FIELD_STEP):
    """Position and direction [3, n] each, 3D path l along the track from p
    [6, n], in ceil(|l| / step) equal fourth-order Runge-Kutta steps."""
    st = torch.sin(p[5])
    kq = KAPPA * p[3] * st
    y = [p[0], p[1], p[2], st * torch.cos(p[4]), st * torch.sin(p[4]), torch.cos(p[5])]
    n = torch.ceil(l.abs() / step)
    h = torch.where(n > 0, l / n.clamp(min=1), 0.0)

    def der(y):
        bx, by, bz = _field(y[0], y[1], y[2])
        return [y[3], y[4], y[5], kq * (y[4] * bz - y[5] * by), kq * (y[5] * bx - y[3] * bz),
                kq * (y[3] * by - y[4] * bx)]
    for i in range(int(n.max())):
        hi = torch.where(i < n, h, 0.0)
        a = der(y)
        b = der([u + 0.5 * hi * v for u, v in zip(y, a)])
        c = der([u + 0.5 * hi * v for u, v in zip(y, b)])
        d = der([u + hi * v for u, v in zip(y, c)])
        y = [u + hi / 6.0 * (e + 2 * f + 2 * k + m) for u, e, f, k, m in zip(y, a, b, c, d)]
    return torch.stack(y[:3]), torch.stack(y[3:])


def _rk_to_radius(p, r, alive):
    """State [6, n] at the outward crossing of radius r in the field, its 3D
    path, and where it exists."""
    h = -KAPPA * _field(p[0], p[1], p[2])[2] * p[3]
    s = _to_radius(p[0], p[1], p[4], h, r)
    ok = alive & torch.isfinite(s)
    l = torch.where(ok, s / torch.sin(p[5]), 0.0)
    ok &= l < 1000.0
    l = torch.where(ok, l, 0.0)
    for k in range(5):
        y, t = _rk(p, l)
        rr = torch.hypot(y[0], y[1])
        dr = (y[0] * t[0] + y[1] * t[1]) / rr.clamp(min=1e-9)
        if k < 4:
            l = torch.where(ok & (dr > 1e-3), l - (rr - r) / dr, l)
    ok = ok & ((rr - r).abs() < 1e-6)
    th = torch.atan2(torch.hypot(t[0], t[1]), t[2])
    q = torch.stack([y[0], y[1], y[2], p[3] * torch.sin(p[5]) / torch.sin(th),
                     torch.atan2(t[1], t[0]), th])
    return q, l, ok


def _simulate_field(geom, st):
    """Crossings of the barrels in order, in the parametrised field."""
    p = st.clone()
    alive = torch.ones(st.shape[1], dtype=torch.bool, device=st.device)
    lay, at = [], []
    for i, L in enumerate(geom):
        q, _, ok = _rk_to_radius(p, torch.full_like(p[0], L["r_or_z"]), alive)
        alive = ok & (q[2].abs() <= L["hi"])
        lay.append(torch.where(alive, i, -1))
        at.append(q)
        p = torch.where(alive, q, p)
    return torch.stack(lay), torch.stack(at)


# ---------------------------------------------------------------- hits
def _smear(g, geom, lay, at, su, sv):
    """Hits [x, y, z] of crossings with layers lay and states at [6, ...]."""
    kind = torch.tensor([L["kind"] for L in geom], device=lay.device)[lay.clamp(min=0)]
    r = torch.hypot(at[0], at[1])
    ph = torch.atan2(at[1], at[0]) + _randn(g, *lay.shape) * su / r
    dv = _randn(g, *lay.shape) * sv
    rh = torch.where(kind == 0, r, r + dv)
    return torch.stack([rh * torch.cos(ph), rh * torch.sin(ph),
                        torch.where(kind == 0, at[2] + dv, at[2])])


def _noise(g, geom, per_event):
    """Uniform noise hits [3, m] with their layers and events; per_event: hits
    per layer of each event."""
    nl = len(geom)
    cnt = torch.as_tensor(np.repeat(per_event, nl), device="cuda")
    seg = torch.repeat_interleave(torch.arange(cnt.numel(), device="cuda"), cnt)
    ev, lay = seg // nl, seg % nl
    col = lambda k: torch.tensor([float(L[k]) for L in geom], dtype=torch.float64, device="cuda")[lay]
    m = seg.numel()
    ph, u = _rand(g, m, -math.pi, math.pi), _rand(g, m)
    lo, hi, rz, barrel = col("lo"), col("hi"), col("r_or_z"), col("kind") == 0
    r = torch.where(barrel, rz, torch.sqrt((lo * lo + u * (hi * hi - lo * lo)).clamp(min=0)))
    z = torch.where(barrel, lo + u * (hi - lo), rz)
    return torch.stack([r * torch.cos(ph), r * torch.sin(ph), z]), lay, ev


def _multiplicities(case, seed):
    """Tracks of each event: all alike, or spread over 0.1 to 1.9 of the mean
    (the same total for every seed)."""
    e, t = case["events"], case["tracks"]
    if not case["uneven"]:
        return np.full(e, t, np.int64)
    n = np.maximum(1, np.round(t * (0.1 + 1.8 * (np.arange(e) + 0.5) / e))).astype(np.int64)
    return np.random.default_rng(seed).permutation(n)


def _find_inputs(case, seed):
    g = _gen(seed)
    n_e = _multiplicities(case, seed)
    geom = _geometry(case["disks"], 0.0 if case["map"] or case["field"] else 0.02)
    matmap = _material_map(geom) if case["map"] else None
    n = int(n_e.sum())
    te = torch.repeat_interleave(torch.arange(len(n_e), device="cuda"),
                                 torch.as_tensor(n_e, device="cuda"))
    st = _vertex(g, n, "uniform" if case["field"] else "power2", 2.5 if case["disks"] else 1.0)
    lay, at = _simulate_field(geom, st) if case["field"] else _simulate(g, geom, st, matmap)
    steps = lay.shape[0]
    pos = _smear(g, geom, lay, at.transpose(0, 1), SIG_U, SIG_V)            # [3, steps, n]
    have = lay >= 0
    parts = [(pos[:, have], lay[have], te.expand(steps, n)[have])]
    dup = None
    if case["overlap"]:
        # module overlaps: a second measurement on the first three crossings
        kind = torch.tensor([L["kind"] for L in geom], device="cuda")[lay[:3].clamp(min=0)]
        dup = have[:3] & (_rand(g, 3 * n).view(3, n) < torch.where(kind == 0, 0.1, 0.3))
        pos2 = _smear(g, geom, lay[:3], at[:3].transpose(0, 1), SIG_U, SIG_V)
        parts.append((pos2[:, dup], lay[:3][dup], te.expand(3, n)[dup]))
    parts.append(_noise(g, geom, case["noise"] * n_e // len(geom)))
    xyz = torch.cat([a[0] for a in parts], dim=1)
    hl, he = torch.cat([a[1] for a in parts]), torch.cat([a[2] for a in parts])
    perm = torch.argsort(he.double() + 0.999 * _rand(g, he.numel()))       # shuffled within events
    inv = torch.empty_like(perm)
    inv[perm] = torch.arange(perm.numel(), device="cuda")
    hit = torch.full(lay.shape, -1, dtype=torch.int64, device="cuda")
    n_sig = int(have.sum())
    hit[have] = inv[:n_sig]
    # one seed per combination of the hits on a track's first three crossings
    first = [hit[:3]]
    if dup is not None:
        second = torch.full((3, n), -1, dtype=torch.int64, device="cuda")
        second[dup] = inv[n_sig:n_sig + int(dup.sum())]
        first.append(second)
    combos = [torch.stack([first[(c >> k) & 1][k] for k in range(3)])
              for c in range(8 if dup is not None else 1)]
    sh = torch.stack(combos, dim=2)                                        # [3, n, combos]
    keep = (sh >= 0).all(dim=0) & have[2][:, None]
    # as many seeds for every seed of the generator: a part left out at random
    want = int((1.5 if dup is not None else 0.93) * n)
    ks = torch.nonzero(keep.reshape(-1))[:, 0]
    ks = ks[torch.randperm(ks.numel(), device="cuda", generator=g)]
    ks = ks[torch.arange(want, device="cuda") % ks.numel()].sort().values
    pick = lambda v: v.reshape(v.shape[0], -1)[:, ks]
    sl = lay[:3, :, None].expand_as(sh)
    off = np.concatenate([[0], np.cumsum(torch.bincount(he, minlength=len(n_e)).cpu().numpy())])
    xyz = xyz[:, perm].float()
    m = perm.numel()
    inp = dict(x=xyz[0], y=xyz[1], z=xyz[2], su=torch.full((m,), SIG_U, device="cuda"),
               sv=torch.full((m,), SIG_V, device="cuda"), layer=hl[perm].int(), event_off=off,
               seed_hits=pick(sh).T.cpu().numpy().astype(np.int32),
               seed_layers=pick(sl).T.cpu().numpy().astype(np.int32),
               seed_event=te[ks // keep.shape[1]].cpu().numpy().astype(np.int32))
    return geom, matmap, inp


def _fit_inputs(case, seed):
    """Hits (step-major, or in shuffled order) and each track's layers and hit
    indices by step [steps, ld]."""
    g = _gen(seed)
    n = case["tracks"]
    ld = K.round_ld(n)
    geom = _geometry(case["disks"], 0.02 if case["disks"] else 0.0)
    steps = len(BARREL_R) if not case["disks"] else 14
    lseq = torch.full((steps, ld), -1, dtype=torch.int32, device="cuda")
    xyz = torch.zeros((3, steps, ld), dtype=torch.float32, device="cuda")
    su = torch.full((steps, ld), SIG_U, dtype=torch.float32, device="cuda")
    for a in range(0, n, 500_000):
        b = min(n, a + 500_000)
        st = _vertex(g, b - a, "mix" if case["mix"] else "uniform", 2.5 if case["disks"] else 1.0)
        lay, at = _simulate_field(geom, st) if case["field"] else _simulate(g, geom, st)
        lay, at = lay[:steps], at[:steps]
        s = torch.full(lay.shape, SIG_U, dtype=torch.float64, device="cuda")
        if case["mix"]:
            s = torch.exp(_rand(g, lay.numel(), math.log(0.002), math.log(0.01))).view(lay.shape)
        k = lay.shape[0]
        xyz[:, :k, a:b] = _smear(g, geom, lay, at.transpose(0, 1), s, 5 * s).float()
        su[:k, a:b] = s.float()
        lseq[:k, a:b] = lay.int()
    idx = torch.arange(steps * ld, device="cuda")
    if case["shuffled"]:
        perm = torch.randperm(steps * ld, device="cuda", generator=g)
        idx[perm] = idx.clone()
        flat = lambda v: v.reshape(-1)[perm]
    else:
        flat = lambda v: v.reshape(-1)
    idx = torch.where(lseq >= 0, idx.view(steps, ld).int(), -1)
    sv = 5 * su
    hits = (flat(xyz[0]), flat(xyz[1]), flat(xyz[2]), flat(su), flat(sv), flat(lseq.clamp(min=0)))
    return geom, ld, hits, lseq, idx


# ---------------------------------------------------------------- learned start
def _features(p, r):
    """The network's inputs [8, n] for barrel radius r, and its target."""
    x, y, z, c, phi, th = p
    h = -KAPPA * BZ * c
    rho = torch.hypot(x, y)
    sn, cs = (x * torch.sin(phi) - y * torch.cos(phi)) / rho, (x * torch.cos(phi) + y * torch.sin(phi)) / rho
    pu = rho * cs
    line = -pu + torch.sqrt((pu * pu - rho * rho + r * r).clamp(min=0.0))
    s = _to_radius(x, y, phi, h, r)
    f = torch.stack([rho / 100, sn, cs, h * r, r / 100, line / 100, 1.0 / torch.tan(th), z / 100])
    return f, (s - line) / (h * line * line), torch.isfinite(s)


def _pairs(g, n):
    """Inputs [8, m] and targets [m] of propagations of the fit throughput
    set, shuffled."""
    geom = _geometry(False, 0.0)
    st = _vertex(g, max(1000, n // 5), "mix", 1.0)
    lay, at = _simulate(g, geom, st)
    fs, ts = [], []
    p = st
    for k in range(lay.shape[0]):
        f, t, ok = _features(p, torch.full_like(p[0], BARREL_R[k]))
        ok &= lay[k] >= 0
        fs.append(f[:, ok])
        ts.append(t[ok])
        p = at[k]
    f, t = torch.cat(fs, dim=1), torch.cat(ts)
    sel = torch.randperm(t.numel(), device="cuda", generator=g)[:n]
    return f[:, sel].float().contiguous(), t[sel].float().contiguous()


def _net_init(seed):
    rng = np.random.default_rng(seed)
    u = lambda fi, fo, s: rng.uniform(-math.sqrt(6 / (fi + fo)), math.sqrt(6 / (fi + fo)), s)
    return np.concatenate([u(8, 64, 512), np.zeros(64), u(64, 64, 4096), np.zeros(64),
                           u(64, 1, 64), np.zeros(1)]).astype(np.float32)


def _net(w, x):
    """Outputs [n] of the network with flat weights w for inputs x [n, 8]."""
    h = torch.tanh((x[:, None, :] * w[:512].view(64, 8)).sum(-1) + w[512:576])
    h = torch.tanh((h[:, None, :] * w[576:4672].view(64, 64)).sum(-1) + w[4672:4736])
    return (h * w[4736:4800]).sum(-1) + w[4800]


@functools.lru_cache(maxsize=1)
def _trained():
    """Weights of a network trained on such pairs (made once, as a program
    loads its trained weights)."""
    g = _gen(77)
    f, t = _pairs(g, 300_000)
    w = torch.as_tensor(_net_init(4), device="cuda").requires_grad_()
    opt = torch.optim.Adam([w], lr=2e-3)
    for k in range(400):
        a = (k * 1024) % (t.numel() - 1024)
        loss = (_net(w, f[:, a:a + 1024].T) - t[a:a + 1024]).square().mean()
        opt.zero_grad()
        loss.backward()
        opt.step()
    return w.detach().cpu().numpy()


# ---------------------------------------------------------------- the cases
def prepare(case, seed):
    if case["kind"] == "find":
        geom, matmap, inp = _find_inputs(case, seed)
        ctx = K.Context(geom, field_z0=FIELD_Z0 if case["field"] else 0.0, field_step=FIELD_STEP)
        if matmap is not None:
            ctx.set_material(matmap)
        if case["steer"]:
            ctx.set_steering(_plans(geom))
        flags = K.CLEAN_SEEDS | K.REMOVE_DUPLICATES if case["overlap"] else 0
        return dict(kind="find", graph=case["graph"], flags=flags,
                    problem=pipeline.FindProblem(ctx, inp))
    if case["kind"] == "fit":
        geom, ld, hits, lseq, idx = _fit_inputs(case, seed)
        ctx = K.Context(geom, field_z0=FIELD_Z0 if case["field"] else 0.0, field_step=FIELD_STEP)
        prec = PREC[case["prec"]]
        flags = prec | (K.PER_LAYER if case["per_layer"] else 0)
        if case["learned"]:
            ctx.mlp_load(_trained())
            flags |= K.INIT_MLP
        return dict(kind="fit", ctx=ctx, hits=K.Hits(*hits), lseq=lseq, idx=idx,
                    seed_hits=idx[:3].contiguous(), steps=lseq.shape[0], prec=prec, flags=flags,
                    tracks=K.Tracks(case["tracks"], ld, prec))
    g = _gen(seed)
    f, t = _pairs(g, case["rows"])
    ctx = K.Context(_geometry(False, 0.0))
    rows = torch.randint(t.numel(), (case["steps"] * case["batch"],), device="cuda", generator=g)
    return dict(kind="train", ctx=ctx, w0=_net_init(seed), feats=f, target=t, n=t.numel(),
                rows=rows.int(), batch=case["batch"], steps=case["steps"],
                loss=torch.zeros(case["steps"], device="cuda"))


def run(state):
    if state["kind"] == "find":
        fp = state["problem"]
        if state["graph"]:
            fp.run_batched(state["flags"])
        else:
            fp.run(state["flags"])
        o = fp.out
        return dict(hits=fp.out_hits, par=o.par, cov=o.cov, chi2=o.chi2, ndf=o.ndf,
                    status=o.status, seed_par=fp.seeds.par, seed_status=fp.seeds.status)
    if state["kind"] == "fit":
        ctx, t = state["ctx"], state["tracks"]
        ctx.seed(state["hits"], state["seed_hits"], t, state["prec"])
        ctx.fit(t, state["hits"], state["lseq"], state["idx"], state["steps"], state["flags"])
        return dict(par=t.par, cov=t.cov, chi2=t.chi2, ndf=t.ndf, status=t.status)
    ctx = state["ctx"]
    ctx.mlp_load(state["w0"])
    ctx.mlp_train(state["feats"], state["target"], state["n"], state["rows"], state["batch"],
                  state["steps"], loss=state["loss"])
    return dict(loss=state["loss"], weights=ctx.mlp_get())


def work(case):
    """Bytes: every input read once, every output written once.  Operations:
    those of the method for these numbers of propagations and updates."""
    if case["kind"] == "find":
        nl = 24 if case["disks"] else 10
        tracks = case["events"] * case["tracks"]
        seeds = tracks * (1.5 if case["overlap"] else 0.93)
        hits = tracks * (case["noise"] + 8)
        par = 27 * 4 + 12
        return dict(bytes=24 * hits + seeds * (28 + 2 * par + 4 * nl),
                    flops=seeds * (70e3 if case["field"] else 30e3))
    if case["kind"] == "fit":
        n, w = case["tracks"], 8 if case["prec"] == "fp64" else 4
        steps = 8.4 if case["mix"] else 9.9
        state = n * (28 * w + 8)
        moved = state * (2 * steps if case["per_layer"] else 1)
        return dict(bytes=moved + n * steps * 28, flops=n * steps * (4.1e3 if case["field"] else 1.1e3))
    return dict(bytes=case["steps"] * case["batch"] * 40 + 3 * 4801 * 4,
                flops=case["steps"] * case["batch"] * 3 * 2 * 4672)


# ---------------------------------------------------------------- exact values
def _pack():
    return [(i, j) for i in range(6) for j in range(i, 6)]


def _exact_seed(h, sh):
    """Circle through three hits [3 coordinates, 3 hits, n]: state at the first."""
    (x1, x2, x3), (y1, y2, y3), (z1, _, z3) = h
    ax, ay, bx, by = x2 - x1, y2 - y1, x3 - x1, y3 - y1
    d13 = torch.hypot(bx, by)
    hc = 2 * (ax * by - ay * bx) / (torch.hypot(ax, ay) * torch.hypot(x3 - x2, y3 - y2) * d13)
    w = (0.5 * hc * d13).clamp(-1, 1)
    s = torch.where(w.abs() < 1e-4, d13 * (1 + w * w / 6), d13 * torch.asin(w) / torch.where(w == 0, 1.0, w))
    p = torch.stack([x1, y1, z1, -hc / (KAPPA * BZ), _wrap(torch.atan2(by, bx) - 0.5 * hc * s),
                     torch.atan2(s, z3 - z1)])
    P = torch.diag(torch.tensor([1, 1, 1, 4, 0.01, 0.01], dtype=torch.float64, device="cuda"))
    return p, P.expand(p.shape[1], 6, 6).clone()


def _jacobian(p, s, h_per_c, kind, zd):
    """F [n, 6, 6] of the helix transport by arc length s to a surface."""
    x, y, z, c, phi, th = p
    h = h_per_c * c
    u = 0.5 * h * s
    sc = _sinc(u)
    dsc = torch.where(u.abs() < 0.05, u * (-1 / 3 + u * u * (1 / 30 - u * u / 840)),
                      (u * torch.cos(u) - torch.sin(u)) / torch.where(u == 0, 1.0, u * u))
    ca, sa = torch.cos(phi + u), torch.sin(phi + u)
    X, Y = x + s * ca * sc, y + s * sa * sc
    f = torch.zeros(6, p.shape[1], dtype=torch.float64, device="cuda")
    f[0], f[1], f[2], f[4] = torch.cos(phi + h * s), torch.sin(phi + h * s), 1 / torch.tan(th), h
    D = torch.eye(6, dtype=torch.float64, device="cuda").expand(p.shape[1], 6, 6).clone()
    D[:, 0, 3] = h_per_c * 0.5 * s * s * (ca * dsc - sa * sc)
    D[:, 1, 3] = h_per_c * 0.5 * s * s * (sa * dsc + ca * sc)
    D[:, 0, 4], D[:, 1, 4] = -s * sa * sc, s * ca * sc
    D[:, 4, 3], D[:, 2, 5] = h_per_c * s, -s / torch.sin(th) ** 2
    d = torch.zeros_like(f)
    den = -1 / (X * f[0] + Y * f[1])
    barrel = kind == 0
    for k, v in ((0, X * den), (1, Y * den), (3, (X * D[:, 0, 3] + Y * D[:, 1, 3]) * den),
                 (4, (X * D[:, 0, 4] + Y * D[:, 1, 4]) * den)):
        d[k] = torch.where(barrel, v, 0.0)
    d[2] = torch.where(barrel, 0.0, -torch.tan(th))
    d[5] = torch.where(barrel, 0.0, (zd - z) / torch.cos(th) ** 2)
    return D + f.T[:, :, None] * d.T[:, None, :]


def _effective_bz(x, y, z, phi, th):
    bx, by, bz = _field(x, y, z)
    return bz - (bx * torch.cos(phi) + by * torch.sin(phi)) / torch.tan(th)


def _exact_fit(case, seed):
    geom, ld, hits, lseq, idx = _fit_inputs(case, seed)
    n, steps = case["tracks"], lseq.shape[0]
    kinds = torch.tensor([L["kind"] for L in geom], device="cuda")
    rz = torch.tensor([L["r_or_z"] for L in geom], dtype=torch.float64, device="cuda")
    x0 = geom[0]["x0"]
    par = torch.zeros((6, ld), dtype=torch.float64, device="cuda")
    cov = torch.zeros((21, ld), dtype=torch.float64, device="cuda")
    chi = torch.zeros(ld, dtype=torch.float64, device="cuda")
    eye = torch.eye(6, dtype=torch.float64, device="cuda")
    for a in range(0, n, 500_000):
        b = min(n, a + 500_000)
        ii, ll = idx[:, a:b].long(), lseq[:, a:b].long()
        good = (ii[:3] >= 0).all(0)
        p, P = _exact_seed([hits[k].double()[ii[:3].clamp(min=0)] for k in range(3)], None)
        c2 = torch.zeros(b - a, dtype=torch.float64, device="cuda")
        alive = good.clone()
        for k in range(steps):
            l = ll[k]
            alive = alive & (l >= 0)
            kind, R = kinds[l.clamp(min=0)], rz[l.clamp(min=0)]
            if case["field"]:
                q, path, ok = _rk_to_radius(p, R, alive)
                mid = [0.5 * (p[j] + q[j]) for j in range(6)]
                mid[4] = p[4] + 0.5 * _wrap(q[4] - p[4])
                be = (_effective_bz(*p[[0, 1, 2, 4, 5]]) + _effective_bz(*q[[0, 1, 2, 4, 5]])
                      + 4 * _effective_bz(mid[0], mid[1], mid[2], mid[4], mid[5])) / 6
                s, hc = path * torch.sin(p[5]), -KAPPA * be
            else:
                hc = torch.full_like(R, -KAPPA * BZ)
                s = torch.where(kind == 0, _to_radius(p[0], p[1], p[4], hc * p[3], R),
                                (R - p[2]) * torch.tan(p[5]))
                ok = alive & torch.isfinite(s) & ((kind == 0) | (s >= 0))
                s = torch.where(ok, s, 0.0)
                X, Y = _at(p[0], p[1], p[4], hc * p[3], s)
                q = torch.stack([X, Y, p[2] + s / torch.tan(p[5]), p[3], _wrap(p[4] + hc * p[3] * s), p[5]])
            alive = ok
            F = _jacobian(p, s, hc, kind, R)
            Q = F @ P @ F.transpose(1, 2).contiguous()
            if x0 > 0:
                t2 = _highland(q, x0 / _cos_incidence(q, kind)) ** 2
                cot = 1 / torch.tan(q[5])
                Q[:, 4, 4] += t2 / torch.sin(q[5]) ** 2
                Q[:, 5, 5] += t2
                Q[:, 3, 5] -= q[3] * cot * t2
                Q[:, 5, 3] -= q[3] * cot * t2
                Q[:, 3, 3] += (q[3] * cot) ** 2 * t2
            i = ii[k].clamp(min=0)
            hx, hy, hz, su, sv = (hits[j][i].double() for j in range(5))
            rho = torch.hypot(hx, hy)
            c, s_ = hx / rho, hy / rho
            z = torch.zeros_like(c)
            H = torch.stack([torch.stack([-s_, c, z, z, z, z], 1),
                             torch.where((kind == 0)[:, None], torch.stack([z, z, z + 1, z, z, z], 1),
                                         torch.stack([c, s_, z, z, z, z], 1))], 1)
            res = (H[:, :, :3] * torch.stack([hx - q[0], hy - q[1], hz - q[2]], 1)[:, None, :]).sum(2)
            B = Q @ H.transpose(1, 2).contiguous()
            V = torch.diag_embed(torch.stack([su, sv], 1) ** 2)
            S = H @ B + V
            det = S[:, 0, 0] * S[:, 1, 1] - S[:, 0, 1] * S[:, 1, 0]
            Si = torch.stack([torch.stack([S[:, 1, 1], -S[:, 0, 1]], 1),
                              torch.stack([-S[:, 1, 0], S[:, 0, 0]], 1)], 1) / det[:, None, None]
            G = B @ Si
            J = eye - G @ H
            Pn = J @ Q @ J.transpose(1, 2).contiguous() + G @ V @ G.transpose(1, 2).contiguous()
            pn = q + (G @ res[:, :, None])[:, :, 0].T
            pn[4] = _wrap(pn[4])
            p = torch.where(alive, pn, p)
            P = torch.where(alive[:, None, None], Pn, P)
            c2 = torch.where(alive, c2 + (res * (Si @ res[:, :, None])[:, :, 0]).sum(1), c2)
        par[:, a:b] = torch.where(good, p, 0.0)
        cov[:, a:b] = torch.where(good, torch.stack([P[:, i, j] for i, j in _pack()]), 0.0)
        chi[a:b] = torch.where(good, c2, 0.0)
    return dict(par=par, cov=cov, chi2=chi, ndf=None, status=None)


def _exact_train(case, seed):
    """Adam on the network whose products take the weights rounded to bf16."""
    g = _gen(seed)
    f, t = _pairs(g, case["rows"])
    rows = torch.randint(t.numel(), (case["steps"] * case["batch"],), device="cuda", generator=g)
    w = torch.as_tensor(_net_init(seed), device="cuda").double()
    m, v, loss = torch.zeros_like(w), torch.zeros_like(w), []
    x, t = f.T.double(), t.double()
    for k in range(case["steps"]):
        r = rows[k * case["batch"]:(k + 1) * case["batch"]]
        wb = w.bfloat16().double().requires_grad_()
        e = (_net(wb, x[r]) - t[r]).square().mean()
        gw, = torch.autograd.grad(e, wb)
        loss.append(e.detach())
        m, v = 0.9 * m + 0.1 * gw, 0.999 * v + 0.001 * gw * gw
        w = w - 1e-3 * (m / (1 - 0.9 ** (k + 1))) / (torch.sqrt(v / (1 - 0.999 ** (k + 1))) + 1e-8)
    return dict(loss=torch.stack(loss), weights=w)


def exact(case, seed):
    """The fits and the training in 64 bits.  A finding pass has no such
    value: what it returns hangs on its hit decisions."""
    if case["kind"] == "fit":
        return _exact_fit(case, seed)
    if case["kind"] == "train":
        return _exact_train(case, seed)
    return None
