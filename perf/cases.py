"""The work that users have this package do, as cases that can be timed.

A case is a dict of plain values. `prepare` puts on the GPU what a program
has in hand before the call (patterns made from the seed, the resident
template library), `run` is one pass through the public entry points,
`exact` the same outputs in 64 bits from plain torch, `work` the bytes and
operations that one pass cannot do without.

Kinds of work
  index       polar transform of a batch of patterns and the search of a
              template library (Section 2.2 of the paper), by the route a
              program chooses: "plain" (every template scored exactly),
              "bound" (exact search with window bounds), "fft" (Fourier
              route, certified rescoring), "fp32" / "bf16" / "fp16" / "fp8"
              (pre-filter in that precision), "maps" (the plain search with
              every template's best score and angle returned as well).
  two_stage   the second phase of a two-phase scan (Section 4.3): mask of the
              dominant phase from the scan's mean, masked polar transform,
              search with unit template intensities.
  preprocess  centring, difference of Gaussians, blur, threshold (Section 4.1).
  simulate    the kinematical template library (Section 2.1).

Libraries and patterns follow the sizes of this repository's workloads: FCC,
orthorhombic and HCP crystals at 200 kV, Gaussian spots, a bright direct
beam, float32 patterns with background and noise or uint16 Poisson counts.
"""
import functools
import math

import numpy as np
import torch

import paper_2111_07347_amd as tm

DEV = "cuda:0"
K0 = 1.0 / 0.025079340           # 1 / wavelength at 200 kV, 1/Angstrom
G_MAX, S_MAX, REL_MIN = 1.2, 0.05, 1e-3
MEAN_SPOTS = {"fcc": 7, "hcp": 13, "ortho": 76}
EXACT_PAIRS = 2e7                # (pattern, template) pairs exact() scores in a few seconds


# ------------------------------------------------------------------ the cases
def _index(name, phase, T, B, H, W, route, dtype="f32", n_theta=360, N=5, R=None, max_spots=120,
           compact=True, angles=False, gamma=1.0, keep=0.1):
    c = dict(kind="index", phase=phase, T=T, B=B, H=H, W=W, route=route, dtype=dtype,
             n_theta=n_theta, N=N, R=R or min(H, W) // 2, max_spots=max_spots, compact=compact,
             angles=angles, gamma=gamma, keep=keep)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # a small map at reduced detector size, as a first look at a data set
        _index("fcc300_64", "fcc", 300, 64, 128, 128, "plain", max_spots=30, compact=False),
        # one pattern at the microscope or in a notebook, orientation and all: latency
        _index("ortho20000_1", "ortho", 20000, 1, 256, 256, "bound", angles=True),
        # a row of a scan streamed from the detector, small library, every template scored
        _index("fcc2000_row256_u16", "fcc", 2000, 256, 256, 256, "plain", "u16", max_spots=100),
        # the same row against the large library
        _index("ortho20000_row256_u16", "ortho", 20000, 256, 256, 256, "bound", "u16"),
        # a whole 128 x 128 scan resident in memory, large library: the benchmark's workload
        _index("ortho20000_scan16384", "ortho", 20000, 16384, 256, 256, "bound"),
        # a whole scan, paper-scale library, every template scored
        _index("fcc2000_scan16384", "fcc", 2000, 16384, 256, 256, "plain", max_spots=100),
        # correlation maps of all templates, ragged detector crop, 2 degree steps
        _index("hcp8000_maps200", "hcp", 8000, 200, 243, 251, "maps", "u16", n_theta=180),
        # pre-filter of the library by radial profiles, then exact scores of the kept tenth
        _index("ortho20000_bf16_1024", "ortho", 20000, 1024, 256, 256, "bf16"),
        # Fourier route over a part of a scan
        _index("hcp8000_fft512", "hcp", 8000, 512, 256, 256, "fft"),
        # second phase of a two-phase scan, dominant phase masked
        dict(name="two_stage_4096", kind="two_stage", T=2000, B=4096, H=256, W=256, N=5),
        # raw counts cleaned before indexing
        dict(name="preprocess_1024_u16", kind="preprocess", B=1024, H=256, W=256, dtype="u16",
             r_box=8, sigma_min=1.0, sigma_max=6.0, sigma_blur=1.0),
        # a library simulated for new orientations
        dict(name="simulate_ortho50000", kind="simulate", phase="ortho", T=50000, max_spots=120),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["index", "two_stage", "preprocess", "simulate"], [9, 1, 1, 1])[0]
    if kind == "simulate":
        return dict(kind=kind, phase=rng.choice(["fcc", "hcp", "ortho"]), T=_log(rng, 200, 100000),
                    max_spots=rng.choice([30, 100, 120, 150]))
    H, W = (rng.choice([rng.randint(96, 300), 128, 256]) for _ in range(2))
    if kind == "preprocess":
        return dict(kind=kind, B=_log(rng, 1, 4096), H=H, W=W, dtype=rng.choice(["u16", "f32"]),
                    r_box=rng.choice([4, 8, 12]), sigma_min=rng.choice([0.5, 1.0, 1.5]),
                    sigma_max=rng.choice([3.0, 6.0, 8.0]), sigma_blur=rng.choice([0.0, 1.0, 2.0]))
    if kind == "two_stage":
        return dict(kind=kind, T=_log(rng, 300, 3000), B=_log(rng, 16, 8192), H=H, W=W,
                    N=rng.randint(1, 10))
    phase, N = rng.choice(["fcc", "hcp", "ortho"]), rng.randint(1, 10)
    R = min(H, W) // 2
    route = rng.choice(["plain", "plain", "bound", "bound", "bound", "maps", "fft",
                        rng.choice(["fp32", "bf16", "fp16", "fp8"])])
    n_theta = rng.choice([90, 180, 180, 360, 360, 360, 360, rng.randint(90, 240), 720])
    if route == "fft":
        n_theta -= n_theta % 2
    if route == "bound" and (R + 1) * (2 * -(-n_theta // 4) + 1) * 4 > 128 * 1024:
        n_theta = 180            # the window image of a larger grid does not fit
    T = _log(rng, 100, 20000)
    # the most patterns that cost no more than the largest listed case
    pairs = {"bound": 16384 * 20000, "maps": 2e6, "fft": 8e6}.get(
        route, 16384 * 2000 * 7 * 360 / (MEAN_SPOTS[phase] * n_theta) * (1 if route == "plain" else 2))
    B = _log(rng, 1, max(2, min(16384, pairs / T)))
    return _index(None, phase, T, B, H, W, route, rng.choice(["f32", "u16"]), n_theta, N, R,
                  rng.choice([100, 120, 150]), rng.random() < 0.8, rng.random() < 0.25,
                  rng.choice([1.0, 1.0, 0.5]), rng.choice([0.05, 0.1, 0.2]))


# ------------------------------------------------- crystals, templates, patterns
def _crystal(phase):
    """Reciprocal basis (rows, 1/Angstrom) and fractional atom positions."""
    if phase == "hcp":
        a, c = 2.95, 2.95 * 1.59
        A = np.array([[a, 0, 0], [-0.5 * a, math.sqrt(3.0) / 2.0 * a, 0], [0, 0, c]])
        X = np.array([[0, 0, 0], [1 / 3, 2 / 3, 0.5]])
    elif phase == "fcc":
        A = np.diag([4.05] * 3)
        X = np.array([[0, 0, 0], [0.5, 0.5, 0], [0.5, 0, 0.5], [0, 0.5, 0.5]])
    else:
        A, X = np.diag([5.1, 7.3, 4.6]), np.zeros((1, 3))
    return np.linalg.inv(A).T, X


def _spiral(phase, T):
    """(Phi, phi2) of T directions spread over the crystal's symmetry sector."""
    n = 64 * T
    i = np.arange(n)
    z = 1.0 - (2.0 * i + 1.0) / n
    r, az = np.sqrt(1.0 - z * z), i * math.pi * (3.0 - math.sqrt(5.0))
    x, y = r * np.cos(az), r * np.sin(az)
    ok = {"fcc": (z >= x) & (x >= y) & (y >= 0), "ortho": (x >= 0) & (y >= 0) & (z >= 0),
          "hcp": (z >= 0) & (y >= 0) & (y <= x * math.tan(math.pi / 6))}[phase]
    at = np.nonzero(ok)[0]
    at = at[np.linspace(0, len(at) - 1, T).round().astype(np.int64)]
    return np.stack([np.arccos(z[at]), np.arctan2(x[at], y[at])], 1)


def _templates(phase, euler, max_spots):
    """Kinematical templates (Section 2.1) in 64 bits: kx, ky, intensity
    [T, max_spots] (0 past a template's count) and count [T]."""
    Bm, X = _crystal(phase)
    lims = [int(math.ceil((G_MAX + 0.2) * np.linalg.norm(a))) + 1 for a in np.linalg.inv(Bm).T]
    hkl = np.stack(np.meshgrid(*[np.arange(-m, m + 1) for m in lims], indexing="ij"), -1).reshape(-1, 3)
    hkl = hkl[np.any(hkl != 0, axis=1)]
    g = hkl @ Bm
    F2 = np.abs(np.exp(2j * math.pi * (hkl @ X.T)).sum(1)) ** 2
    ok = (np.linalg.norm(g, axis=1) <= G_MAX + 0.2) & (F2 > 1e-6)
    hx, hy, hz = (torch.from_numpy(np.ascontiguousarray(v)).to(DEV)[None] for v in g[ok].T)
    F2 = torch.from_numpy(F2[ok]).to(DEV)[None]
    outs = []
    for e in torch.split(euler, 4096):
        c, s, c2, s2 = e[:, :1].cos(), e[:, :1].sin(), e[:, 1:].cos(), e[:, 1:].sin()
        gx = c2 * hx - s2 * hy
        gy = s2 * c * hx + c2 * c * hy - s * hz
        gz = s2 * s * hx + c2 * s * hy + c * hz
        err = K0 - (gx * gx + gy * gy + (gz - K0) ** 2).sqrt()
        shape = (1.0 - err.abs() / S_MAX).clamp_min(0.0)
        inten = torch.where((gx * gx + gy * gy).sqrt() <= G_MAX, F2 * shape, 0.0)
        top = inten.amax(1, keepdim=True)
        inten = torch.where(inten >= REL_MIN * top, inten, 0.0)
        inten, at = torch.sort(inten, dim=1, descending=True, stable=True)
        inten, at = inten[:, :max_spots], at[:, :max_spots]
        live = inten > 0
        pad = max(0, max_spots - inten.shape[1])
        outs.append([torch.nn.functional.pad(torch.where(live, v, 0.0), (0, pad))
                     for v in (gx.gather(1, at), gy.gather(1, at), inten / top.clamp_min(1e-300))]
                    + [live.sum(1, dtype=torch.int32)])
    return [torch.cat(v) for v in zip(*outs)]


def _grid(c):
    return tm.PolarGrid(R=c["R"], n_theta=c["n_theta"], cx=c["W"] / 2.0, cy=c["H"] / 2.0)


def _px(R):
    return (R - 4) / G_MAX


@functools.lru_cache(maxsize=2)
def _spots(phase, T, max_spots):
    """Templates spread over the sector, on the device, and their (Phi, phi2)."""
    euler = torch.from_numpy(_spiral(phase, T)).to(DEV)
    return _templates(phase, euler, max_spots), euler


@functools.lru_cache(maxsize=2)
def _library(phase, T, max_spots, R, n_theta, unit, fft):
    """The library a program loads once and indexes many scans with."""
    kx, ky, inten, cnt = _spots(phase, T, max_spots)[0]
    off = np.zeros(T + 1, np.int64)
    off[1:] = np.cumsum(cnt.cpu().numpy())
    live = (torch.arange(max_spots, device=DEV)[None] < cnt[:, None])
    host = [v[live].cpu().numpy() for v in (kx, ky, inten)]
    return tm.Library(*host, off, _px(R), tm.PolarGrid(R=R, n_theta=n_theta), unit_intensity=unit,
                      fft=fft)


def _patterns(spots, B, H, W, R, dtype, gen, shift=0.0, weak=1.0, common=None, diffuse=0.0):
    """Patterns of randomly chosen templates at random in-plane angles, half
    of them mirrored: Gaussian spots (sigma 1.5 px) and a direct beam."""
    kx, ky, inten, cnt = spots
    S = int(cnt.max())
    rand = functools.partial(torch.rand, generator=gen, device=DEV)
    randn = functools.partial(torch.randn, generator=gen, device=DEV)
    out = torch.empty((B, H, W), dtype=torch.float32 if dtype == "f32" else torch.int16, device=DEV)
    ys, xs = (torch.arange(n, device=DEV, dtype=torch.float32) for n in (H, W))
    step = max(1, min(1024, int(1.2e8 // ((S + 1) * (H + W)))))

    def drawn(x, y, a):
        gx, gy = (torch.where((d := ax - p[..., None]).abs() <= 6.0, torch.exp(d * d / -4.5), 0.0)
                  for ax, p in ((xs, x), (ys, y)))
        return torch.bmm((gy * a[..., None]).transpose(1, 2).contiguous(), gx)

    for b0 in range(0, B, step):
        n = min(step, B - b0)
        t = (rand(n) * kx.shape[0]).long().clamp_max(kx.shape[0] - 1)
        phi, sign = rand(n, 1) * (2 * math.pi), torch.where(rand(n, 1) < 0.5, 1.0, -1.0)
        cx, cy = (v / 2.0 + shift * (2.0 * rand(n, 1) - 1.0) for v in (W, H))
        fx, fy = kx[t, :S].float() * _px(R), ky[t, :S].float() * sign * _px(R)
        a = inten[t, :S].float() * torch.exp(0.5 * randn(n, S) - 0.125) * weak
        x = torch.cat([cx + phi.cos() * fx - phi.sin() * fy, cx], 1)
        y = torch.cat([cy + phi.sin() * fx + phi.cos() * fy, cy], 1)
        img = drawn(x, y, torch.cat([a, torch.full((n, 1), 4.0, device=DEV)], 1))
        if common is not None:   # the dominant phase, the same in every pattern
            img += drawn(*[v[None] for v in common])
        if diffuse:
            r2 = (xs - W / 2.0)[None, :] ** 2 + (ys - H / 2.0)[:, None] ** 2
            img += diffuse * torch.exp(r2 / (-2.0 * (W / 5.0) ** 2))
        if dtype == "f32":
            out[b0:b0 + n] = img.add_(0.01).add_(randn(n, H, W), alpha=0.02)
        else:
            out[b0:b0 + n] = torch.poisson(img.mul_(120.0).add_(0.5), generator=gen).to(torch.int16)
    return out if dtype == "f32" else out.view(torch.uint16)


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _full(c):
    """An indexing case with the choices that its kind settles."""
    if c["kind"] == "two_stage":
        return dict(c, phase="fcc", max_spots=100, R=min(c["H"], c["W"]) // 2, n_theta=360,
                    dtype="f32", gamma=1.0, route="bound", compact=True, angles=False)
    return c


def _inputs(c, seed):
    """The patterns of an indexing case (as _full gives it)."""
    gen = _gen(seed)
    spots = _spots(c["phase"], c["T"], c["max_spots"])[0]
    more = {}
    if c["kind"] == "two_stage":
        t = int(torch.randint(c["T"], (1,), generator=gen, device=DEV))
        more = dict(weak=0.25, common=(spots[0][t].float() * _px(c["R"]) + c["W"] / 2.0,
                                       spots[1][t].float() * _px(c["R"]) + c["H"] / 2.0,
                                       spots[2][t].float()))
    return _patterns(spots, c["B"], c["H"], c["W"], c["R"], c["dtype"], gen, **more)


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind == "preprocess":
        return dict(case=c, x=_raw(c, seed))
    if kind == "simulate":
        Bm, X = _crystal(c["phase"])
        return dict(case=c, basis=Bm, atoms=X, f=np.ones(len(X)), euler=_directions(c, seed))
    c = _full(c)
    lib = _library(c["phase"], c["T"], c["max_spots"], c["R"], c["n_theta"], kind == "two_stage",
                   c["route"] == "fft")
    return dict(case=c, x=_inputs(c, seed), lib=lib, grid=_grid(c),
                euler=_spots(c["phase"], c["T"], c["max_spots"])[1])


def _raw(c, seed):
    """Raw patterns: beam off centre by up to 3 px, diffuse background."""
    R = min(c["H"], c["W"]) // 2
    spots = _templates("fcc", torch.from_numpy(_spiral("fcc", 200)).to(DEV), 100)
    return _patterns(spots, c["B"], c["H"], c["W"], R, c["dtype"], _gen(seed), shift=3.0, diffuse=0.2)


def _directions(c, seed):
    u = torch.rand((c["T"], 2), generator=_gen(seed), device=DEV, dtype=torch.float64)
    return torch.stack([torch.arccos(u[:, 0]), u[:, 1] * (2 * math.pi)], 1).contiguous()


# --------------------------------------------------------------------- a pass
def run(state):
    c = state["case"]
    if c["kind"] == "preprocess":
        return tm.preprocess(state["x"], r_box=c["r_box"], sigma_min=c["sigma_min"],
                             sigma_max=c["sigma_max"], sigma_blur=c["sigma_blur"])
    if c["kind"] == "simulate":
        kx, ky, inten, cnt = tm.simulate_library(
            state["basis"], state["atoms"], state["f"], G_MAX + 0.2, state["euler"], K0, S_MAX,
            G_MAX, REL_MIN, c["max_spots"], csr=False)
        # rows hold count[t] spots; the rest of a row is not written
        live = torch.arange(c["max_spots"], device=DEV)[None] < cnt[:, None]
        return tuple(torch.where(live, v, 0.0) for v in (kx, ky, inten)) + (cnt,)
    lib, grid, N = state["lib"], state["grid"], c["N"]
    if c["kind"] == "two_stage":
        mask = tm.mask_from_mean(state["x"], 0.15)
        polar, norms, _ = tm.polar_transform(state["x"], grid, lib=lib, mask=mask,
                                             want_profile=False)
        return (mask,) + tm.match_batch(lib, polar, norms, N, coarse="bound")
    route = c["route"]
    pre = route in tm.PRECISIONS
    polar, norms, prof = tm.polar_transform(state["x"], grid, gamma=c["gamma"], want_profile=pre,
                                            lib=lib if c["compact"] else None)
    if pre:
        out = tm.match_batch(lib, polar, norms, N, profiles=prof, prefilter_keep=c["keep"],
                             prefilter_prec=route)
    else:
        out = tm.match_batch(lib, polar, norms, N, with_best=route == "maps",
                             coarse=route if route in ("bound", "fft") else None)
    if c["angles"]:
        deg = tm.refine_angles(lib, polar, norms, out[0], out[1])
        out += (deg, tm.orientations(state["euler"], out[0], angle_deg=deg, n_theta=c["n_theta"]))
    return out


# -------------------------------------------------------------- in 64 bits
def exact(case, seed):
    c = case
    if c["kind"] == "preprocess":
        return _exact_preprocess(c, _raw(c, seed)) if c["B"] * c["H"] * c["W"] < 3e8 else None
    if c["kind"] == "simulate":
        # (positions of spots of equal intensity may come in another order)
        return [None, None, _templates(c["phase"], _directions(c, seed), c["max_spots"])[2], None]
    if c["B"] * 2 * c["T"] > EXACT_PAIRS or c.get("route") in tm.PRECISIONS:
        return None              # (a pre-filter's result hangs on its kept set)
    c = _full(c)
    x, spots = _inputs(c, seed), _spots(c["phase"], c["T"], c["max_spots"])[0]
    two = c["kind"] == "two_stage"
    mask = _exact_mask(x, 0.15) if two else None
    best = _exact_scores(x, _grid(c), spots, two, c["gamma"], mask)
    # templates and angles: near-equal scores may come in another order
    out = [None, None, torch.topk(best, c["N"], dim=1).values]
    out += [best, None] if c["route"] == "maps" else []
    return ([mask] if two else []) + out + ([None, None] if c["angles"] else [])


def _exact_scores(x, grid, spots, unit, gamma, mask):
    """Best Q of Eq. (1) per pattern and template (mirrors after the base
    templates) [B, 2 T], by transforms along the azimuth."""
    kx, ky, inten, cnt = spots
    R, n, px, T = grid.R, grid.n_theta, _px(grid.R), kx.shape[0]
    live = torch.arange(kx.shape[1], device=DEV)[None] < cnt[:, None]
    j = torch.round(torch.hypot(kx, ky) * px).long()
    k = torch.round(torch.atan2(ky, kx) * (n / (2 * math.pi))).long() % n
    live &= j < R
    w = torch.where(live, torch.ones_like(inten) if unit else inten, 0.0)
    best = torch.empty((x.shape[0], 2 * T), dtype=torch.float64, device=DEV)
    tstep, bstep = max(1, int(4e7 // (R * n))), max(1, min(int(4e7 // (R * n)), 64))
    for t0 in range(0, T, tstep):
        m = slice(t0, min(T, t0 + tstep))
        img = torch.zeros((m.stop - t0, R * n), dtype=torch.float64, device=DEV)
        img.scatter_add_(1, (j[m].clamp_max(R - 1) * n + k[m]), w[m])
        img /= img.norm(dim=1, keepdim=True).clamp_min(1e-300)
        ft = torch.fft.rfft(img.view(-1, R, n)).permute(2, 1, 0).contiguous()    # [F, R, t]
        for b0 in range(0, x.shape[0], bstep):
            P, norm = _exact_polar(x[b0:b0 + bstep], grid, gamma, mask)
            fp = torch.fft.rfft(P).permute(2, 0, 1).contiguous()                 # [F, b, R]
            for half, f in ((0, ft.conj().resolve_conj()), (T, ft)):
                q = torch.empty((fp.shape[1], f.shape[2]), dtype=torch.float64, device=DEV)
                for a in range(0, f.shape[2], 1000):
                    C = torch.bmm(fp, f[:, :, a:a + 1000].contiguous())
                    q[:, a:a + 1000] = torch.fft.irfft(C.permute(1, 2, 0), n=n).amax(2)
                best[b0:b0 + bstep, half + t0:half + m.stop] = torch.where(
                    norm[:, None] > 0, q / norm[:, None].clamp_min(1e-300), 0.0)
    return best


def _exact_polar(x, grid, gamma, mask):
    p = x.to(torch.float64)
    if gamma != 1.0:
        p = p.clamp_min(0.0) ** gamma
    if mask is not None:
        p = p * mask
    H, W = p.shape[1:]
    r = torch.arange(grid.R, device=DEV, dtype=torch.float64)[:, None]
    th = torch.arange(grid.n_theta, device=DEV, dtype=torch.float64)[None] * (2 * math.pi / grid.n_theta)
    out = _bilinear(p, grid.cx + r * th.cos(), grid.cy + r * th.sin(), H, W)
    return out, out.flatten(1).norm(dim=1)


def _bilinear(p, x, y, H, W):
    """Samples of images p [B, H, W] at (x, y), zero outside."""
    x0, y0 = x.floor(), y.floor()
    out = 0.0
    for dx in (0, 1):
        for dy in (0, 1):
            xi, yi = x0 + dx, y0 + dy
            w = (1 - (x - xi).abs()) * (1 - (y - yi).abs())
            ok = (xi >= 0) & (xi < W) & (yi >= 0) & (yi < H)
            at = (yi.clamp(0, H - 1) * W + xi.clamp(0, W - 1)).long()
            v = p.flatten(1)[:, at.flatten()].view(-1, *at.shape) if at.dim() == 2 else \
                p.flatten(1).gather(1, at.flatten(1)).view(at.shape)
            out = out + torch.where(ok, w, 0.0) * v
    return out


def _exact_mask(x, threshold):
    mean = torch.zeros(x.shape[1:], dtype=torch.float64, device=DEV)
    for p in torch.split(x, 256):
        mean += p.double().sum(0)
    bright = (mean / x.shape[0] > threshold)[None, None].double()

    def dilate(v):
        return torch.nn.functional.max_pool2d(torch.nn.functional.pad(v, (1, 1, 1, 1)), 3, 1)

    eroded = 1.0 - dilate(torch.nn.functional.pad(1.0 - bright, (1, 1, 1, 1), value=1.0))[..., 1:-1, 1:-1]
    return 1.0 - dilate(dilate(dilate(eroded)))[0, 0]


def _gauss(n, sigma):
    """[n, n] Gaussian correlation along an axis with mirrored borders."""
    r = int(4.0 * sigma + 0.5)
    t = np.arange(-r, r + 1)
    w = np.exp(-t * t / (2.0 * sigma * sigma)) if sigma > 0 else np.ones(1)
    i = (np.arange(n)[:, None] + t[None]) % (2 * n)
    G = np.zeros((n, n))
    np.add.at(G, (np.arange(n)[:, None].repeat(len(t), 1), np.where(i < n, i, 2 * n - 1 - i)), w / w.sum())
    return torch.from_numpy(G).to(DEV)


def _exact_preprocess(c, x):
    B, H, W = x.shape
    xs, ys = (torch.arange(n, device=DEV, dtype=torch.float64) for n in (W, H))
    box = ((xs - W / 2.0).abs() <= c["r_box"])[None, :] & ((ys - H / 2.0).abs() <= c["r_box"])[:, None]
    Gy, Gx = ([_gauss(n, c[s]) for s in ("sigma_min", "sigma_max", "sigma_blur")] for n in (H, W))
    out, centre = torch.empty((B, H, W), dtype=torch.float64, device=DEV), []
    for b0 in range(0, B, 64):
        p = x[b0:b0 + 64].double()
        top = torch.where(box, p, -math.inf).amax((1, 2), keepdim=True)
        w = torch.where(box & (p >= 0.5 * top), p, 0.0)
        s = w.sum((1, 2))
        ok = (top > 0).flatten()
        cx = torch.where(ok, (w * xs).sum((1, 2)) / s, W / 2.0)
        cy = torch.where(ok, (w * ys[:, None]).sum((1, 2)) / s, H / 2.0)
        centre.append(torch.stack([cx, cy], 1))
        at_x = (xs[None, None, :] + (cx - W / 2.0)[:, None, None]).expand(-1, H, -1)
        at_y = (ys[None, :, None] + (cy - H / 2.0)[:, None, None]).expand(-1, -1, W)
        p = _bilinear(p, at_x, at_y, H, W)
        d = Gy[0] @ p @ Gx[0].T - Gy[1] @ p @ Gx[1].T
        out[b0:b0 + 64] = (Gy[2] @ d @ Gx[2].T).clamp_min(0.0)
    return [out, torch.cat(centre)]


# ----------------------------------------------------------- what it has to do
def work(case):
    c = case
    if c["kind"] == "simulate":
        refl = {"fcc": 760, "hcp": 820, "ortho": 1970}[c["phase"]]
        spots = min(c["max_spots"], MEAN_SPOTS[c["phase"]])
        return {"bytes": c["T"] * (16 + 24 * spots + 4), "flops": 30 * c["T"] * refl}
    px = c["B"] * c["H"] * c["W"]
    if c["kind"] == "preprocess":
        taps = sum(2 * int(4 * c[s] + 0.5) + 1 for s in ("sigma_min", "sigma_max", "sigma_blur"))
        return {"bytes": px * (2 + 4 if c["dtype"] == "u16" else 8), "flops": px * (4 * taps + 12)}
    spots = 2 * c["T"] * MEAN_SPOTS[c.get("phase", "fcc")]       # with the mirrors
    maps = c.get("route") == "maps"
    # every pattern read and resampled; every template pixel taken at least
    # once per pattern (at every shift where each template's maximum is asked for)
    flops = 2.0 * c["B"] * spots * (c["n_theta"] if maps else 1) + 8.0 * px
    size = px * (2 if c.get("dtype") == "u16" else 4) + 8 * spots + 12 * c["B"] * c["N"]
    return {"bytes": size + (6 * c["B"] * 2 * c["T"] if maps else 0), "flops": flops}
