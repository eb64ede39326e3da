"""The work that a program using this library has it do, as measurable cases.

Every case is one call (a blocking solve, or one multi-grid batch) through
`paper_2110_15640_amd.mcrt.Context` on resident grids and opacity tables, the
way the paper's post-processing runs are made: 1D and 3D geometric albedo,
thermal emission phase curves, Doppler-shifted high-resolution emission,
raytrace and multiple-scattering transmission, and batches over uneven grids.
Grids and tables come from `paper_2110_15640_amd.inputs`; sizes go from one
wavelength of a few hundred packets to the grids the benchmark solves.

Outputs are the whole result arrays of the call: band values, their standard
errors, per-g values, raw sums, counters and (emission) total luminosities.
"""
import math
import random

import numpy as np
import torch

from paper_2110_15640_amd import inputs as I
from paper_2110_15640_amd import mcrt as M

PRECISION = {"fp64": M.MCRT_FP64, "mixed": M.MCRT_MIXED}
OUTPUTS = ("value", "stderr", "per_g", "sums", "counters", "l_tot")
A_ORBIT = 0.03 * 1.496e13


def listed():
    return [
        # the smallest call: one wavelength of a 1D column, a quick look (latency)
        dict(name="slab_quick", kind="slab", nlay=50, nlam=1, packets=1000, precision="fp64", clouds=False, mu0=0.0, nobs=0),
        # the 1D albedo spectrum: 50 layers, 10 wavelengths x 1e5 packets, library defaults
        dict(name="slab_spectrum", kind="slab", nlay=50, nlam=10, packets=100000, precision="fp64", clouds=False, mu0=0.0,
             nobs=0),
        # a coarse 3D run while setting a model up: few packets, few bands (launches and latency)
        dict(name="emission_coarse", kind="emission", nlon=32, nlat=16, nlay=30, nband=2, ng=8, packets=1000, nobs=2,
             precision="fp64", clouds=False),
        # the 3D emission phase curve on its grid, defaults (FP64), some of its bands
        dict(name="emission_curve_fp64", kind="emission", nlon=128, nlat=64, nlay=50, nband=6, ng=8, packets=100000, nobs=4,
             precision="fp64", clouds=False),
        # the same in the mixed form with more bands: the throughput run
        dict(name="emission_curve_mixed", kind="emission", nlon=128, nlat=64, nlay=50, nband=25, ng=8, packets=100000, nobs=4,
             precision="mixed", clouds=False),
        # scattered-light phase curve of a cloudy planet
        dict(name="sphere_albedo_cloudy", kind="sphere", nlon=64, nlat=32, nlay=40, nband=5, ng=4, packets=50000, nobs=4,
             precision="mixed", clouds=True),
        # Doppler-shifted high-resolution emission toward one observer
        dict(name="emission_hires", kind="emission_hires", nlon=64, nlat=32, nlay=45, nlam=40, packets=40000,
             precision="fp64"),
        # transmission with multiple scattering in clouds behind a limb-darkened star
        dict(name="transit_scattering", kind="transit_ms", nlon=64, nlat=32, nlay=40, nband=4, ng=4, packets=30000, law=2,
             precision="mixed"),
        # high-resolution transmission with winds: the 128 x 64 x 60 grid and its 256 x 360 chords
        dict(name="transit_hires_mixed", kind="transit_hires", nlon=128, nlat=64, nlay=60, nlam=6000, n_b=256, n_alpha=360,
             precision="mixed"),
        # a ragged FP64 high-resolution window on a smaller grid
        dict(name="transit_hires_fp64", kind="transit_hires", nlon=90, nlat=46, nlay=53, nlam=500, n_b=200, n_alpha=181,
             precision="fp64"),
        # low-resolution transmission spectrum from correlated-k opacities, defaults
        dict(name="transit_ck", kind="transit_ck", nlon=64, nlat=32, nlay=50, nband=30, ng=8, n_b=256, n_alpha=360,
             precision="fp64"),
        # several requests on grids of uneven size in one batch
        dict(name="batch_uneven", kind="batch", items=6, bands=12, ng=8, packets=20000, precision="mixed"),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes over the whole range of the listed ones."""
    kind = rng.choice(["slab", "emission", "emission", "sphere", "emission_hires", "transit_hires", "transit_hires",
                       "transit_ck", "transit_ms", "batch"])
    prec = rng.choice(["fp64", "mixed"])
    if kind == "slab":
        nlam = _logint(rng, 1, 40)
        return dict(kind=kind, nlay=_logint(rng, 7, 150), nlam=nlam, packets=_logint(rng, 300, 1500000 // nlam), precision=prec,
                    clouds=rng.random() < 0.5, mu0=rng.choice([0.0, round(rng.uniform(0.2, 1.0), 3)]),
                    nobs=rng.choice([0, 0, 1, 3]))
    nlon = 2 * _logint(rng, 8, 64)
    geo = dict(nlon=nlon, nlat=max(4, nlon // 2 - rng.choice([0, 0, 1])), nlay=_logint(rng, 12, 64), precision=prec)
    if kind in ("emission", "sphere"):
        nband, ng = _logint(rng, 1, 12), rng.choice([1, 4, 8])
        top = (5000000 if kind == "emission" else 1500000) // (nband * ng)
        return dict(geo, kind=kind, nband=nband, ng=ng, packets=_logint(rng, 300, max(400, min(top, 400000))),
                    nobs=rng.randint(1, 4), clouds=rng.random() < 0.5)
    if kind == "emission_hires":
        nlam = _logint(rng, 4, 60)
        return dict(geo, kind=kind, nlam=nlam, packets=_logint(rng, 500, 2000000 // nlam))
    if kind == "transit_hires":
        return dict(geo, kind=kind, nlam=_logint(rng, 30, 3000), n_b=_logint(rng, 32, 256), n_alpha=_logint(rng, 40, 360))
    if kind == "transit_ck":
        return dict(geo, kind=kind, nband=_logint(rng, 1, 40), ng=rng.choice([4, 8]), n_b=_logint(rng, 32, 256),
                    n_alpha=_logint(rng, 40, 360))
    if kind == "transit_ms":
        nband = _logint(rng, 1, 8)
        return dict(geo, kind=kind, nband=nband, ng=4, packets=_logint(rng, 500, 400000 // nband), law=rng.randint(0, 4))
    return dict(kind=kind, items=rng.randint(2, 8), bands=_logint(rng, 2, 16), ng=rng.choice([4, 8]),
                packets=_logint(rng, 500, 20000), precision=prec)


# ------------------------------------------------------------------ inputs
def _clouds(grid, rng):
    """A grey cloud deck: opacity falling with height, mostly forward scattering."""
    k = np.repeat(np.arange(grid.nlay), grid.nlon * grid.nlat) / grid.nlay
    patch = rng.uniform(0.2, 1.0, grid.ncell)
    grid.cld_ksca = (2e-2 * patch * np.exp(-3.0 * k)).astype(np.float32)
    grid.cld_kabs = (1e-3 * patch * np.exp(-3.0 * k)).astype(np.float32)
    grid.cld_g = rng.uniform(0.2, 0.85, grid.ncell).astype(np.float32)


def _inputs(case, seed):
    """Grid(s), table and the call's parameters, from the seed alone."""
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    p = dict(seed=int(rng.integers(1, 1 << 40)), precision=PRECISION[case["precision"]])
    if kind == "slab":
        grid, table = I.make_albedo_slab(nlay=case["nlay"], nlam=case["nlam"], T=float(rng.uniform(900.0, 1500.0)),
                                         k_abs=float(10.0 ** rng.uniform(-3.5, -2.5)))
        if case["clouds"]:
            _clouds(grid, rng)
        p.update(n_packets=case["packets"], mu0=case["mu0"])
        if case["nobs"]:
            th, ph = rng.uniform(0.1, 1.3, case["nobs"]), rng.uniform(0.0, 2.0 * math.pi, case["nobs"])
            p["obs_dir"] = np.stack([np.sin(th) * np.cos(ph), np.sin(th) * np.sin(ph), np.cos(th)], axis=1)
        return [grid], table, p
    no = int(seed) % 1000003
    if kind in ("emission", "sphere", "transit_ck", "transit_ms"):
        grid, table, _ = I.make_emission_3d(case["nlon"], case["nlat"], case["nlay"], nband=case["nband"], ng=case["ng"],
                                            config_no=no)
        if case.get("clouds") or kind == "transit_ms":
            _clouds(grid, rng)
        if kind in ("emission", "sphere"):
            ph = np.arange(case["nobs"]) / case["nobs"]
            p.update(n_packets=case["packets"], obs_phase=ph if kind == "emission" else math.pi * ph * 0.9)
            if kind == "sphere":
                p["decorrelate"] = 1
        elif kind == "transit_ck":
            p.update(n_b=case["n_b"], n_alpha=case["n_alpha"], r_star=I.R_SUN)
        else:
            p.update(n_packets=case["packets"], ms_transmission=1, a_orbit=A_ORBIT, r_star=I.R_SUN, ld_law=case["law"],
                     ld_c1=0.45, ld_c2=0.2, transit_y=0.3 * I.R_SUN, transit_z=-0.2 * I.R_SUN)
        return [grid], table, p
    if kind in ("emission_hires", "transit_hires"):
        grid, table = I.make_transmission_hires(case["nlon"], case["nlat"], case["nlay"], nlam=case["nlam"],
                                                lam_hi=1.0 + 0.1 * case["nlam"] / 20000.0, config_no=no)
        if kind == "emission_hires":
            p.update(n_packets=case["packets"], obs_phase=[float(rng.uniform(0.2, 0.8))])
        else:
            p.update(n_b=case["n_b"], n_alpha=case["n_alpha"], r_star=I.R_SUN)
        return [grid], table, p
    # batch: grids of uneven size (as inputs.make_batch_mix makes them, each seed its own atmospheres) sharing one table
    r = random.Random(case["items"])
    grids = []
    for q in range(case["items"]):
        nlon = 32 + 16 * r.randint(0, 4)
        grids.append(I.make_sphere(nlon, nlon // 2, r.randint(30, 50), no * 1000 + q))
    table = I.make_ck_table(rng, nband=2 * case["bands"], ng=case["ng"])
    p.update(obs_phase=[0.0, 0.5])
    return grids, table, p


def _batch_items(case, seed):
    r, pick = random.Random(case["bands"]), random.Random(int(seed))
    items = []
    for q in range(case["items"]):
        nb = r.randint(max(1, case["bands"] // 2), case["bands"])
        items.append(dict(mode="emission" if q % 2 == 0 else "albedo",
                          spec_idx=sorted(pick.sample(range(2 * case["bands"]), nb)),
                          n_packets=max(300, int(case["packets"] * r.uniform(0.25, 1.0)))))
    return items


_CTX = []


def _context():
    if not _CTX:
        _CTX.append(M.Context(0))
    return _CTX[0]


class _State:
    """Resident grids and table of one program, freed with it."""

    def __init__(self, case, seed):
        grids, self.table, self.params = _inputs(case, seed)
        self.ctx = _context()
        self.kind = case["kind"]
        self.gids = [self.ctx.upload_grid(g) for g in grids]
        self.oid = self.ctx.upload_opacity(self.table)
        if self.kind == "batch":
            self.items = [dict(it, gid=self.gids[q], oid=self.oid, table=self.table)
                          for q, it in enumerate(_batch_items(case, seed))]

    def __del__(self):
        try:
            for g in self.gids:
                self.ctx.free_grid(g)
            self.ctx.free_opacity(self.oid)
        except Exception:  # the context is already gone
            pass


def prepare(case, seed):
    return _State(case, seed)


def run(state):
    c, k, p = state.ctx, state.kind, state.params
    if k == "batch":
        return [{n: out[n] for n in OUTPUTS} for out in c.solve_batch(state.items, **p)]
    solve = {"slab": c.solve_albedo, "sphere": c.solve_albedo, "emission": c.solve_emission,
             "emission_hires": c.solve_emission}.get(k, c.solve_transmission)
    out = solve(state.gids[0], state.oid, state.table, **p)
    return {n: out[n] for n in OUTPUTS}


# ------------------------------------------------------------------ work
def work(case):
    """Inputs read once, results written once, and the arithmetic of the cell
    crossings (or slab events, or chord sums) that the estimator consists of."""
    k = case["kind"]
    nobs = max(1, case.get("nobs", 1))
    if k == "slab":
        ncell, tab, rows = case["nlay"], case["nlam"] * 16, case["nlam"]
        # about ten interactions per packet, each a flight and nobs peel-offs
        flops = case["nlam"] * case["packets"] * 10.0 * (1 + nobs) * 100.0
    elif k == "batch":
        ncell, tab, rows = case["items"] * 64 * 32 * 40, 2 * case["bands"] * case["ng"] * 1600, \
            case["items"] * 0.75 * case["bands"] * case["ng"]
        flops = rows * 0.6 * case["packets"] * 3.0 * 36.0 * 88.0
    else:
        ncell = case["nlon"] * case["nlat"] * case["nlay"]
        cross = 0.6 * case["nlay"] + 0.1 * (case["nlon"] + case["nlat"])  # cells met by one ray from inside to the top
        rows = case["nlam"] if "nlam" in case else case["nband"] * case["ng"]
        tab = rows * 1600
        if k in ("transit_hires", "transit_ck"):
            seg = case["n_b"] * case["n_alpha"] * (1.0 * case["nlay"] + 0.15 * (case["nlon"] + case["nlat"]))
            # one multiply-add per (segment, row); the interpolated extinction of every (cell, row)
            flops = 2.0 * seg * rows + 30.0 * ncell * rows + 88.0 * seg
        else:
            flops = rows * case["packets"] * (1.3 * nobs + 1.0) * cross * 88.0
    return {"bytes": 40.0 * ncell + tab + rows * (8.0 * 11 + 32.0 * nobs), "flops": flops}


# ------------------------------------------------------------------ exact values
# The same estimators in plain numpy / torch, 64 bits: Philox4x32-10 packets of
# the slab, raytrace chords, and the luminosities of the emitting cells.
def exact(case, seed):
    k = case["kind"]
    if k == "slab":
        if case["nlam"] * case["packets"] > 1100000:
            return None
        return _exact_slab(case, seed)
    if k in ("transit_hires", "transit_ck"):
        return _exact_chords(case, seed)
    if k in ("emission", "emission_hires"):
        grids, table, p = _inputs(case, seed)
        return dict({n: None for n in OUTPUTS}, l_tot=_exact_ltot(grids[0], table, p))
    return None


def _philox(seed, tag, packet, event, block):
    """Uniform pairs ((m + 1/2) 2^-52) of counter (packet, event, block)."""
    m32 = np.uint64(0xFFFFFFFF)
    n = packet.shape[0]
    c0, c1 = packet & m32, packet >> np.uint64(32)
    c2, c3 = np.full(n, event, np.uint64), np.full(n, block, np.uint64)
    k0, k1 = seed & 0xFFFFFFFF, ((seed >> 32) & 0xFFFFFFFF) ^ tag
    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
        p0, p1 = c0 * np.uint64(0xD2511F53), c2 * np.uint64(0xCD9E8D57)
        c0, c2 = (p1 >> np.uint64(32)) ^ c1 ^ np.uint64(k0), (p0 >> np.uint64(32)) ^ c3 ^ np.uint64(k1)
        c1, c3 = p1 & m32, p0 & m32
    a = (c0 << np.uint64(20)) | (c1 >> np.uint64(12))
    b = (c2 << np.uint64(20)) | (c3 >> np.uint64(12))
    return (a.astype(np.float64) + 0.5) * 2.0 ** -52, (b.astype(np.float64) + 0.5) * 2.0 ** -52


def _results(case, sums, counters, scale, weights, l_tot=None):
    """The result arrays from raw sums [spec][g][obs][2]: value = scale mean."""
    n = float(case["packets"])
    m = sums[..., 0] / n
    se = scale * np.sqrt(np.maximum(sums[..., 1] / n - m * m, 0.0) / n)
    per_g = scale * m
    w = weights[None, :, None]
    return dict(value=(w * per_g).sum(1), stderr=np.sqrt((w * w * se * se).sum(1)), per_g=per_g, sums=sums, counters=counters,
                l_tot=np.zeros(sums.shape[:2]) if l_tot is None else l_tot)


def _ck_kappa(table, T, P):
    """kappa of every (band, g) at the given temperatures and pressures."""
    with np.errstate(divide="ignore"):
        lnk = np.log(table.kappa.astype(np.float64))
    Tg, lp = table.T_grid, np.log(table.P_grid)

    def bracket(g, x):
        if len(g) == 1:
            return np.zeros(len(x), int), np.zeros(len(x), int), np.zeros(len(x))
        i = np.clip(np.searchsorted(g, x, side="right") - 1, 0, len(g) - 2)
        return i, i + 1, np.clip((x - g[i]) / (g[i + 1] - g[i]), 0.0, 1.0)

    t0, t1, t = bracket(Tg, T)
    p0, p1, u = bracket(lp, np.log(P))
    return lnk, (t0, t1, t, p0, p1, u)


def _interp(lnk, br):
    t0, t1, t, p0, p1, u = br
    return np.exp((1 - t) * (1 - u) * lnk[t0, p0] + (1 - t) * u * lnk[t0, p1] + t * (1 - u) * lnk[t1, p0] + t * u * lnk[t1, p1])


def _exact_slab(case, seed):
    grids, table, p = _inputs(case, seed)
    g = grids[0]
    z, nlay, N = g.r_edges, g.nlay, case["packets"]
    ks = np.zeros(nlay) if g.cld_ksca is None else g.cld_ksca.astype(np.float64)
    ka = np.zeros(nlay) if g.cld_kabs is None else g.cld_kabs.astype(np.float64)
    gc = np.zeros(nlay) if g.cld_g is None else g.cld_g.astype(np.float64)
    lnk, br = _ck_kappa(table, g.T.astype(np.float64), g.P.astype(np.float64))
    obs = p.get("obs_dir")
    no = 1 if obs is None else len(obs)
    sums, cnt = np.zeros((case["nlam"], 1, no, 2)), np.zeros((case["nlam"], 1, 11))
    for s in range(case["nlam"]):
        kr = float(table.k_ray[s])
        kab = _interp(lnk[s, 0], br) + ka
        ksc = kr + ks
        a = g.rho * (kab + ksc)
        om, pg = ksc / (kab + ksc), np.where(ksc > 0, kr / np.where(ksc > 0, ksc, 1.0), 1.0)
        F, c = _slab_packets(z, a, om, pg, gc, N, p["seed"], case["mu0"], obs)
        sums[s, 0, :, 0], sums[s, 0, :, 1] = F.sum(0), (F * F).sum(0)
        cnt[s, 0] = c
    return _results(case, sums, cnt, math.pi, np.ones(1))


def _slab_packets(z, a, om, pg, gc, N, seed, mu0, obs):
    nlay = len(a)
    cum = np.concatenate([[0.0], np.cumsum(a * np.diff(z))])  # vertical optical depth from the bottom
    idx = np.arange(N, dtype=np.uint64)
    u, _ = _philox(seed, 0, idx, 0, 0)
    m0 = np.full(N, mu0) if mu0 > 0.0 else np.sqrt(1.0 - u)
    d0 = np.stack([np.sqrt(np.maximum(1.0 - m0 * m0, 0.0)), np.zeros(N), -m0], axis=1)
    no = 1 if obs is None else len(obs)
    F, c = np.zeros((N, no)), np.zeros(11)
    c[10] = N
    zz, k, d, W = np.full(N, z[-1]), np.full(N, nlay - 1), d0.copy(), np.ones(N)
    act = np.arange(N)
    e = 1
    while len(act):
        q = idx[act]
        ua, usel = _philox(seed, 0, q, e, 0)
        dz = d[:, 2]
        here = cum[k] + a[k] * (zz - z[k])
        goal = here + dz * -np.log(ua)
        up, down = goal >= cum[-1], goal <= 0.0
        kk = np.clip(np.searchsorted(cum, goal, side="right") - 1, 0, nlay - 1)
        c[7] += np.where(up, nlay - k, np.where(down, k + 1, np.abs(kk - k))).sum()
        c[0] += W[up].sum()
        c[1] += W[down].sum()
        hit = ~(up | down)
        act, q, usel, d, W, k, goal = act[hit], q[hit], usel[hit], d[hit], W[hit], kk[hit], goal[hit]
        if not len(act):
            break
        zz = z[k] + (goal - cum[k]) / a[k]
        c[6] += len(act)
        for o in range(no):
            v = -d0[act] if obs is None else np.broadcast_to(obs[o], (len(act), 3))
            oz = v[:, 2]
            seen = oz > 0.0
            ozs = np.where(seen, oz, 1.0)
            tau = (cum[-1] - goal) / ozs
            # cells crossed: up to the top, or to the first cell past the optical-depth cut
            cut = np.searchsorted(cum[1:], goal + 50.0 * ozs, side="right")
            c[7] += np.where(seen, np.minimum(cut, nlay - 1) - k + 1, 0).sum()
            mu = (d * v).sum(1)
            den = 1.0 + gc[k] ** 2 - 2.0 * gc[k] * mu
            ph = pg[k] * 0.75 * (1.0 + mu * mu) + (1.0 - pg[k]) * (1.0 - gc[k] ** 2) / (den * np.sqrt(den))
            F[act, o] += np.where(seen & (tau <= 50.0), W * om[k] * ph / (4.0 * math.pi) * np.exp(-tau), 0.0)
        c[2] += (W * (1.0 - om[k])).sum()
        W = W * om[k]
        x, ps = _philox(seed, 0, q, e, 1)
        qq = 4.0 * x - 2.0
        w = np.cbrt(qq + np.sqrt(qq * qq + 1.0))
        gk = gc[k]
        gs = np.where(np.abs(gk) < 1e-6, 1.0, gk)
        t = (1.0 - gs * gs) / (1.0 - gs + 2.0 * gs * x)
        hg = np.where(np.abs(gk) < 1e-6, 2.0 * x - 1.0, (1.0 + gs * gs - t * t) / (2.0 * gs))
        mu = np.clip(np.where(usel < pg[k], w - 1.0 / w, hg), -1.0, 1.0)
        st, cp, sp = np.sqrt(np.maximum(1.0 - mu * mu, 0.0)), np.cos(2.0 * math.pi * ps), np.sin(2.0 * math.pi * ps)
        dx, dy, dz = d.T
        flat = np.abs(dz) < 0.99999
        t = np.sqrt(np.where(flat, 1.0 - dz * dz, 1.0))
        n = np.stack([np.where(flat, st * (dx * dz * cp - dy * sp) / t + dx * mu, st * cp),
                      np.where(flat, st * (dy * dz * cp + dx * sp) / t + dy * mu, st * sp),
                      np.where(flat, -st * cp * t + dz * mu, np.where(dz >= 0.0, 1.0, -1.0) * mu)], axis=1)
        d = n / np.sqrt((n * n).sum(1))[:, None]
        low = W < 1e-3
        if low.any():
            live, _ = _philox(seed, 0, q, e, 2)
            wn = np.where(live < 0.1, W / 0.1, 0.0)
            c[3] += (W - wn)[low].sum()
            W = np.where(low, wn, W)
            keep = W > 0.0
            act, d, W, k, zz = act[keep], d[keep], W[keep], k[keep], zz[keep]
        e += 1
    return F, c


def _exact_ltot(g, table, p):
    h, cl, kb = 6.62607015e-27, 2.99792458e10, 1.380649e-16
    T, P = g.T.astype(np.float64), g.P.astype(np.float64)
    lnk, br = _ck_kappa(table, T, P)
    hires = not hasattr(table, "g_weights")
    cloud = np.zeros((2, g.ncell)) if g.cld_ksca is None else np.stack([g.cld_ksca, g.cld_kabs]).astype(np.float64)
    vol = (np.diff(g.r_edges ** 3) / 3.0)[:, None, None] * np.diff(np.sin(g.lat_edges))[None, :, None] * \
        np.diff(g.lon_edges)[None, None, :]
    dr = np.diff(g.r_edges)[:, None, None]
    if hires:
        lam = math.pi * (1.0 - 2.0 * p["obs_phase"][0])
        x = _doppler(g, table, (math.cos(lam), math.sin(lam), 0.0))
    ns, ng = (table.nlam, 1) if hires else (table.nband, table.ng)
    out = np.zeros((ns, ng))
    for s in range(ns):
        for q in range(ng):
            if hires:
                pos = s + x
                n0 = np.clip(np.floor(pos).astype(int), 0, max(table.nlam - 2, 0))
                fr = np.clip(pos - n0, 0.0, 1.0)
                kg = (1.0 - fr) * _interp_at(lnk, n0, br) + fr * _interp_at(lnk, np.minimum(n0 + 1, table.nlam - 1), br)
                lc = table.lam_min_um * math.exp(s * table.dlnlam) * 1e-4
            else:
                kg = _interp(lnk[s, q], br)
                lc = float(table.lam_um[s]) * 1e-4
            kab = kg + cloud[1]
            ext = (g.rho * (kab + float(table.k_ray[s]) + cloud[0])).reshape(g.nlay, g.nlat, g.nlon)
            B = 2.0 * h * cl * cl / lc ** 5 / np.expm1(h * cl / (lc * kb * T))
            L = 4.0 * math.pi * vol * (g.rho * kab * B).reshape(g.nlay, g.nlat, g.nlon)
            dt = ext * dr
            above = np.cumsum(dt[::-1], axis=0)[::-1] - dt
            out[s, q] = np.where(above > 30.0, 0.0, L).sum()
    return out


def _interp_at(lnk, n, br):
    t0, t1, t, p0, p1, u = br
    return np.exp((1 - t) * (1 - u) * lnk[n, t0, p0] + (1 - t) * u * lnk[n, t0, p1] + t * (1 - u) * lnk[n, t1, p0]
                  + t * u * lnk[n, t1, p1])


def _doppler(g, table, o):
    """Shift of every cell in table points toward the observer direction o."""
    rc, th, ph = (0.5 * (e[1:] + e[:-1]) for e in (g.r_edges, g.lat_edges, g.lon_edges))
    k, j, i = np.meshgrid(np.arange(g.nlay), np.arange(g.nlat), np.arange(g.nlon), indexing="ij")
    k, j, i = k.ravel(), j.ravel(), i.ravel()
    st, ct, sp, cp = np.sin(th)[j], np.cos(th)[j], np.sin(ph)[i], np.cos(ph)[i]
    u, v, w = (np.zeros(g.ncell) if x is None else x.astype(np.float64) for x in (g.u, g.v, g.w))
    ue = u + g.omega_rot * rc[k] * ct
    vx, vy, vz = -sp * ue - st * cp * v + ct * cp * w, cp * ue - st * sp * v + ct * sp * w, ct * v + st * w
    return np.log1p((vx * o[0] + vy * o[1] + vz * o[2]) / 2.99792458e10) / table.dlnlam


def _exact_chords(case, seed):
    nch = case["n_b"] * case["n_alpha"]
    rows = case["nlam"] if case["kind"] == "transit_hires" else case["nband"] * case["ng"]
    if nch * float(rows) * (case["nlay"] + 0.2 * (case["nlon"] + case["nlat"])) > 7e10:
        return None
    grids, table, p = _inputs(case, seed)
    g = grids[0]
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    ch, cell, length, wb, ok = _trace_chords(g, case["n_b"], case["n_alpha"], p["seed"], dev)
    lnk, br = _ck_kappa(table, g.T.astype(np.float64), g.P.astype(np.float64))
    td = lambda x: torch.as_tensor(np.ascontiguousarray(x), device=dev)  # noqa: E731
    t0, t1, t, p0, p1, u = (td(x) for x in br)
    w4 = [((1 - t) * (1 - u))[:, None], ((1 - t) * u)[:, None], (t * (1 - u))[:, None], (t * u)[:, None]]
    nP = len(table.P_grid)
    at = [t0 * nP + p0, t0 * nP + p1, t1 * nP + p0, t1 * nP + p1]
    rho = td(g.rho)[:, None]
    hires = case["kind"] == "transit_hires"
    tab = td(lnk.reshape(rows, -1).T)  # [T P][row]
    kr = td(np.asarray(table.k_ray) if hires else np.repeat(table.k_ray, table.ng))
    if hires:
        x = td(_doppler(g, table, (-1.0, 0.0, 0.0)))[:, None]

    def interp(n):  # n: [cell][row]
        return torch.exp(sum(w * tab.reshape(-1)[a[:, None] * rows + n] for w, a in zip(w4, at)))

    sums = torch.zeros((rows, 2), dtype=torch.float64, device=dev)
    per = 16
    part = max(1, int(6e7) // per)
    for r0 in range(0, rows, per):
        n = torch.arange(r0, min(rows, r0 + per), device=dev)[None, :]
        if hires:
            pos = n + x
            n0 = torch.clamp(torch.floor(pos).long(), 0, max(rows - 2, 0))
            fr = torch.clamp(pos - n0, 0.0, 1.0)
            kg = (1.0 - fr) * interp(n0) + fr * interp(torch.clamp(n0 + 1, max=rows - 1))
        else:
            kg = interp(n.expand(g.ncell, -1))
            if g.cld_ksca is not None:
                kg = kg + td(g.cld_ksca.astype(np.float64) + g.cld_kabs.astype(np.float64))[:, None]
        alpha = rho * (kg + kr[n])
        tau = torch.zeros((nch, n.shape[1]), dtype=torch.float64, device=dev)
        for s0 in range(0, len(ch), part):
            sl = slice(s0, s0 + part)
            tau.index_add_(0, ch[sl], alpha[cell[sl]] * length[sl, None])
        v = torch.where(ok[:, None], 1.0 - torch.exp(-tau), 1.0) * wb[:, None]
        sums[r0:r0 + per, 0] = v.sum(0)
        sums[r0:r0 + per, 1] = (v * v).sum(0)
    s = sums.cpu().numpy()
    m = s[:, 0] / nch
    dr, rs2 = g.r_toa - g.r0, p["r_star"] ** 2
    per_g = (g.r0 ** 2 + 2.0 * dr * m) / rs2
    se = 2.0 * dr * np.sqrt(np.maximum(s[:, 1] / nch - m * m, 0.0) / nch) / rs2
    ng = 1 if hires else table.ng
    w = (np.ones(1) if hires else table.g_weights)[None, :]
    per_g, se = per_g.reshape(-1, ng), se.reshape(-1, ng)
    return dict(value=(w * per_g).sum(1)[:, None], stderr=np.sqrt((w * w * se * se).sum(1))[:, None], per_g=per_g[:, :, None],
                sums=s.reshape(-1, ng, 1, 2), counters=np.zeros((rows // ng, ng, 11)), l_tot=np.zeros((rows // ng, ng)))


def _trace_chords(g, n_b, n_alpha, seed, dev):
    """Segments (chord, cell, length) of the jittered chords along -x, all
    chords advanced together cell by cell; their weights b; which leave."""
    nch = n_b * n_alpha
    u, v = _philox(seed, 0, np.arange(nch, dtype=np.uint64), 0, 0)
    r0, rt = g.r0, g.r_toa
    b = r0 + (np.arange(nch) // n_alpha + u) * (rt - r0) / n_b
    al = 2.0 * math.pi * (np.arange(nch) % n_alpha + v) / n_alpha
    T = lambda a: torch.as_tensor(a, device=dev)  # noqa: E731
    x, y, z = T(np.sqrt(np.maximum(rt * rt - b * b, 0.0))), T(b * np.cos(al)), T(b * np.sin(al))
    R, la, lo = T(g.r_edges), T(g.lat_edges), T(g.lon_edges)
    ls2, lc2 = torch.sin(la) ** 2, torch.cos(la) ** 2
    los, loc = torch.sin(lo[:-1]), torch.cos(lo[:-1])
    find = lambda e, q: torch.clamp(torch.searchsorted(e, q, right=True) - 1, 0, len(e) - 2)  # noqa: E731
    j, i = find(la, torch.atan2(z, torch.sqrt(x * x + y * y))), find(lo, torch.atan2(y, x))
    k, ef = torch.full_like(j, g.nlay - 1), torch.zeros_like(j)
    act = torch.arange(nch, device=dev)
    ok = torch.zeros(nch, dtype=torch.bool, device=dev)
    inf = torch.tensor(math.inf, dtype=torch.float64, device=dev)
    out = []
    while len(act):
        rr, B = x * x + y * y + z * z, -x

        def cone(e, there, tol):
            tb = la[e]
            s2, c2 = ls2[e], lc2[e]
            A, bb, C = -s2, x * s2, z * z * c2 - (x * x + y * y) * s2
            disc = bb * bb - A * C
            q = -(bb + torch.where(bb >= 0.0, 1.0, -1.0) * torch.sqrt(torch.clamp(disc, min=0.0)))
            best = inf
            for s in (q / A, torch.where(q != 0.0, C / q, inf)):
                good = there & (tb != 0.0) & (disc >= 0.0) & (s >= tol) & (z * tb > 0.0)
                best = torch.minimum(best, torch.where(good, s, inf))
            return best

        ro, ri = R[k + 1], R[k]
        D = torch.sqrt(torch.clamp(B * B - (rr - ro * ro), min=0.0))
        s_out = torch.clamp(torch.where(B <= 0.0, D - B, -(rr - ro * ro) / (B + D)), min=0.0)
        Di = B * B - (rr - ri * ri)
        s_in = torch.where((B < 0.0) & (Di >= 0.0),
                           torch.clamp((rr - ri * ri) / (-B + torch.sqrt(torch.clamp(Di, min=0.0))), min=0.0), inf)
        tol = 1e-9 * torch.sqrt(rr)
        s_ll = cone(j, j > 0, torch.where(ef == 2, tol, 0.0))
        s_lh = cone(j + 1, j < g.nlat - 1, torch.where(ef == 3, tol, 0.0))

        def plane(e, sign):
            dn = los[e]  # (-1, 0, 0) . (-sin, cos, 0)
            s = torch.clamp(-(y * loc[e] - x * los[e]) / dn, min=0.0)
            return torch.where((sign * dn > 0.0) & (loc[e] * (x - s) + los[e] * y > 0.0), s, inf)

        far = torch.full_like(s_out, math.inf)
        s_wl, s_wh = (plane(i, -1.0), plane((i + 1) % g.nlon, 1.0)) if g.nlon > 1 else (far, far)
        s, f = torch.stack([s_out, s_in, s_ll, s_lh, s_wl, s_wh]).min(0)
        out.append((act, (k * g.nlat + j) * g.nlon + i, s))
        x = x - s
        k = k + (f == 0).long() - (f == 1).long()
        j = j - (f == 2).long() + (f == 3).long()
        i = (i - (f == 4).long() + (f == 5).long()) % g.nlon
        ef = f ^ 1
        ok[act[k >= g.nlay]] = True
        on = (k >= 0) & (k < g.nlay)
        act, x, y, z, i, j, k, ef = (a[on] for a in (act, x, y, z, i, j, k, ef))
    c, cell, s = (torch.cat([o[n] for o in out]) for n in range(3))
    return c, cell, s, T(b), ok
