"""The workloads whose speed this repository keeps an eye on.

One case is one call (or, for batches, one batched call) of a public entry
point on synthetic events of the shapes that the benchmark and the tests use:
TPC events tracked alone, in batches and as time frames, segments merged, the
calibration gradient, and ITS events.  The events are drawn on the GPU from
the distributions of the repository's generator (helices with log-uniform pT,
Gaussian smearing, uniform noise, doubled crossings, shuffled clusters), so
that a case is ready within a fraction of a second.
"""
import math
from functools import lru_cache
from types import SimpleNamespace

import numpy as np
import torch

from paper_1712_09434_amd import FitTracks, Tracker
from paper_1712_09434_amd.its import ItsTracker

C_LIGHT = 2.99792458e-3           # GeV / (T cm)
ROWS, WEDGES, SECTORS = 159, 18, 36
BZ, Z_MAX = 0.5, 250.0
TAN_A = math.tan(math.radians(10.0))
ROW_X = np.float32(85.0 + np.arange(ROWS) * (162.0 / 158.0))
SIG_Y, SIG_Z = 0.1, 0.15
ITS_INTS = ("tl0", "tl1", "ok", "cls", "ncls", "out_layer", "out_stave", "in_ok", "in_stave")


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # one sector (both drift sides of one wedge) of a quiet event, 17 k clusters: the
        # smallest call, as in a display or a per-sector test stand; launches and latency
        dict(name="track-sector", kind="track", primaries=200, secondaries=0, noise=0.01, doubling=0.0, sector=True,
             calib=False),
        # a minimum-bias event with a calibration installed, as every event after the
        # first turn of the feedback loop
        dict(name="track-minbias-calib", kind="track", primaries=1237, secondaries=0, noise=0.02, doubling=0.0,
             sector=False, calib=True),
        # a mid-central event (5000 primaries, 0.77 M clusters)
        dict(name="track-event", kind="track", primaries=5000, secondaries=0, noise=0.02, doubling=0.0, sector=False,
             calib=False),
        # a central Pb-Pb-shaped event: secondaries, noise, doubled clusters, 3.8 M clusters
        dict(name="track-central", kind="track", primaries=18000, secondaries=4000, noise=0.05, doubling=0.1,
             sector=False, calib=False),
        # 64 events of lognormal multiplicity in one call (12 M clusters): full chip, small rows
        dict(name="batch-64", kind="batch", events=64, primaries=1000, noise=0.02),
        # seven small events per call: an online farm that cannot wait for a long batch
        dict(name="batch-7-small", kind="batch", events=7, primaries=150, noise=0.02),
        # continuous readout: 24 collisions over six drift lengths, sliced, tracked and merged
        dict(name="frame-24", kind="frame", collisions=24, slices=6, primaries=1000, noise=0.02),
        # the sector merger on a central event's segments
        dict(name="merge-central", kind="merge", primaries=18000, secondaries=4000, noise=0.05, doubling=0.1),
        # the calibration gradient of one event's tracks, and of a calibration run of twenty
        dict(name="grad-event", kind="grad", events=1, primaries=5000),
        dict(name="grad-20", kind="grad", events=20, primaries=5000),
        # ITS standalone tracking: one pp-like event (latency), a batch of central ones
        dict(name="its-pp", kind="its", events=1, primaries=60, batch=False),
        dict(name="its-central-20", kind="its", events=20, primaries=3000, batch=True),
    ]


def draw(rng):
    def logu(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    kind = rng.choice(["track", "track", "track", "batch", "batch", "frame", "merge", "grad", "grad", "its", "its"])
    noise = round(rng.uniform(0.0, 0.05), 4)
    if kind == "track":
        if rng.random() < 0.2:
            return dict(kind=kind, primaries=logu(20, 700), secondaries=0, noise=noise, doubling=0.0, sector=True,
                        calib=False)
        n = logu(50, 18000)
        return dict(kind=kind, primaries=n, secondaries=int(n * rng.choice([0.0, 0.1, 0.22])), noise=noise,
                    doubling=rng.choice([0.0, 0.1]), sector=False, calib=rng.random() < 0.3)
    if kind == "batch":
        n = logu(50, 1000)
        return dict(kind=kind, events=min(logu(2, 64), 40000 // n), primaries=n, noise=noise)
    if kind == "frame":
        s = rng.randint(1, 8)
        c = rng.randint(1, 4 * s)
        return dict(kind=kind, collisions=c, slices=s, primaries=logu(50, min(2000, 24000 // c)), noise=noise)
    if kind == "merge":
        n = logu(100, 18000)
        return dict(kind=kind, primaries=n, secondaries=int(n * rng.choice([0.0, 0.22])), noise=noise,
                    doubling=rng.choice([0.0, 0.1]))
    if kind == "grad":
        e = rng.randint(1, 20)
        return dict(kind=kind, events=e, primaries=logu(50, 5000))
    if rng.random() < 0.5:
        return dict(kind="its", events=1, primaries=logu(10, 3000), batch=False)
    return dict(kind="its", events=rng.randint(2, 20), primaries=logu(20, 3000), batch=True)


# ------------------------------------------------------------------ the events
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 2654435761 % (1 << 62) + 17)
    opt = dict(generator=g, device="cuda", dtype=torch.float64)
    return SimpleNamespace(u=lambda n, a=0.0, b=1.0: a + (b - a) * torch.rand(n, **opt),
                           n=lambda n, s=1.0: s * torch.randn(n, **opt))


def _tracks(g, n, ev, prim=True, phi=2.0 * math.pi):
    pt = torch.exp(g.u(n, math.log(0.1), math.log(10.0)))
    q = torch.where(g.u(n) < 0.5, -1.0, 1.0)
    eta, phi0 = g.u(n, -0.9, 0.9), g.u(n, 0.0, phi)
    zero = torch.zeros(n, device="cuda", dtype=torch.float64)
    t = SimpleNamespace(ev=ev, k=q / pt, tgl=torch.sinh(eta), phi=phi0, x=zero, y=zero, z=zero,
                        prim=torch.full((n,), prim, device="cuda"))
    if not prim:   # displaced: vertex radius up to 60 cm
        rho, az = g.u(n, 0.0, 60.0), g.u(n, 0.0, 2.0 * math.pi)
        t.x, t.y, t.z = rho * torch.cos(az), rho * torch.sin(az), rho * torch.sinh(g.u(n, -0.9, 0.9))
    return t


def _join(a, b):
    return SimpleNamespace(**{k: torch.cat([v, getattr(b, k)]) for k, v in vars(a).items()})


def _events(g, counts, secondaries, noise, doubling, sector):
    """Clusters of len(counts) TPC events, shuffled within each event: track (-1 for noise), event,
    sector, row, x, y, z (FP64), and whether a cluster is the first of a crossing on the outward leg."""
    dev = "cuda"
    phi = math.radians(20.0) if sector else 2.0 * math.pi
    cnt = torch.tensor(counts, device=dev)
    eid = torch.arange(len(counts), device=dev)
    t = _tracks(g, int(sum(counts)), torch.repeat_interleave(eid, cnt), True, phi)
    if secondaries:
        t = _join(t, _tracks(g, secondaries, torch.zeros(secondaries, dtype=torch.int64, device=dev), False, phi))
    X = torch.tensor(ROW_X, device=dev, dtype=torch.float64)
    kap = (-C_LIGHT * BZ * t.k)[:, None]
    parts = []
    for w in range(1 if sector else WEDGES):
        a = (w + 0.5) * math.radians(20.0)
        xl, yl, psi = t.x * math.cos(a) + t.y * math.sin(a), -t.x * math.sin(a) + t.y * math.cos(a), (t.phi - a)[:, None]
        v = torch.sin(psi) + kap * (X - xl[:, None])
        base = torch.asin(v.clamp(-1.0, 1.0))
        for out, th in ((True, base), (False, math.pi - base)):
            dpsi = torch.remainder(torch.where(kap > 0, th - psi, psi - th), 2.0 * math.pi)
            ell = dpsi / kap.abs()
            y = yl[:, None] - (torch.cos(th) - torch.cos(psi)) / kap
            z = t.z[:, None] + t.tgl[:, None] * ell
            ok = (v.abs() <= 1.0) & (ell > 0) & (dpsi <= math.pi) & (y.abs() <= X * TAN_A) & (z.abs() <= Z_MAX)
            i, r = torch.nonzero(ok, as_tuple=True)
            zz = z[i, r]
            s = torch.zeros_like(i) if sector else w + WEDGES * (zz < 0)
            parts.append((i, t.ev[i], s, r, y[i, r], zz, torch.full_like(i, out, dtype=torch.bool)))
    trk, ev, sec, row, y, z, first = (torch.cat(p) for p in zip(*parts))
    yt, zt, n = y, z, trk.numel()
    y, z = yt + g.n(n, SIG_Y), zt + g.n(n, SIG_Z)
    if doubling:
        m = torch.nonzero(g.u(n) < doubling).squeeze(1)
        y, z = torch.cat([y, yt[m] + g.n(m.numel(), SIG_Y)]), torch.cat([z, zt[m] + g.n(m.numel(), SIG_Z)])
        trk, ev, sec, row = (torch.cat([v, v[m]]) for v in (trk, ev, sec, row))
        first = torch.cat([first, torch.zeros_like(m, dtype=torch.bool)])
    m = int(round(noise * trk.numel()))
    if m:
        # noise follows the events' sizes
        e = ev[(g.u(m) * trk.numel()).long()]
        r = (g.u(m) * ROWS).long()
        s = torch.zeros_like(r) if sector else (g.u(m) * SECTORS).long()
        zu = g.u(m, 0.0, Z_MAX)
        flip = g.u(m) < 0.5 if sector else s >= WEDGES
        y, z = torch.cat([y, g.u(m, -1.0, 1.0) * X[r] * TAN_A]), torch.cat([z, torch.where(flip, -zu, zu)])
        trk, ev, sec, row = torch.cat([trk, torch.full_like(r, -1)]), torch.cat([ev, e]), torch.cat([sec, s]), torch.cat([row, r])
        first = torch.cat([first, torch.zeros_like(r, dtype=torch.bool)])
    o = torch.argsort(ev + g.u(trk.numel()))
    return t, SimpleNamespace(trk=trk[o], ev=ev[o], sec=sec[o], row=row[o], x=X[row[o]], y=y[o], z=z[o], first=first[o])


def _soa(c, m=None, z=None):
    m = slice(None) if m is None else m
    return (c.x[m].float().contiguous(), c.y[m].float().contiguous(), (c.z if z is None else z)[m].float().contiguous(),
            c.row[m].to(torch.int16).contiguous(), c.sec[m].to(torch.uint8).contiguous())


def _theta(g, scale):
    """drift scale, time offset (cm), radial map (cm), spread as an expected miscalibration."""
    return (scale * torch.cat([g.n(SECTORS, 2e-3), g.n(SECTORS, 0.1), g.u(SECTORS * 64, -0.3, 0.3)])).float()


def _multiplicities(n, median):
    r = np.random.default_rng([n, median])
    return [int(v) for v in np.clip(np.exp(r.normal(math.log(median), math.log(400.0) / 6.0, n)), 20, 5 * median)]


def _fit_tracks(g, t, c):
    """The hit lists of the primaries' segments with at least 40 hits that start on one of the first 11
    rows: what is left of tracks matched to the inner detector."""
    m = torch.nonzero(c.first & (c.trk >= 0) & t.prim[c.trk.clamp(min=0)]).squeeze(1)
    key = (c.trk[m] * SECTORS + c.sec[m]) * ROWS + c.row[m]
    o = torch.argsort(key)
    m, seg = m[o], torch.div(key[o], ROWS, rounding_mode="floor")
    _, inv, n = torch.unique_consecutive(seg, return_inverse=True, return_counts=True)
    start = torch.cumsum(n, 0) - n
    keep = (n >= 40) & (c.row[m[start]] <= 10)
    m, n, trk = m[keep[inv]], n[keep], c.trk[m[start]][keep]
    off = torch.zeros(n.numel() + 1, dtype=torch.int32, device="cuda")
    off[1:] = torch.cumsum(n, 0)
    k = (t.k[trk] * (1.0 + g.n(trk.numel(), 0.02))).float()
    return FitTracks(clusters=_soa(c), hit_off=off, hit_id=m.to(torch.int32), k_prior=k,
                     ext_tgl=(t.tgl[trk] + g.n(trk.numel(), 1e-3)).float(),
                     use_vertex=torch.ones(trk.numel(), dtype=torch.uint8, device="cuda"))


ITS_R = [3.9, 7.6, 15.0, 23.9, 38.0, 43.0]
ITS_GEOM = SimpleNamespace(n_layers=6, radius=ITS_R, n_staves=[20, 40, 14, 22, 34, 38], bz=BZ,
                           half_z=[14.1, 14.1, 22.2, 29.7, 43.1, 48.9],
                           x_over_x0=[0.0114, 0.0114, 0.0113, 0.0126, 0.0083, 0.0086],
                           sigma_y=[0.0012, 0.0012, 0.0035, 0.0035, 0.0020, 0.0020],
                           sigma_z=[0.0100, 0.0100, 0.0025, 0.0025, 0.0830, 0.0830])


def _its_event(g, n):
    """Clusters of one ITS event: n primaries through six layers of staves with multiple scattering."""
    dev = "cuda"
    v = [float(g.n(1, s)) for s in (0.005, 0.005, 5.0)]
    t = _tracks(g, n, torch.zeros(n, dtype=torch.int64, device=dev))
    X, Y, Z = (torch.full((n,), a, device=dev, dtype=torch.float64) for a in v)
    psi, tgl, kap = t.phi, t.tgl, -C_LIGHT * BZ * t.k
    alive = torch.ones(n, dtype=torch.bool, device=dev)
    parts = []
    for l in range(6):
        r, ns = ITS_R[l], ITS_GEOM.n_staves[l]
        dk = 2.0 * math.pi / ns
        far = (r - torch.hypot(X, Y)).clamp(min=0.0)
        k0 = torch.floor(torch.remainder(torch.atan2(Y + far * torch.sin(psi), X + far * torch.cos(psi)), 2 * math.pi) / dk)
        hit = torch.zeros_like(alive)
        ky, yy, zz, pp = torch.zeros_like(X), torch.zeros_like(X), torch.zeros_like(X), psi
        for d in (0, -1, 1):
            k = torch.remainder(k0 + d, ns)
            a = (k + 0.5) * dk
            xl, yl, p0 = X * torch.cos(a) + Y * torch.sin(a), -X * torch.sin(a) + Y * torch.cos(a), psi - a
            s = torch.sin(p0) + kap * (r - xl)
            th = torch.asin(s.clamp(-1.0, 1.0))
            dpsi = torch.remainder(torch.where(kap > 0, th - p0, p0 - th), 2.0 * math.pi)
            y1, z1 = yl - (torch.cos(th) - torch.cos(p0)) / kap, Z + tgl * dpsi / kap.abs()
            ok = alive & ~hit & (s.abs() <= 1.0) & (dpsi <= math.pi) & (y1.abs() <= r * math.tan(math.pi / ns)) & (
                z1.abs() <= ITS_GEOM.half_z[l])
            ky, yy, zz, pp = (torch.where(ok, b, c) for b, c in ((k, ky), (y1, yy), (z1, zz), (th + a, pp)))
            hit |= ok
        alive = alive & hit
        i = torch.nonzero(alive).squeeze(1)
        parts.append((torch.full_like(i, l), ky[i], yy[i] + g.n(i.numel(), ITS_GEOM.sigma_y[l]),
                      zz[i] + g.n(i.numel(), ITS_GEOM.sigma_z[l])))
        a = (ky + 0.5) * dk
        X, Y, Z, psi = r * torch.cos(a) - yy * torch.sin(a), r * torch.sin(a) + yy * torch.cos(a), zz, pp
        lam = torch.atan(tgl)
        depth = ITS_GEOM.x_over_x0[l] / (torch.cos(lam) * torch.cos(psi - a).abs().clamp(min=1e-3))
        th0 = 0.0136 * torch.cos(lam) * kap.abs() / (C_LIGHT * BZ) * torch.sqrt(depth) * (1.0 + 0.038 * torch.log(depth))
        lam2 = (lam + th0 * g.n(n)).clamp(-1.5, 1.5)
        psi, kap, tgl = psi + th0 * g.n(n) / torch.cos(lam), kap * torch.cos(lam) / torch.cos(lam2), torch.tan(lam2)
    lay, stv, y, z = (torch.cat(p) for p in zip(*parts))
    m = int(round(0.01 * lay.numel()))
    nl = (g.u(m) * 6).long()
    ns, rr, hz = (torch.tensor(a, device=dev, dtype=torch.float64)[nl] for a in (ITS_GEOM.n_staves, ITS_R, ITS_GEOM.half_z))
    lay, stv = torch.cat([lay, nl]), torch.cat([stv, torch.floor(g.u(m) * ns)])
    y, z = torch.cat([y, g.u(m, -1.0, 1.0) * rr * torch.tan(math.pi / ns)]), torch.cat([z, g.u(m, -1.0, 1.0) * hz])
    o = torch.argsort(g.u(lay.numel()))
    x = torch.tensor(ITS_R, device=dev, dtype=torch.float32)[lay[o]]
    return (x, y[o].float(), z[o].float(), lay[o].to(torch.int8), stv[o].to(torch.int16))


# --------------------------------------------------------- what a program holds
def _new_tracker():
    return Tracker(ROW_X, float(np.float32(TAN_A)), Z_MAX, BZ, SECTORS)


@lru_cache(maxsize=None)
def _tracker():
    """The tracker of a program that tracks one event after the other."""
    return _new_tracker()


@lru_cache(maxsize=None)
def _its_tracker():
    return ItsTracker(ITS_GEOM)


def _clusters(case):
    """The expected number of clusters of a TPC case, about 150 a track."""
    kind = case["kind"]
    tracks = case["primaries"] * (84 / 150 if case.get("sector") else 1.0) + case.get("secondaries", 0)
    if kind in ("batch", "frame"):
        tracks = sum(_multiplicities(case["events" if kind == "batch" else "collisions"], case["primaries"]))
    return 150 * tracks * (1.0 + case["noise"]) * (1.0 + case.get("doubling", 0.0))


def _buffers(case):
    """The flat buffers, of a size fixed by the case, that results are shipped in (zero past their end)."""
    def z(dtype, *shape):
        return torch.zeros(*shape, dtype=dtype, device="cuda")

    f32, i32 = torch.float32, torch.int32
    if case["kind"] == "its":
        n = int(case["events"] * (1.2 * case["primaries"] + 20))
        return SimpleNamespace(ints=z(i32, 14 * n), chi2=z(f32, n), out=z(f32, n, 21), inw=z(f32, n, 20))
    hits = int(1.3 * _clusters(case)) + 2000
    n = hits // 25 + 100
    return SimpleNamespace(sector=z(torch.uint8, n), state=z(f32, n, 7), cov=z(f32, n, 15), chi2=z(f32, n),
                           ints=z(i32, 2 * n + hits + 64))


def prepare(case, seed):
    g, kind = _gen(seed), case["kind"]
    st = SimpleNamespace(kind=kind, tracker=None)
    if kind != "grad":
        st.to = _buffers(case)
    if kind in ("track", "merge"):
        _, c = _events(g, [case["primaries"]], case["secondaries"], case["noise"], case["doubling"],
                       case.get("sector", False))
        st.tracker, st.event = _tracker(), _soa(c)
        if case.get("calib"):
            st.tracker = _new_tracker()
            st.tracker.set_calib(_theta(g, 0.5))
        if kind == "merge":
            st.segments = st.tracker.track(*st.event)
    elif kind == "batch":
        counts = _multiplicities(case["events"], case["primaries"])
        _, c = _events(g, counts, 0, case["noise"], 0.0, False)
        at = torch.searchsorted(c.ev, torch.arange(len(counts) + 1, device="cuda")).tolist()
        st.tracker, st.events = _tracker(), [_soa(c, slice(a, b)) for a, b in zip(at, at[1:])]
    elif kind == "frame":
        counts = _multiplicities(case["collisions"], case["primaries"])
        _, c = _events(g, counts, 0, case["noise"], 0.0, False)
        length = case["slices"] * Z_MAX
        when = g.u(len(counts), 0.0, length)
        side = torch.where(c.sec < WEDGES, 1.0, -1.0)
        tau = when[c.ev] + (Z_MAX - side * c.z)
        m = torch.nonzero((tau >= 0.0) & (tau.float() < length)).squeeze(1)
        m = m[torch.argsort(g.u(m.numel()))]
        st.tracker, st.frame, st.slices = _tracker(), _soa(c, m, tau), case["slices"]
    elif kind == "grad":
        t, c = _events(g, [case["primaries"]] * case["events"], 0, 0.02, 0.0, False)
        st.tracker, st.fit, st.theta = _tracker(), _fit_tracks(g, t, c), _theta(g, 0.5)
    else:
        st.tracker = _its_tracker()
        st.events = [_its_event(g, case["primaries"]) for _ in range(case["events"])]
        st.plan = None   # (one event: tracked as it comes)
        if case["batch"]:
            st.plan = st.tracker.prepare_batch(st.events)
    torch.cuda.synchronize()
    return st


def _put(to, parts, dim=0):
    """The parts, one behind the other, at the start of the buffer `to`."""
    n = sum(p.shape[0] for p in parts) if dim == 0 else parts[0].shape[0]
    torch.cat(parts, dim, out=to[:n])


def _ship(to, out, more=()):
    """The tracks `out` of one or more events in flat buffers: records, then ndf, hit offsets and hit ids
    (and `more`), the events one behind the other."""
    state = [torch.cat([t.x_ref[:, None], t.p, t.k_prior[:, None]], 1) for t in out]
    _put(to.state, state)
    _put(to.sector, [t.sector for t in out])
    _put(to.cov, [t.cov for t in out])
    _put(to.chi2, [t.chi2 for t in out])
    _put(to.ints, [getattr(t, f) for f in ("ndf", "hit_off", "hit_id") for t in out] + list(more))
    return vars(to)


def _ship_its(to, out):
    _put(to.ints, [getattr(r, f).flatten() for f in ITS_INTS for r in out])
    _put(to.chi2, [r.chi2 for r in out])
    # the states of accepted tracks and of successful inward fits (the others are not written)
    cat = (lambda f: getattr(out[0], f)) if len(out) == 1 else lambda f: torch.cat([getattr(r, f) for r in out])
    ok, iok = cat("ok"), cat("in_ok")
    n, zero = ok.numel(), to.chi2[-1]   # (past the results' end)
    torch.where(ok[:, None] != 0, torch.cat([cat("out_x")[:, None], cat("out_p"), cat("out_cov")], 1), zero, out=to.out[:n])
    torch.where(iok[:, None] != 0, torch.cat([cat("in_p"), cat("in_cov")], 1), zero, out=to.inw[:n])
    scalars = [[r.n_pairs, r.peak, r.vz_ok, r.vz, r.vfit_ok, r.vfit_n, r.vfit_sumw, *r.vertex] for r in out]
    return dict(vars(to), event=np.array(scalars, dtype=np.float64))


def run(st):
    if st.kind == "track":
        return _ship(st.to, [st.tracker.track(*st.event)])
    if st.kind == "merge":
        m, links = st.tracker.merge(st.segments, st.event, links=True)
        return _ship(st.to, [m], [links])
    if st.kind == "batch":
        return _ship(st.to, st.tracker.track_batch(st.events))
    if st.kind == "frame":
        return _ship(st.to, [st.tracker.track_timeframe(*st.frame, Z_MAX, st.slices)])
    if st.kind == "grad":
        chi2, ndf, grad = st.tracker.refit_grad(st.fit, st.theta)
        return dict(chi2=chi2, ndf=ndf, grad=grad)
    return _ship_its(st.to, st.plan() if st.plan else [st.tracker.track(*st.events[0])])


def work(case):
    kind = case["kind"]
    if kind == "its":
        # six clusters of 15 bytes in, one tracklet of 226 bytes out; two fits of six layers
        n = case["events"] * case["primaries"]
        return {"bytes": n * (6 * 15 + 226 * 0.85), "flops": n * 2 * 6 * 900}
    if kind == "grad":
        # per hit: id, coordinates, sector in; forward and reverse sweep.  0.8 tracks of 130 hits a primary
        n = case["events"] * case["primaries"] * 0.8
        return {"bytes": n * (130 * 17 + 13) + 2376 * 12, "flops": n * 130 * 3000}
    n = _clusters(case)
    seg = 0.93 * n * 4 + n / 110 * 101   # hit ids and track records
    if kind == "merge":
        # segments and their clusters in, merged tracks out; one more fit of the joined third
        return {"bytes": 0.93 * n * 14 + 1.8 * seg, "flops": 0.6 * n * 350}
    # clusters in, tracks out; links of about eight pairs, following and final fit
    return {"bytes": 15 * n + seg, "flops": n * (8 * 20 + 2 * 350) + (0.6 * n * 350 if kind == "frame" else 0.0)}


# ------------------------------------------------------------------ 64 bits
def _bsplines(u):
    """The eight clamped uniform cubic B-splines at u, by Cox-de Boor."""
    t = [0.0, 0.0, 0.0, 0.0, 0.2, 0.4, 0.6, 0.8, 1.0, 1.0, 1.0, 1.0]
    u = u.clamp(0.0, 1.0)
    N = [((t[i] <= u) & (u < t[i + 1])).double() for i in range(11)]
    N[7] = torch.where(u >= 1.0, 1.0, N[7])
    for p in range(1, 4):
        N = [sum(f * b for f, b in (((u - t[i]) / (t[i + p] - t[i]) if t[i + p] > t[i] else None, N[i]),
                                    ((t[i + p + 1] - u) / (t[i + p + 1] - t[i + 1]) if t[i + p + 1] > t[i + 1] else None,
                                     N[i + 1])) if f is not None) + 0.0 * u for i in range(11 - p)]
    return N


def _asinc(u2):
    return 1.0 + u2 * (1 / 6 + u2 * (3 / 40 + u2 * (5 / 112 + u2 * (35 / 1152))))


def _step(p, C, dx, use):
    """Helix step by dx of the states p [T, 5] with covariances C [T, 5, 5] where `use`; also which succeeded."""
    kf = -C_LIGHT * BZ
    y, z, s0, t, k = p.unbind(1)
    dx = torch.where(use, dx, 1.0)
    kap, f = kf * k, kf * dx
    s1 = s0 + kap * dx
    ok = use & (s1.abs() < 0.99)
    s1 = torch.where(ok, s1, s0)
    c0, c1 = torch.sqrt(1 - s0 * s0), torch.sqrt(1 - s1 * s1)
    tn = (s0 + s1) / (c0 + c1)
    dy = dx * tn
    d = torch.sign(dx) * torch.sqrt(dx * dx + dy * dy)
    u = 0.5 * kap * d
    gg, gp = _asinc(u * u), u * (1 / 3 + u * u * (3 / 10 + u * u * (15 / 56 + u * u * (35 / 144))))
    l = d * gg
    t0, t1 = s0 / c0, s1 / c1
    a, b = dx * (2 + tn * (t0 + t1)) / (c0 + c1), dx * f * (1 + tn * t1) / (c0 + c1)
    ds, dk = dy * a / d, dy * b / d
    ls, lk = ds * gg + d * gp * 0.5 * kap * ds, dk * gg + d * gp * 0.5 * (kf * d + kap * dk)
    o, i = torch.zeros_like(a), torch.ones_like(a)
    F = torch.stack([i, o, a, o, b, o, i, t * ls, l, t * lk, o, o, i, o, f, o, o, o, i, o, o, o, o, o, i], 1).view(-1, 5, 5)
    q = torch.stack([y + dy, z + t * l, s1, t, k], 1)
    # (products by sums: no batched matrix product)
    M = (F[:, :, :, None] * C[:, None, :, :]).sum(2)
    Q = (M[:, :, None, :] * F[:, None, :, :]).sum(3)
    return torch.where(ok[:, None], q, p), torch.where(ok[:, None, None], Q, C), ok


def _update(p, C, m, var, use):
    """Kalman update with the measurement m [T, 2] of (y, z)."""
    r = m - p[:, :2]
    S00, S01, S11 = C[:, 0, 0] + var[0], C[:, 0, 1], C[:, 1, 1] + var[1]
    det = S00 * S11 - S01 * S01
    W = torch.stack([S11, -S01, -S01, S00], 1).view(-1, 2, 2) / det[:, None, None]
    K = (C[:, :, :2, None] * W[:, None, :, :]).sum(2)
    q = p + (K * r[:, None, :]).sum(2)
    Q = C - (K[:, :, :, None] * C[:, None, :2, :]).sum(2)
    chi = (r[:, :, None] * W * r[:, None, :]).sum((1, 2))
    return torch.where(use[:, None], q, p), torch.where(use[:, None, None], Q, C), torch.where(use, chi, 0.0)


def _exact_grad(fit, theta):
    """Total chi2 of the refit of every hit list (outermost hit first, then the vertex and the external
    tan lambda) under the correction theta, and its derivative by automatic differentiation, in FP64."""
    x, y, z = (v.double() for v in fit.clusters[:3])
    sec, off, ids = fit.clusters[4].long(), fit.hit_off.long(), fit.hit_id.long()
    n = off[1:] - off[:-1]
    th = theta.double().requires_grad_(True)
    # correct every hit
    s = sec[ids]
    side = torch.where(s < WEDGES, 1.0, -1.0)
    hx, hy, hz = x[ids], y[ids], z[ids]
    Ba, Bb = _bsplines((hx - float(ROW_X[0])) / float(ROW_X[-1] - ROW_X[0])), _bsplines((hy / hx + TAN_A) / (2 * TAN_A))
    dl, tau, cm = th[:SECTORS][s], th[SECTORS:2 * SECTORS][s], th[2 * SECTORS:].view(SECTORS, 64)[s]
    hz = side * (Z_MAX - (1 + dl) * (Z_MAX - side * hz - tau))
    hx = hx + (cm * (torch.stack(Ba, 1)[:, :, None] * torch.stack(Bb, 1)[:, None, :]).flatten(1)).sum(1)
    # [T, steps] outermost first
    step = torch.arange(int(n.max()), device="cuda")
    live = step[None, :] < n[:, None]
    at = (off[1:, None] - 1 - step[None, :]).clamp(min=0)
    H = torch.stack([hx[at], hy[at], hz[at]], 2)
    d = H[:, 0] - H[:, 2]
    rho = torch.sqrt(d[:, 0] ** 2 + d[:, 1] ** 2)
    p = torch.stack([H[:, 0, 1], H[:, 0, 2], d[:, 1] / rho, d[:, 2] / rho, fit.k_prior.double()], 1)
    C = torch.diag(torch.tensor([SIG_Y ** 2, SIG_Z ** 2, 0.25, 0.25, 100.0], device="cuda", dtype=torch.float64))
    C = C.expand(p.shape[0], 5, 5)
    good = p[:, 2].abs() < 0.99
    chi, xc = torch.zeros_like(rho), H[:, 0, 0]
    for k in range(1, H.shape[1]):
        use = live[:, k] & good
        p, C, ok = _step(p, C, H[:, k, 0] - xc, use)
        good = good & (ok | ~use)
        p, C, c = _update(p, C, H[:, k, 1:], (SIG_Y ** 2, SIG_Z ** 2), ok)
        chi, xc = chi + c, torch.where(ok, H[:, k, 0], xc)
    # to the beam axis in steps of at most 10 cm; where a step is refused the hits alone count
    nsub = torch.ceil(xc / 10.0)
    vert, q, Q, xv = good.clone(), p, C, xc
    for m in range(int(nsub.max()) - 1, -1, -1):
        use = vert & (nsub > m)
        q, Q, ok = _step(q, Q, 10.0 * m - xv, use)
        vert = vert & (ok | ~use)
        xv = torch.where(ok, 10.0 * m, xv)
    q, Q, c = _update(q, Q, torch.zeros_like(q[:, :2]), (0.01 ** 2, 0.01 ** 2), vert)
    r = fit.ext_tgl.double() - q[:, 3]
    c = c + torch.where(vert, r * r / (Q[:, 3, 3] + 1e-3 ** 2), 0.0)
    total = torch.where(good, chi + c, 0.0).sum()
    grad, = torch.autograd.grad(total, th)
    return float(total.detach()), grad


def exact(case, seed):
    # the tracks, links and fits of the other cases follow from choices (which cluster, which link) that
    # are made on FP32 values by definition: they have no value in 64 bits
    if case["kind"] != "grad":
        return None
    st = prepare(case, seed)
    chi2, grad = _exact_grad(st.fit, st.theta)
    return dict(chi2=chi2, ndf=None, grad=grad)
