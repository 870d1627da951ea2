"""Performance cases of the transient F-statistic maps.

Each case is one call that a search pipeline makes through the public entry
points (Context.fmap, Batch.run, submit / poll, logB), over the range that
such a pipeline meets: one short candidate whose map takes as long as its
launches, the 1-bin map of a 100-day observation, hundreds of frequency bins
that share their antenna patterns, grids on and off the SFT slots, both
window types, every precision, batches and bursts of uneven candidates.

Atoms are simulated as the pipeline's: per-SFT antenna products of a sidereal
day and Gaussian noise on a grid of 1800 s slots with gaps; the first bin
carries a weak transient in one case out of two.  The resident atoms, the
planned batch and the map's buffer are what such a program keeps.

Results: the whole 2F map where the call writes one, and max 2F and logB of
every bin.  The argmax (t0, tau) of a bin is an index into that map, defined
up to near-ties (cells whose 2F is equal to within the precision of the sums
are equally right), so the maximum itself is returned and not its place.  Max
2F has the precision of the sums: float32 where the caller asks for single
precision or split half-precision sums, float64 for float64 sums.  The logB
of a map call adds single-precision exponentials in every mode (float32); the
logB of a stored map is float64 throughout.
"""
import math
import random
import types

import numpy as np
import torch

T = 1800                   # SFT length (s)
SIDEREAL = 86164.0
ARENA = 24 << 30           # the context's device arena: many resident candidates
DEGENERATE = 1e-10         # 2F = 0 where D <= this * A * B

_CTX = None


def _ctx():
    """The program's one context."""
    global _CTX
    if _CTX is None:
        import paper_1805_05652_amd as tf
        _CTX = tf.Context(0, arena_bytes=ARENA)
    return _CTX


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # one short candidate, one bin: the smallest rect call, all latency
        dict(name="rect_small", call="fmap", window="rect", prec="fp32", slots=200, gaps=0.10, bins=1,
             grid="slots", step=1, n_t0=100, n_tau=199),
        # a quick look at one candidate with the decaying window: the smallest exp call
        dict(name="exp_small", call="fmap", window="exp", prec="fp32", slots=300, gaps=0.10, bins=2,
             grid="linspace", step=0, n_t0=64, n_tau=48),
        # the 1-bin map of a 104-day observation, tau to 30 days (the headline workload)
        dict(name="exp_1bin", call="fmap", window="exp", prec="fp32", slots=5000, gaps=0.15, bins=1,
             grid="days30", step=1, n_t0=1000, n_tau=1000),
        # a narrow band around a pulsar: many bins, rows off the slots, the
        # default precision
        dict(name="exp_64bins", call="fmap", window="exp", prec="fp32", slots=3001, gaps=0.12, bins=64,
             grid="linspace", step=0, n_t0=611, n_tau=703),
        # a wide band in the mixed precision made for it
        dict(name="exp_256bins_f16x3", call="fmap", window="exp", prec="f16x3", slots=2000, gaps=0.10, bins=256,
             grid="slots", step=1, n_t0=500, n_tau=500),
        # the same band with rectangular windows: the map's bytes
        dict(name="rect_256bins", call="fmap", window="rect", prec="fp32", slots=2000, gaps=0.10, bins=256,
             grid="slots", step=1, n_t0=500, n_tau=500),
        # a candidate checked in double precision, ragged sizes
        dict(name="exp_fp64", call="fmap", window="exp", prec="fp64", slots=1501, gaps=0.20, bins=5,
             grid="linspace", step=0, n_t0=401, n_tau=299),
        # the double-precision recurrence on a regular grid
        dict(name="exp_recur64", call="fmap", window="exp", prec="recur64", slots=4000, gaps=0.15, bins=3,
             grid="days30", step=2, n_t0=1000, n_tau=800),
        # follow-up of uneven candidates as one planned batch, default precision
        dict(name="batch_fp32", call="batch", prec="fp32", count=24, max_slots=8000, max_grid=1500, max_bins=16),
        # the same kind of batch in the mixed precision
        dict(name="batch_f16x3", call="batch", prec="f16x3", count=32, max_slots=8000, max_grid=1500, max_bins=16),
        # a burst of served requests, submitted at once and polled to the last
        dict(name="serve_burst", call="serve", prec="f16x3", count=16, max_slots=6000, max_grid=1200, max_bins=48),
        # logB of a band's stored maps
        dict(name="logB_maps", call="logB", maps=128, n_t0=500, n_tau=500),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw(rng):
    kind = rng.choice(["fmap", "fmap", "fmap", "fmap", "fmap", "batch", "serve", "logB"])
    if kind == "logB":
        return dict(call="logB", maps=_log_int(rng, 1, 128), n_t0=_log_int(rng, 50, 1000), n_tau=_log_int(rng, 50, 1000))
    if kind == "batch":
        return dict(call="batch", prec=rng.choice(["fp32", "f16x3"]), count=rng.randint(4, 32),
                    max_slots=_log_int(rng, 1500, 8000), max_grid=_log_int(rng, 300, 1500), max_bins=rng.randint(3, 16))
    if kind == "serve":
        return dict(call="serve", prec=rng.choice(["fp32", "f16x3"]), count=rng.randint(4, 16),
                    max_slots=_log_int(rng, 1000, 6000), max_grid=_log_int(rng, 300, 1200), max_bins=rng.randint(4, 48))
    window = rng.choice(["rect", "exp", "exp", "exp"])
    prec = rng.choice(["fp32", "fp32", "fp32", "f16x3", "fp64", "recur64"]) if window == "exp" else "fp32"
    slots = _log_int(rng, 200, 8000)
    grid = rng.choice(["slots", "linspace", "days30"])
    if prec == "recur64" and grid == "linspace":
        grid = "slots"
    hi = min(slots - 2, 1500)
    n_t0, n_tau = _log_int(rng, 50, hi), _log_int(rng, 40, hi)
    step = 0 if grid == "linspace" else max(1, min(rng.randint(1, 4), slots // n_t0))
    return dict(call="fmap", window=window, prec=prec, slots=slots, gaps=round(rng.uniform(0.0, 0.3), 3),
                bins=_log_int(rng, 1, 256), grid=grid, step=step, n_t0=n_t0, n_tau=n_tau)


def draw(rng):
    """One more case of the same ranges: no more cells, window terms or bytes
    than the largest listed case has."""
    most = [_cost(c) for c in listed()]
    top = [max(m[i] for m in most) for i in range(3)]
    while True:
        c = _draw(rng)
        if all(v <= t for v, t in zip(_cost(c), top)):
            return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _grid(case_grid, slots, step, n_t0, n_tau):
    """(t0, tau, regular t0 or None, regular tau or None) of a grid over
    `slots` slots: rows every `step` slots and tau every slot; or tau to 30
    days in whole seconds; or both evenly spaced over the data, off the slots."""
    td = slots * T
    if case_grid == "linspace":
        t0 = np.unique(np.round(np.linspace(0, td - 2 * T, n_t0)).astype(np.int64))
        tau = np.unique(np.round(np.linspace(2 * T, td, n_tau)).astype(np.int64))
        return t0, tau, None, None
    t0 = T * step * np.arange(n_t0, dtype=np.int64)
    if case_grid == "slots":
        return t0, T * (2 + np.arange(n_tau, dtype=np.int64)), (0, T * step, n_t0), (2 * T, T, n_tau)
    hi = max(30 * 86400, 2 * T + 7 * n_tau)
    tau = 2 * T + np.round(np.arange(n_tau) * ((hi - 2 * T) / max(n_tau - 1, 1))).astype(np.int64)
    return t0, tau, (0, T * step, n_t0), None


def _window(kind, grid):
    t0, tau, r0, r1 = grid
    return types.SimpleNamespace(kind=kind, t0=t0, tau=tau, t0_regular=r0, tau_regular=r1)


def _atoms(seed, slots, gaps, bins):
    """Per-SFT antenna products and matched-filter values: sidereal antenna
    patterns, unit complex Gaussian noise, gaps inside the span; odd seeds
    add a decaying transient to the first bin.  Single-precision values."""
    rng = np.random.default_rng(seed)
    keep = np.ones(slots, dtype=bool)
    drop = int(round(gaps * slots))
    if drop:
        keep[1 + rng.choice(slots - 2, size=min(drop, slots - 4), replace=False)] = False
    ts = np.nonzero(keep)[0].astype(np.int64) * T
    while True:
        pa, pb = rng.uniform(0, 2 * math.pi, 2)
        if abs(math.cos(pb - pa)) >= 0.2:
            break
    ph = 2 * math.pi * ts / SIDEREAL
    a, b = 0.5 * np.cos(ph + pa), 0.5 * np.sin(ph + pb)
    x = rng.standard_normal((bins, ts.size, 2)) * math.sqrt(0.5)
    x = x[..., 0] + 1j * x[..., 1]
    if seed % 2:
        t0, tau = T * int(rng.integers(0, slots // 2)), T * int(rng.integers(4, max(5, slots // 6)))
        on = (ts >= t0) & (ts < t0 + 3 * tau)
        x[0] += 0.25 * np.exp(1j * rng.uniform(0, 6.28)) * np.where(on, np.exp(-np.where(on, ts - t0, 0) / tau), 0) * (a - 1j * b)
    fa, fb = (a * x).astype(np.complex64), (b * x).astype(np.complex64)
    f = [np.stack([v.real, v.imag], -1).astype(np.float64) for v in (fa, fb)]
    return types.SimpleNamespace(ts=ts, a2=a * a, b2=b * b, ab=a * b, fa=f[0], fb=f[1], bins=bins)


def _shapes(case):
    """Shapes of the maps of a batch or burst: slots log-uniform, grids and
    bins uniform, windows in turn.  They follow from the case alone, as the
    candidates of one search do; the data come from the seed."""
    rng = random.Random("%s %d %d %d %d" % (case["call"], case["count"], case["max_slots"], case["max_grid"], case["max_bins"]))
    out = []
    for i in range(case["count"]):
        slots = _log_int(rng, 200 if case["call"] == "serve" else 500, case["max_slots"])
        out.append(dict(window=("rect", "exp")[i % 2], slots=slots, gaps=rng.uniform(0.0, 0.3), bins=rng.randint(1, case["max_bins"]),
                        n_t0=min(rng.randint(100, case["max_grid"]), slots - 1),
                        n_tau=min(rng.randint(100, case["max_grid"]), slots - 1)))
    return out


def _maps(case, seed):
    """(atoms, window) of every map of a case."""
    if case["call"] == "fmap":
        win = _window(case["window"], _grid(case["grid"], case["slots"], case["step"], case["n_t0"], case["n_tau"]))
        return [(_atoms(seed, case["slots"], case["gaps"], case["bins"]), win)]
    out = []
    for i, s in enumerate(_shapes(case)):
        win = _window(s["window"], _grid("linspace", s["slots"], 0, s["n_t0"], s["n_tau"]))
        out.append((_atoms(seed * 131 + i, s["slots"], s["gaps"], s["bins"]), win))
    return out


def _stored(case, seed):
    """Stored maps as a noise search leaves them: 2F of chi-square with four
    degrees of freedom, smooth along tau, a loud cell in the first map."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    shape = (case["maps"], case["n_t0"], case["n_tau"])
    m = torch.rand(shape, generator=g, device="cuda").clamp_(min=1e-7).log_()
    m = -2.0 * (m + torch.rand(shape, generator=g, device="cuda").clamp_(min=1e-7).log_())
    m[0, case["n_t0"] // 3, case["n_tau"] // 2] = 180.0 + seed % 7
    return m.contiguous()


class _State:
    """What the program holds; gives its atoms and plan back when dropped."""
    ctx = batch = None
    ids = ()

    def __del__(self):
        try:
            if self.batch is not None:
                self.batch.close()
            for i in self.ids:
                self.ctx.free(i)
        except Exception:
            pass


def prepare(case, seed):
    s = _State()
    s.ctx, s.case = _ctx(), case
    if case["call"] == "logB":
        s.maps = _stored(case, seed)
        return s
    maps = _maps(case, seed)
    s.ids = [s.ctx.upload(a.ts, a.a2, a.b2, a.ab, a.fa, a.fb, T) for a, _ in maps]
    s.wins = [w for _, w in maps]
    s.bins = [a.bins for a, _ in maps]
    if case["call"] == "fmap":
        s.out = torch.empty((s.bins[0], s.wins[0].t0.size, s.wins[0].tau.size), dtype=torch.float32, device="cuda")
    elif case["call"] == "batch":
        s.batch = s.ctx.batch(list(zip(s.ids, s.wins)), case["prec"])
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def _results(case, per_map):
    """Max 2F and logB of every bin of every map."""
    kind = np.float64 if case["prec"] in ("fp64", "recur64") else np.float32
    flat = [r for res in per_map for r in res]
    return dict(max2F=np.array([r["max2F"] for r in flat], dtype=kind),
                logB=np.array([r["logB"] for r in flat], dtype=np.float32))


def run(s):
    c = s.case
    if c["call"] == "logB":
        return dict(logB=s.ctx.logB(s.maps))
    if c["call"] == "fmap":
        res, twoF = s.ctx.fmap(s.ids[0], s.wins[0], c["prec"], out=s.out)
        return dict(twoF=twoF, **_results(c, [res]))
    if c["call"] == "batch":
        return _results(c, s.batch.run())
    tickets = [s.ctx.submit(i, w, c["prec"]) for i, w in zip(s.ids, s.wins)]
    done = [None] * len(tickets)
    left = list(range(len(tickets)))
    while left:
        for k in list(left):
            done[k] = s.ctx.poll(tickets[k], s.bins[k])
            if done[k] is not None:
                left.remove(k)
    return _results(c, done)


# ---------------------------------------------------------------------------
# Necessary work, and the exact results
# ---------------------------------------------------------------------------
def _map_work(window, slots, bins, n_t0, n_tau):
    """Bytes and operations of one map: the atoms once; per cell and bin the
    quadratic form of four sums, its maximum and one exponential (about 24),
    per cell D and its inverse (about 12); the sums by their recurrences:
    one prefix term per slot and channel for rect (then a difference per
    cell), one term into and one out of the window per slot, tau and channel
    for exp."""
    ch = 4 * bins + 3
    cells = n_t0 * n_tau
    flops = cells * (24 * bins + 12)
    flops += slots * ch + cells * ch if window == "rect" else 4 * n_tau * slots * ch
    return 8 * ch * slots, flops


def _each(case):
    """(window, slots, bins, n_t0, n_tau) of the maps of a case."""
    if case["call"] == "fmap":
        return [(case["window"], case["slots"], case["bins"], case["n_t0"], case["n_tau"])]
    return [(s["window"], s["slots"], s["bins"], s["n_t0"], s["n_tau"]) for s in _shapes(case)]


def work(case):
    if case["call"] == "logB":
        cells = case["maps"] * case["n_t0"] * case["n_tau"]
        return {"bytes": 4.0 * cells + 8.0 * case["maps"], "flops": 16.0 * cells}
    byts = flops = 0.0
    for w in _each(case):
        b, f = _map_work(*w)
        byts, flops = byts + b, flops + f
    if case["call"] == "fmap":
        byts += 4.0 * case["bins"] * case["n_t0"] * case["n_tau"]
    return {"bytes": byts, "flops": flops}


def _cost(case):
    """(bytes, operations, window terms of the plain sums)."""
    w = work(case)
    terms = 0
    if case["call"] != "logB":
        for kind, slots, bins, n_t0, n_tau in _each(case):
            terms += n_t0 * n_tau * bins * (slots // 2 if kind == "exp" else 1)
    return w["bytes"], w["flops"], terms


def _exact_map(a, win):
    """2F [bins, n_t0, n_tau] in 64 bits by direct sums over the SFTs."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    f64 = dict(dtype=torch.float64, device=dev)
    ts = torch.as_tensor(a.ts, **f64)
    t0 = torch.as_tensor(win.t0, **f64)
    ant = torch.as_tensor(np.stack([a.a2, a.b2, a.ab], 1), **f64)
    x = torch.as_tensor(np.concatenate([a.fa, a.fb], 2).transpose(1, 0, 2).reshape(a.ts.size, -1), **f64)
    out = torch.empty((a.bins, t0.numel(), len(win.tau)), **f64)
    dt = ts[None, :] - t0[:, None]
    after = dt >= 0
    for n, tau in enumerate(win.tau.tolist()):
        if win.kind == "rect":
            w = (after & (dt < tau)).to(torch.float64)
        else:
            w = torch.where(after & (dt < 3 * tau), torch.exp(dt * (-1.0 / tau)), 0.0)
        A, B, C = (w * w @ ant).unbind(1)
        f = (w @ x).view(-1, a.bins, 4)
        D = A * B - C * C
        ok = (D > DEGENERATE * A * B)[:, None]
        num = B[:, None] * (f[..., 0] ** 2 + f[..., 1] ** 2) + A[:, None] * (f[..., 2] ** 2 + f[..., 3] ** 2) \
            - 2 * C[:, None] * (f[..., 0] * f[..., 2] + f[..., 1] * f[..., 3])
        out[:, :, n] = torch.where(ok, 2 * num / torch.where(ok, D[:, None], 1.0), 0.0).T
    return out


def _exact_logB(twoF):
    v = twoF.reshape(twoF.shape[0], -1)
    return (torch.logsumexp(0.5 * v, 1) - math.log(v.shape[1])).cpu().numpy()


def exact(case, seed):
    if case["call"] == "logB":
        return dict(logB=_exact_logB(_stored(case, seed).double()))
    # direct sums of every cell: weights per (t0, tau, slot), and products
    weights = sum(n_t0 * n_tau * slots for _, slots, _, n_t0, n_tau in _each(case))
    if weights > 7e10:
        return None
    mx, lb = [], []
    for a, win in _maps(case, seed):
        m = _exact_map(a, win)
        mx.append(m.amax(dim=(1, 2)).cpu().numpy())
        lb.append(_exact_logB(m))
    got = dict(max2F=np.concatenate(mx), logB=np.concatenate(lb))
    if case["call"] == "fmap":
        got["twoF"] = m
    return got
