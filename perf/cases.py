"""Performance cases: the calls that a user of this track finder makes, over the sizes it is used at.

The stages of the chain, each through its public entry point: track finding (the plain search, the
learned proposal, a field map), the Kalman-filter fit, clustering of cells, triplet seeding, ambiguity
resolution, and the network's training step.  Sizes are the ones of this repository's benchmark and
tests: the 100-muon event, mu = 20 ... 200 pileup events, batches of up to 64 events, 4096-row training
batches.  One-event cases are the online use (latency and launches count), batches the offline use.

Inputs: particles and their exact module crossings come from the simulator (``synth``) for a few events;
a batch's further events share those crossings, and hit efficiency, smearing, noise hits, seeds and cell
charges are drawn anew for each event, on the GPU.
"""
import functools
import math
import os
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

import paper_2505_22822_amd as ckf
from synth import barrel10, barrel_endcap, make_event
from synth.cells import NOISE_SIGMA, THRESHOLD, cell_grid, make_cells
from synth.events import MUON_MASS, C_LIGHT, SEED_SIGMA
from synth.field import solenoid_field, solenoid_map

DEV = "cuda"
BZ = 2.0
N_PARAMS = 6752  # the network 7 -> 64 -> 64 -> 32
MODEL_FILE = os.path.join("tests", "golden", "learned_model.txt")  # a trained network kept in the repository


def listed():
    return [
        # the 100-muon event of the parity tests and the smoke run: one small event, all latency
        dict(name="find_tiny", kind="find", det="barrel10", events=1, mu=2.0, form="plain", states=False, graph=False),
        # one dense event at a time, with the states that the fit and the pair capture need
        dict(name="find_event", kind="find", det="barrel_endcap", events=1, mu=200.0, form="plain", states=True,
             graph=False),
        # the benchmark's batch, replayed from a graph as the benchmark does
        dict(name="find_batch", kind="find", det="barrel_endcap", events=64, mu=200.0, form="plain", states=False,
             graph=True),
        # the learned proposal with a trained network
        dict(name="find_learned", kind="find", det="barrel_endcap", events=8, mu=200.0, form="learned", states=False,
             graph=False),
        # the (r, z) field map of the precision study
        dict(name="find_map", kind="find", det="barrel_endcap", events=32, mu=20.0, form="map", states=False,
             graph=False),
        # the fit of one event's tracks, and of a batch's
        dict(name="fit_event", kind="fit", events=1, mu=200.0, smoother="two_filter"),
        dict(name="fit_batch", kind="fit", events=32, mu=200.0, smoother="rts"),
        # cells to measurements, one event and a batch
        dict(name="cluster_event", kind="cluster", events=1, mu=200.0),
        dict(name="cluster_batch", kind="cluster", events=32, mu=200.0),
        # triplet seeds of one dense event
        dict(name="seed_event", kind="seed", events=1, mu=200.0),
        # duplicate removal on a batch of found tracks
        dict(name="resolve_batch", kind="resolve", events=16, mu=200.0),
        # one optimiser step of the network at the training's batch size
        dict(name="train_step", kind="train", rows=4096, pool=200000),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["find", "find", "find", "find", "fit", "fit", "cluster", "cluster", "seed", "resolve", "train"])
    if kind == "train":
        return dict(kind=kind, rows=int(_log(rng, 100, 16384)), pool=rng.randrange(50000, 200000))
    mu = round(_log(rng, 5.0, 200.0), 2)
    most = {"find": 64, "fit": 32, "cluster": 32, "seed": 8, "resolve": 16}[kind]
    events = max(1, int(_log(rng, 1.0, most + 0.99)))
    if kind == "fit":
        return dict(kind=kind, events=events, mu=mu, smoother=rng.choice(["rts", "two_filter"]))
    if kind != "find":
        return dict(kind=kind, events=events, mu=mu)
    form = rng.choice(["plain", "plain", "learned", "map"])
    if form != "plain":
        events = min(events, 32)
    if form == "map":
        mu = min(mu, 20.0)  # (the simulator integrates the truth through the map step by step)
    return dict(kind=kind, det="barrel_endcap", events=events, mu=mu, form=form,
                states=rng.random() < 0.3, graph=rng.random() < 0.3)


# --------------------------------------------------------------------------
# what a program makes once: detector, geometry, field, stream

@functools.lru_cache(None)
def _det(name):
    return barrel10() if name == "barrel10" else barrel_endcap()


@functools.lru_cache(None)
def _geo(name):
    return ckf.Geometry(_det(name).as_arrays())


@functools.lru_cache(None)
def _field(form):
    return ckf.FieldMap(solenoid_map()) if form == "map" else ckf.UniformField(0.0, 0.0, BZ)


@functools.lru_cache(None)
def _stream():
    return torch.cuda.Stream()


@functools.lru_cache(None)
def _table(name):
    """The detector's modules as device tensors (float64)."""
    d = _det(name)
    t = lambda a: torch.as_tensor(np.asarray(a, np.float64), device=DEV)  # noqa: E731
    return dict(center=t(d.center), rot=t(d.rot), half=t(d.half), thick=t(d.thick), sigma=t(d.sigma()))


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) % (1 << 60))
    return g


# --------------------------------------------------------------------------
# inputs

def _truths(case, seed):
    """A few simulated events: one for each event of a small batch, at most three."""
    det = _det(case.get("det", "barrel_endcap"))
    k = 1 if case.get("form") == "map" else min(case["events"], 3)
    kw = dict(kind="tiny") if det.name == "barrel10" else dict(mu=case["mu"])
    if case.get("form") == "map":
        kw["field"] = solenoid_field
    with ThreadPoolExecutor(3) as ex:
        return list(ex.map(lambda i: make_event(det, 16 * int(seed) + i, **kw), range(k)))


def _sample(case, seed, truths):
    """The batch's measurements and seeds, drawn from the simulated crossings: a dict with the fields of
    ckf.Batch and, for every kept hit in track order, its measurement and its track."""
    name = case.get("det", "barrel_endcap")
    det, tab, g = _det(name), _table(name), _gen(seed)
    S, E = det.n_surfaces, case["events"]
    surf, loc, part, ev_of, seeds = [], [], [], [], []
    n_part = 0
    for e in range(E):
        ev = truths[e % len(truths)]
        tr = ev.truth
        t = lambda a, dt=torch.float64: torch.as_tensor(np.ascontiguousarray(a), device=DEV).to(dt)  # noqa: E731
        keep = torch.rand(len(tr.surface), generator=g, device=DEV) < 0.99
        surf.append(t(tr.surface, torch.int64)[keep] + e * S)
        loc.append(t(tr.loc)[keep])
        ev_of.append(e)
        # tracks are numbered by seed: one seed for every particle that crosses a module
        rank = np.full(len(ev.particle_pt), -1, np.int64)
        rank[ev.seed_particle] = np.arange(ev.n_seeds)
        part.append(t(rank[tr.particle], torch.int64)[keep] + n_part)
        n_part += ev.n_seeds
        truth5 = t(ev.seed_truth)
        sig = torch.tensor(SEED_SIGMA, dtype=torch.float64, device=DEV).expand(ev.n_seeds, 5).clone()
        sig[:, 4] *= truth5[:, 4].abs()
        par = truth5 + sig * torch.randn(truth5.shape, generator=g, device=DEV, dtype=torch.float64)
        cov = torch.zeros((ev.n_seeds, 15), dtype=torch.float64, device=DEV)
        cov[:, [0, 5, 9, 12, 14]] = sig ** 2
        seeds.append((torch.full((ev.n_seeds,), e, dtype=torch.int32, device=DEV), t(ev.seed_surface, torch.int32),
                      par, cov))
    surf, loc, part = torch.cat(surf), torch.cat(loc), torch.cat(part)
    n_hit = surf.numel()
    loc = loc + tab["sigma"][surf % S] * torch.randn(loc.shape, generator=g, device=DEV, dtype=torch.float64)
    # one noise hit on 1 % of the modules
    ns = torch.nonzero(torch.rand(E * S, generator=g, device=DEV) < 0.01).flatten()
    nl = (2 * torch.rand((ns.numel(), 2), generator=g, device=DEV, dtype=torch.float64) - 1) * tab["half"][ns % S]
    row, loc = torch.cat([surf, ns]), torch.cat([loc, nl])
    order = torch.argsort(row, stable=True)
    row, loc = row[order], loc[order]
    ids = torch.empty_like(order)
    ids[order] = torch.arange(order.numel(), device=DEV)
    off = torch.zeros(E * S + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(torch.bincount(row, minlength=E * S), 0)
    batch = ckf.Batch(E, S, off.to(torch.int32), loc.to(torch.float32).contiguous(),
                      (tab["sigma"][row % S] ** 2).to(torch.float32).contiguous(),
                      *(torch.cat([s[k] for s in seeds]).contiguous() for k in range(4)))
    return dict(batch=batch, hit_meas=ids[:n_hit], hit_track=part, hit_surface=surf % S)


def _fill(t, n, value):
    """t in a buffer of n rows; the rows beyond hold `value`."""
    if t.numel() > n:
        raise ValueError("capacity")
    return torch.cat([t, torch.full((n - t.numel(),), int(value), dtype=t.dtype, device=DEV)])


def _tracks(s, lo=6, hi=48):
    """Tracks in ckf_find's layout from the hits of the particles with lo ... hi of them (the first hi), in
    buffers with room for every seed's track."""
    n = s["batch"].n_seeds
    cnt = torch.bincount(s["hit_track"], minlength=n)
    start = torch.cumsum(cnt, 0) - cnt
    pos = torch.arange(s["hit_track"].numel(), device=DEV) - start[s["hit_track"]]
    good = cnt >= lo
    use = good[s["hit_track"]] & (pos < hi)
    seed = torch.nonzero(good).flatten()
    off = torch.zeros(seed.numel() + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(cnt[seed].clamp(max=hi), 0)
    return dict(n_tracks=torch.tensor([seed.numel()], dtype=torch.int32, device=DEV),
                offsets=_fill(off.to(torch.int32), n + 1, off[-1]),
                meas=_fill(s["hit_meas"][use].to(torch.int32), 12 * n, 0),
                meas_surface=_fill(s["hit_surface"][use].to(torch.int32), 12 * n, 0),
                seed=_fill(seed.to(torch.int32), n, 0))


def _with_duplicates(tr, seed):
    """A third of the tracks found a second time, from a seed one or two layers further out: the copy lacks
    the first hits.  (Triplet seeding makes several seeds per particle, so such copies are the common case.)"""
    g = _gen(seed + 7)
    n = int(tr["n_tracks"])
    off = tr["offsets"][: n + 1].to(torch.int64)
    cnt = off[1:] - off[:-1]
    dup = torch.nonzero(torch.rand(n, generator=g, device=DEV) < 0.33).flatten()
    skip = 1 + (torch.rand(dup.numel(), generator=g, device=DEV) < 0.5).to(torch.int64)
    src = torch.cat([torch.arange(n, device=DEV), dup])
    drop = torch.cat([torch.zeros(n, dtype=torch.int64, device=DEV), skip])
    o = torch.argsort(src, stable=True)
    src, drop = src[o], drop[o]
    new = cnt[src] - drop
    noff = torch.zeros(src.numel() + 1, dtype=torch.int64, device=DEV)
    noff[1:] = torch.cumsum(new, 0)
    at = torch.repeat_interleave(off[src] + drop - noff[:-1], new) + torch.arange(int(noff[-1]), device=DEV)
    chi2 = torch.rand((src.numel(), 1), generator=g, device=DEV, dtype=torch.float64).add(0.5).flatten() * 2 * new
    cap = 3 * (tr["offsets"].numel() - 1) // 2
    return dict(n_tracks=torch.tensor([src.numel()], dtype=torch.int32, device=DEV),
                offsets=_fill(noff.to(torch.int32), cap + 1, noff[-1]), meas=_fill(tr["meas"][at], 12 * cap, 0),
                chi2=_fill(chi2, cap, 0), ndf=_fill((2 * new - 5).to(torch.int32), cap, 0))


def _n_cells(case):
    return int(720 * case["mu"] + 1500)


def _cells(case, seed):
    """The batch's activated cells: simulated charges with new electronic noise for every event, and a few
    per cent of the cells dead, so that every event has the same number of them."""
    det, g = _det("barrel_endcap"), _gen(seed)
    truths = _truths(case, seed)
    base = [make_cells(det, ev, 16 * int(seed) + i) for i, ev in enumerate(truths)]
    S, E = det.n_surfaces, case["events"]
    row, c0, c1, q = [], [], [], []
    for e in range(E):
        b = base[e % len(base)]
        r = np.repeat(np.arange(S), np.diff(b.offsets))
        qq = torch.as_tensor(b.q, device=DEV)
        qq = qq + NOISE_SIGMA * torch.randn(qq.shape, generator=g, device=DEV)
        keep = torch.nonzero(qq > THRESHOLD).flatten()
        keep = keep[torch.randperm(keep.numel(), generator=g, device=DEV)[: _n_cells(case)]].sort().values
        row.append(torch.as_tensor(r, device=DEV)[keep] + e * S)
        c0.append(torch.as_tensor(b.c0, device=DEV)[keep])
        c1.append(torch.as_tensor(b.c1, device=DEV)[keep])
        q.append(qq[keep])
    row = torch.cat(row)
    off = torch.zeros(E * S + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(torch.bincount(row, minlength=E * S), 0)
    return ckf.CellBatch(E, S, off.to(torch.int32), torch.cat(c0).contiguous(), torch.cat(c1).contiguous(),
                         torch.cat(q).contiguous()), row


def _pairs(case, seed):
    """Training pairs with the inputs' ranges (fractional position, direction, q/p, layer) and labels spread
    around the window's middle cells as the crossings' neighbours are; FP32 parameters and Adam moments."""
    g = _gen(seed)
    n = case["pool"]
    u = lambda *s: torch.rand(s, generator=g, device=DEV)  # noqa: E731
    x = torch.empty((n, 7), device=DEV)
    x[:, :2] = u(n, 2) - 0.5
    d = torch.randn((n, 3), generator=g, device=DEV) * torch.tensor([0.2, 0.6, 1.0], device=DEV)
    d[:, 2] = d[:, 2].abs() + 0.2
    x[:, 2:5] = d / d.norm(dim=1, keepdim=True)
    x[:, 5] = 2 * u(n) - 1
    x[:, 6] = torch.floor(u(n) * 22) / 22
    iu = torch.floor(x[:, 0] + 8 * x[:, 2] + 0.4 * torch.randn(n, generator=g, device=DEV) + 4.5).clamp(0, 7)
    iv = torch.floor(x[:, 1] + x[:, 3] + 0.2 * torch.randn(n, generator=g, device=DEV) + 2.5).clamp(0, 3)
    lab = (8 * iv + iu).to(torch.int32)
    rows = torch.randperm(n, generator=g, device=DEV)[: case["rows"]].to(torch.int32)
    par = torch.cat([(2 * u(a * b) - 1) * math.sqrt(6.0 / b) if b else torch.zeros(a, device=DEV)
                     for a, b in ((64, 7), (64, 0), (64, 64), (64, 0), (32, 64), (32, 0))]).contiguous()
    mom = 1e-3 * torch.randn(N_PARAMS, generator=g, device=DEV)
    return dict(x=x.contiguous(), labels=lab, rows=rows.contiguous(), params=par, m=mom, v=mom.square() + 1e-8)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        s = _pairs(case, seed)
        return dict(kind=kind, ws=ckf.MlpWorkspace(case["rows"], DEV), grad=torch.empty(N_PARAMS, device=DEV),
                    loss=torch.empty(1, device=DEV), step=0, **s)
    if kind == "cluster":
        cells, _ = _cells(case, seed)
        pitch = torch.as_tensor(cell_grid(_det("barrel_endcap"))[1], device=DEV).contiguous()
        return dict(kind=kind, clusterer=ckf.Clusterer(_geo("barrel_endcap"), cells, pitch), pitch=pitch)
    s = _sample(case, seed, _truths(case, seed))
    b = s["batch"]
    name = case.get("det", "barrel_endcap")
    if kind == "find":
        model = None
        if case["form"] == "learned":
            par = torch.as_tensor(np.loadtxt(MODEL_FILE, dtype=np.float32), device=DEV).contiguous()
            model = ckf.Model(par)
            torch.cuda.synchronize()
        f = ckf.Finder(_geo(name), _field(case["form"]), b, counters=False, model=model, meas_states=case["states"])
        if case["graph"]:
            f.capture(_stream())
        return dict(kind=kind, finder=f, graph=case["graph"], model=model)
    if kind == "fit":
        tr = _tracks(s)
        return dict(kind=kind, fitter=ckf.Fitter(_geo(name), _field("plain"), b, tr, smoother=case["smoother"]))
    if kind == "seed":
        tab = _table(name)
        row = torch.repeat_interleave(torch.arange(b.n_events * b.n_surfaces, device=DEV), torch.diff(b.offsets))
        m = row % b.n_surfaces
        l64 = b.loc.to(torch.float64)
        sp = tab["center"][m] + l64[:, :1] * tab["rot"][m, 0] + l64[:, 1:] * tab["rot"][m, 1]
        # room for a little fewer seeds than such events have: the finder downstream takes at most that many
        cap = int(b.n_events * 50 * case["mu"] * (2.6 + 0.0042 * case["mu"]))
        return dict(kind=kind, batch=b, sp=sp.to(torch.float32).contiguous(), geo=_geo(name), cap=cap)
    return dict(kind=kind, tracks=_with_duplicates(_tracks(s), seed), n_meas=b.n_meas)  # resolve


# --------------------------------------------------------------------------
# one pass

def run(state):
    kind = state["kind"]
    if kind == "find":
        f = state["finder"]
        if state["graph"]:
            f.launch_graph(_stream())
        else:
            f.enqueue()
        return {k: v for k, v in f.out.items() if v is not None}
    if kind == "fit":
        f = state["fitter"]
        f.enqueue()
        return dict(params=f.params, cov=f.cov, chi2=f.chi2, ok=f.ok)
    if kind == "cluster":
        c = state["clusterer"]
        c.enqueue()
        return dict(offsets=c.offsets, loc=c.loc, var=c.var, spacepoints=c.spacepoints, cell_cluster=c.cell_cluster,
                    status=c.status)
    if kind == "seed":
        b = state["batch"]
        out, n = ckf.seed(state["geo"], b.n_events, b.offsets, state["sp"], b.loc, [0, 1, 2, 3], bz=BZ,
                          cap_seeds=state["cap"])
        return dict(n=n, **out)
    if kind == "resolve":
        keep, info = ckf.resolve(state["tracks"], state["n_meas"], sync=False)
        return dict(keep=keep, info=info)
    state["step"] += 1
    ckf.mlp_grad(state["params"], state["x"], state["labels"], rows=state["rows"], workspace=state["ws"],
                 grad=state["grad"], loss=state["loss"])
    ckf.mlp_adam(state["params"], state["m"], state["v"], state["grad"], state["step"])
    return {k: state[k] for k in ("grad", "loss", "params", "m", "v")}


# --------------------------------------------------------------------------
# the work of one pass

def work(case):
    """Inputs read once and outputs written once; operations counted from the method's steps (the units
    of the search and the seeding that the benchmark reports for its mu = 200 batch, per seed)."""
    if case["kind"] == "train":
        r = case["rows"]
        return dict(bytes=32.0 * r + 4.0 * N_PARAMS * 10, flops=r * 6.0 * (7 * 64 + 64 * 64 + 64 * 32))
    E, mu = case["events"], case["mu"]
    S = _det(case.get("det", "barrel_endcap")).n_surfaces
    seeds, meas = E * 50.0 * mu, E * (398.0 * mu + 0.01 * S)
    per = 8.0  # measurements of a track
    if case["kind"] == "find":
        flops = {"plain": 45e3, "learned": 240e3, "map": 50e3}[case["form"]]
        out = 230 + per * (4 + (44 if case["states"] else 0))
        return dict(bytes=4.0 * E * S + 16 * meas + seeds * (168 + 0.88 * out), flops=seeds * flops)
    if case["kind"] == "fit":
        k = 0.88 * seeds * per  # per measurement: its inputs, the smoothed state; leg, transport, update, smoother
        return dict(bytes=k * (24 + 160) + 0.88 * seeds * 180, flops=k * (3000 if case["smoother"] == "rts" else 4500))
    if case["kind"] == "cluster":
        cells = float(E * _n_cells(case))
        return dict(bytes=8.0 * E * S + 16 * cells + 0.54 * cells * 28, flops=cells * 12.0)
    if case["kind"] == "seed":
        return dict(bytes=4.0 * E * S + 20 * meas + E * 36000.0 * (mu / 200) * 188,
                    flops=E * 0.78e9 * (mu / 200) ** 2.5)
    tracks = 0.88 * seeds * 1.33
    return dict(bytes=tracks * (4 * per + 4 + 12 + 4) + 4 * meas, flops=tracks * per * 4)


# --------------------------------------------------------------------------
# the results in 64 bits

def exact(case, seed):
    """Fit, clustering and training in float64.  None for the search (a branching search with thousands of
    seeds: minutes in plain numpy), for the seeding (its definition is the float64 arithmetic itself, with
    every cut's decision part of it) and for the resolution (whole numbers only)."""
    if case["kind"] == "fit":
        return _exact_fit(case, seed)
    if case["kind"] == "cluster":
        return _exact_cluster(case, seed)
    if case["kind"] == "train":
        return _exact_train(case, seed)
    return None


_PK = [[min(i, j) * 5 - min(i, j) * (min(i, j) - 1) // 2 + abs(i - j) for j in range(5)] for i in range(5)]
_UP = [(i, j) for i in range(5) for j in range(i, 5)]


def _leg(p, A, B):
    """Bound parameters on modules A -> on modules B along the helix in the axial field (closed form; the
    path from Newton's method)."""
    sp, cp, st, ct = torch.sin(p[:, 2]), torch.cos(p[:, 2]), torch.sin(p[:, 3]), torch.cos(p[:, 3])
    r = A["center"] + p[:, :1] * A["rot"][:, 0] + p[:, 1:2] * A["rot"][:, 1]
    om = -C_LIGHT * p[:, 4] * BZ
    n = B["rot"][:, 2]
    T = torch.stack([cp * st, sp * st, ct], 1)

    def at(s):
        a = om * s
        S, Cc = torch.sin(a) / om, (1 - torch.cos(a)) / om
        x = r[:, 0] + T[:, 0] * S - T[:, 1] * Cc
        y = r[:, 1] + T[:, 1] * S + T[:, 0] * Cc
        d = torch.stack([T[:, 0] * torch.cos(a) - T[:, 1] * torch.sin(a),
                         T[:, 1] * torch.cos(a) + T[:, 0] * torch.sin(a), ct], 1)
        return torch.stack([x, y, r[:, 2] + ct * s], 1), d

    s = ((B["center"] - r) * n).sum(1) / (T * n).sum(1)
    for _ in range(10):
        x, d = at(s)
        s = s - ((x - B["center"]) * n).sum(1) / (d * n).sum(1)
    x, d = at(s)
    q = x - B["center"]
    return torch.stack([(q * B["rot"][:, 0]).sum(1), (q * B["rot"][:, 1]).sum(1), torch.atan2(d[:, 1], d[:, 0]),
                        torch.atan2(torch.hypot(d[:, 0], d[:, 1]), d[:, 2]), p[:, 4]], 1)


def _scattering(p, C, M):
    """C with the Highland width of modules M added to the angles' variances."""
    st = torch.sin(p[:, 3])
    cosa = (M["rot"][:, 2, 0] * torch.cos(p[:, 2]) * st + M["rot"][:, 2, 1] * torch.sin(p[:, 2]) * st
            + M["rot"][:, 2, 2] * torch.cos(p[:, 3])).abs()
    x = M["thick"] / cosa
    mom = 1 / p[:, 4].abs()
    beta = mom / torch.sqrt(mom * mom + MUON_MASS ** 2)
    th = torch.where(M["thick"] > 0, 0.0136 / (beta * mom) * torch.sqrt(x) * (1 + 0.038 * torch.log(x / beta ** 2)),
                     torch.zeros_like(x))
    C = C.clone()
    C[:, 2, 2] += (th / st) ** 2
    C[:, 3, 3] += th ** 2
    return C


def _wrap(d):
    d = d.clone()
    d[:, 2] = torch.remainder(d[:, 2] + math.pi, 2 * math.pi) - math.pi
    return d


def _exact_fit(case, seed):
    """The forward Kalman filter and the Rauch-Tung-Striebel smoother (the two-filter smoother on the same
    linearised model is the same estimate)."""
    s = _sample(case, seed, _truths(case, seed))
    tr, b, tab = _tracks(s), s["batch"], _table("barrel_endcap")
    off, meas, msurf = (tr[k].to(torch.int64) for k in ("offsets", "meas", "meas_surface"))
    sid = tr["seed"].to(torch.int64)
    n = int(tr["n_tracks"])
    sid, off = sid[:n], off[: n + 1]
    cnt = off[1:] - off[:-1]
    mod = lambda i: {k: tab[k][i] for k in ("center", "rot", "thick")}  # noqa: E731
    full = torch.tensor(_PK, device=DEV)
    up = torch.tensor([5 * i + j for i, j in _UP], device=DEV)
    p, C = b.seed_params[sid].clone(), b.seed_cov[sid][:, full].clone()
    cur = b.seed_surface[sid].to(torch.int64)
    chi2 = torch.zeros(n, dtype=torch.float64, device=DEV)
    eye = torch.eye(5, dtype=torch.float64, device=DEV)
    steps = []
    for k in range(int(cnt.max())):
        t = torch.nonzero(cnt > k).flatten()
        at = off[t] + k
        dst = msurf[at]
        F = eye.expand(t.numel(), 5, 5).clone()
        pp, Cp = p[t], C[t]
        go = torch.nonzero(dst != cur[t]).flatten()
        if go.numel():
            A, B, p0 = mod(cur[t][go]), mod(dst[go]), pp[go]
            cols = []
            for j in range(5):
                new, col = torch.func.jvp(lambda z: _leg(z, A, B), (p0,), (eye[j].expand_as(p0).contiguous(),))
                cols.append(col)
            F[go] = torch.stack(cols, 2)
            pp[go] = new
            Cp[go] = F[go] @ Cp[go] @ F[go].transpose(1, 2).contiguous()
        z, V = b.loc[meas[at]].to(torch.float64), torch.diag_embed(b.var[meas[at]].to(torch.float64))
        res = (z - pp[:, :2])[:, :, None]
        Si = torch.linalg.inv(Cp[:, :2, :2] + V)
        chi2[t] += (res.transpose(1, 2) @ Si @ res)[:, 0, 0]
        K = Cp[:, :, :2].contiguous() @ Si
        pf = _wrap(pp + (K @ res)[:, :, 0])
        IK = eye - torch.cat([K, K.new_zeros(K.shape[0], 5, 3)], 2)
        Cf = IK @ Cp @ IK.transpose(1, 2).contiguous() + K @ V @ K.transpose(1, 2).contiguous()
        steps.append((t, at, F, pp, Cp, pf, Cf))
        p[t], C[t] = pf, _scattering(pf, Cf, mod(dst))
        cur[t] = dst
    out_p = torch.zeros((meas.numel(), 5), dtype=torch.float64, device=DEV)
    out_C = torch.zeros((meas.numel(), 15), dtype=torch.float64, device=DEV)
    xs, Cs = torch.zeros_like(p), torch.zeros_like(C)
    for k in reversed(range(len(steps))):
        t, at, _, _, _, pf, Cf = steps[k]
        xn, Cn = pf.clone(), Cf.clone()
        if k + 1 < len(steps):
            t1, _, F1, pp1, Cp1, _, _ = steps[k + 1]
            i = torch.searchsorted(t, t1)
            A = torch.linalg.solve(Cp1, F1 @ Cf[i]).transpose(1, 2).contiguous()
            xn[i] = _wrap(pf[i] + (A @ _wrap(xs[t1] - pp1)[:, :, None])[:, :, 0])
            Cn[i] = Cf[i] + A @ (Cs[t1] - Cp1) @ A.transpose(1, 2).contiguous()
        xs[t], Cs[t] = xn, Cn
        out_p[at], out_C[at] = xn, Cn.reshape(-1, 25)[:, up]
    return dict(params=out_p, cov=out_C, chi2=torch.cat([chi2, chi2.new_zeros(b.n_seeds - n)]), ok=None)


def _exact_cluster(case, seed):
    cells, row = _cells(case, seed)
    tab, n = _table("barrel_endcap"), cells.n_cells
    S = cells.n_surfaces
    c0, c1 = cells.c0.to(torch.int64), cells.c1.to(torch.int64)
    key = (row * 1024 + c1) * 1024 + c0
    me = torch.arange(n, device=DEV)
    pairs = []
    for d0, d1 in ((-1, 0), (-1, -1), (0, -1), (1, -1)):
        ok = (c0 + d0 >= 0) & (c1 + d1 >= 0)
        at = torch.searchsorted(key, key + d1 * 1024 + d0).clamp(max=n - 1)
        ok &= key[at] == key + d1 * 1024 + d0
        pairs.append((me[ok], at[ok]))
    a, b = torch.cat([x for x, _ in pairs]), torch.cat([x for _, x in pairs])
    lab = me.clone()
    while True:
        new = lab.scatter_reduce(0, a, lab[b], "amin").scatter_reduce(0, b, lab[a], "amin")
        new = torch.minimum(new, new[new])
        if torch.equal(new, lab):
            break
        lab = new
    first, inv = torch.unique(lab, return_inverse=True)
    m = first.numel()
    q = cells.q.to(torch.float64)
    total = lambda w: torch.zeros(m, dtype=torch.float64, device=DEV).index_add_(0, inv, w)  # noqa: E731
    W = total(q)
    s = row[first] % S
    pitch = torch.as_tensor(cell_grid(_det("barrel_endcap"))[1].astype(np.float64), device=DEV)[s]
    x = torch.stack([total(q * (c0 + 0.5)) / W, total(q * (c1 + 0.5)) / W], 1)
    loc = torch.zeros((n, 2), dtype=torch.float64, device=DEV)
    var, sp = torch.zeros_like(loc), torch.zeros((n, 3), dtype=torch.float64, device=DEV)
    loc[:m] = pitch * x - tab["half"][s]
    var[:m] = pitch ** 2 / 12
    sp[:m] = tab["center"][s] + loc[:m, :1] * tab["rot"][s, 0] + loc[:m, 1:] * tab["rot"][s, 1]
    return dict(offsets=None, loc=loc, var=var, spacepoints=sp, cell_cluster=None, status=None)


def _exact_train(case, seed):
    s = _pairs(case, seed)
    P = s["params"].to(torch.float64).requires_grad_(True)
    i = s["rows"].to(torch.int64)
    x, lab = s["x"][i].to(torch.float64), s["labels"][i].to(torch.int64)
    W1, b1, W2, b2, W3, b3 = torch.split(P, [448, 64, 4096, 64, 2048, 32])
    h = torch.relu(x @ W1.view(64, 7).T + b1)
    h = torch.relu(h @ W2.view(64, 64).T + b2)
    loss = torch.nn.functional.cross_entropy(h @ W3.view(32, 64).T + b3, lab)
    (g,) = torch.autograd.grad(loss, P)
    m = 0.9 * s["m"].to(torch.float64) + 0.1 * g
    v = 0.999 * s["v"].to(torch.float64) + 0.001 * g * g
    new = P.detach() - 1e-3 * (m / 0.1) / (torch.sqrt(v / 0.001) + 1e-8)
    return dict(grad=g, loss=loss.detach().reshape(1), params=new, m=m, v=v)
