"""The work that programs have this library do, as cases that can be timed and checked.

A pass is a stretch of a molecular-dynamics run as a program sees it: some
steps pushed into a correlator that is already running, then a readout of its
groups (the correlation functions and their running Green-Kubo integrals).
The correlator of a sample-fed case has taken ``fill`` steps before the first
pass, so that a pass meets the steady state of a long run and not its first
steps.

The frames are synthetic: Ornstein-Uhlenbeck series for velocities, stress and
heat flux, uniform positions with a small thermal displacement for atoms.  A
state holds ``rows`` frames in device memory and its steps go through them
again and again, as a program goes through its own few buffers.

Readouts are returned in the precision that the group's sums are kept in:
double for FP64 sums, single for compensated FP32 sums.

Families (``kind``):
  samples   per-atom or global series handed in by the caller
  cross     pairs of series (x, y) handed in by the caller
  rhok      n(k) of atom positions, evaluated and correlated on every step
  currents  longitudinal and transverse currents of positions and velocities
  kgap      currents and n(k) in one long window each
  massflux  partial momentum densities against the heat flux, and the heat flux
  batched   per-atom series, n(k) and global series in one context
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2503_07526_amd import Correlator, GroupDesc

DEV = "cuda:0"
BOX = 100.0
LIF = (6.941, 18.998)  # the masses of the two species of molten LiF
_T = {"f32": torch.float32, "f64": torch.float64}


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # The smallest program: six stress and three heat-flux components in
        # double, one call a step, viscosity read out.  Latency and launches.
        dict(name="stress_heat_9", kind="samples", n=9, dtype="f64", accum="f64", levels=20,
             points=16, steps=128, rows=64, fill=300, mode="push", every=1, gk=1, per=9),
        # A small cell: 83349 atoms (an odd count), compensated sums, correlated
        # every 10th MD step, a few atoms looked at by themselves.
        dict(name="vaf_83349_atoms", kind="samples", n=250047, dtype="f32", accum="kahan",
             levels=10, points=16, steps=512, rows=100, fill=300, mode="push", every=10, gk=0, per=33),
        # The velocity autocorrelation of 10^6 atoms with double sums.
        dict(name="vaf_1e6_atoms", kind="samples", n=3000000, dtype="f32", accum="f64",
             levels=12, points=16, steps=256, rows=32, fill=300, mode="push", every=1, gk=0, per=0),
        # The largest: 4 x 10^6 atoms with compensated sums.
        dict(name="vaf_4e6_atoms", kind="samples", n=12000000, dtype="f32", accum="kahan",
             levels=12, points=16, steps=256, rows=24, fill=300, mode="push", every=1, gk=0, per=0),
        # A stored history read back: 3 x 10^5 atoms, 700 frames in one call,
        # whole blocks and a remainder.
        dict(name="replay_700_frames", kind="samples", n=900000, dtype="f32", accum="kahan",
             levels=12, points=16, steps=700, rows=700, fill=0, mode="replay", every=1, gk=0, per=0),
        # Cross-correlations of 33333 atoms' vectors with 32 points a level:
        # updated on every step.
        dict(name="cross_99999", kind="cross", n=99999, dtype="f32", accum="kahan", levels=10,
             points=32, steps=64, rows=32, fill=64, mode="push", every=1, gk=0, per=7),
        # The intermediate scattering function of 10^6 atoms at 2048 k-vectors.
        dict(name="rhok_2048_1e6", kind="rhok", nk=2048, atoms=1000000, levels=16, points=32,
             steps=16, rows=4),
        # The same for a small cell, its smallest k-vectors only.
        dict(name="rhok_300_20011", kind="rhok", nk=300, atoms=20011, levels=10, points=32,
             steps=64, rows=16),
        # Longitudinal and transverse currents of 10^6 atoms at 2048 k-vectors.
        dict(name="currents_2048_1e6", kind="currents", nk=2048, atoms=1000000, levels=16,
             points=32, steps=12, rows=4),
        # A k-gap run: both producers, one long window each, every 10th step.
        dict(name="kgap_512_200000", kind="kgap", nk=512, atoms=200000, points=4096, steps=64,
             rows=8),
        # The mass-flux correction of the thermal conductivity, 5 x 10^6 atoms.
        dict(name="massflux_5e6", kind="massflux", atoms=5000000, levels=12, points=16, steps=32,
             rows=4),
        # Everything at once, stretches of 16 steps replayed as one HIP graph
        # (four of them between readouts) with the launch shape that the
        # autotuner keeps for this mix.
        dict(name="batched_6e6_2048", kind="batched", n=6000000, nk=2048, atoms=1000000,
             steps=64, rows=16, fill=260),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["samples", "samples", "replay", "cross", "rhok", "rhok", "currents", "kgap",
                       "massflux", "batched"])
    if kind == "samples":
        dtype, accum = rng.choice([("f32", "kahan"), ("f32", "kahan"), ("f32", "f64"), ("f64", "f64")])
        n = _logint(rng, 6, 3000 if dtype == "f64" else 8000000)
        return dict(kind="samples", n=n, dtype=dtype, accum=accum, levels=rng.randint(8, 20),
                    points=16, steps=rng.randint(100, 400), rows=rng.randint(8, 24),
                    fill=rng.randint(256, 400), mode="push", every=rng.choice([1, 10]), gk=rng.randint(0, 2),
                    per=min(n, rng.randint(0, 40)))
    if kind == "replay":
        steps = rng.randint(200, 800)
        return dict(kind="samples", n=_logint(rng, 3000, 900000), dtype="f32", accum="kahan",
                    levels=rng.randint(8, 12), points=16, steps=steps, rows=steps,
                    fill=rng.choice([0, 256, 100]), mode="replay", every=1, gk=0, per=0)
    if kind == "cross":
        return dict(kind="cross", n=_logint(rng, 9, 150000), dtype="f32", accum="kahan",
                    levels=rng.randint(6, 12), points=rng.choice([16, 24, 32]),
                    steps=rng.randint(32, 80), rows=rng.randint(8, 32), fill=64, mode="push", every=1, gk=0, per=5)
    if kind in ("rhok", "currents"):
        atoms = _logint(rng, 2000, 1000000)
        return dict(kind=kind, nk=_logint(rng, 40, 2048), atoms=atoms, levels=rng.randint(8, 16),
                    points=rng.choice([16, 32]), steps=8 if atoms > 200000 else rng.randint(16, 48),
                    rows=4)
    if kind == "kgap":
        return dict(kind="kgap", nk=_logint(rng, 64, 512), atoms=_logint(rng, 5000, 200000),
                    points=rng.randint(1000, 4096), steps=rng.randint(32, 80), rows=4)
    if kind == "massflux":
        return dict(kind="massflux", atoms=_logint(rng, 20000, 5000000), levels=rng.randint(8, 12),
                    points=16, steps=rng.randint(16, 48), rows=4)
    rows = rng.randint(8, 24)
    return dict(kind="batched", n=_logint(rng, 100000, 5000000), nk=_logint(rng, 200, 2048),
                atoms=_logint(rng, 20000, 800000), steps=2 * rows, rows=rows,
                fill=rng.randint(256, 300))


# ------------------------------------------------------------------ the inputs
def _kvectors(nk):
    """The first nk lattice vectors of the half space, by length."""
    n = 12
    g = np.arange(-n, n + 1)
    v = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    x, y, z = v.T
    half = (x > 0) | ((x == 0) & (y > 0)) | ((x == 0) & (y == 0) & (z > 0))
    r2 = (v * v).sum(1)
    v, r2 = v[half & (r2 <= n * n)], r2[half & (r2 <= n * n)]
    order = np.lexsort((v[:, 2], v[:, 1], v[:, 0], r2))
    return np.ascontiguousarray(v[order][:nk], dtype=np.int32)


def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + stream) % (1 << 62))
    return g


def _ou(seed, stream, rows, n, dtype="f32", lo=20.0, hi=200.0, sigma=1.0):
    """[rows][n] consecutive values of n stationary series, each with its own time."""
    g, t = _gen(seed, stream), _T[dtype]
    tau = lo + (hi - lo) * torch.rand(n, generator=g, device=DEV, dtype=t)
    a = torch.exp(-1.0 / tau)
    b = sigma * torch.sqrt(1.0 - a * a)
    out = torch.empty(rows, n, device=DEV, dtype=t)
    x = sigma * torch.randn(n, generator=g, device=DEV, dtype=t)
    for r in range(rows):
        out[r] = x
        x = a * x + b * torch.randn(n, generator=g, device=DEV, dtype=t)
    return out


def _positions(seed, stream, rows, atoms):
    """[rows][3][atoms]: atoms of a cubic box moving about their sites."""
    r0 = BOX * torch.rand(3 * atoms, generator=_gen(seed, stream), device=DEV)
    d = _ou(seed, stream + 1, rows, 3 * atoms, lo=50.0, hi=50.0, sigma=0.1)
    return (r0 + d).reshape(rows, 3, atoms)


def _species(seed, atoms):
    return np.random.default_rng(int(seed) + 77).integers(0, 2, atoms).astype(np.int32)


def _groups(case, seed):
    """The groups of a case, without their inputs."""
    kind = case["kind"]
    if kind in ("samples", "cross"):
        return [GroupDesc(case["n"], case["levels"], case["points"], 2, dtype=case["dtype"],
                          accum=case["accum"], update_every=case["every"], dt=0.001,
                          pair=kind == "cross")]
    if kind == "massflux":
        return [GroupDesc(6, case["levels"], case["points"], 2, dtype="f32", accum="kahan",
                          source="momentum", n_atoms=case["atoms"], box=BOX,
                          species=_species(seed, case["atoms"]), masses=np.array(LIF), pair=True, dt=0.001),
                GroupDesc(3, case["levels"], case["points"], 2, dtype="f32", accum="kahan", dt=0.001)]
    kv = _kvectors(case["nk"])
    if kind == "batched":
        return [GroupDesc(case["n"], 10, 16, 2, dtype="f32", accum="kahan", dt=0.001),
                GroupDesc(len(kv), 16, 32, 2, dtype="cf32", accum="kahan", source="rhok", kvec=kv,
                          n_atoms=case["atoms"], box=BOX, dt=0.001),
                GroupDesc(9, 20, 16, 2, dtype="f64", accum="f64", dt=0.001)]
    lv, u = (1, 10) if kind == "kgap" else (case["levels"], 1)
    one = [GroupDesc((3 if s == "currents" else 1) * len(kv), lv, case["points"], 2, dtype="cf32",
                     accum="kahan", source=s, kvec=kv, n_atoms=case["atoms"], box=BOX,
                     update_every=u, dt=0.001)
           for s in (("currents", "rhok") if kind == "kgap" else (kind,))]
    return one


def _inputs(case, seed):
    """The frames of every group: one tensor each, steps along the first axis."""
    kind, rows = case["kind"], case["rows"]
    if kind == "samples":
        return [_ou(seed, 1, rows, case["n"], case["dtype"])]
    if kind == "cross":
        x = _ou(seed, 1, rows, case["n"], case["dtype"])
        y = 0.6 * x + 0.8 * _ou(seed, 2, rows, case["n"], case["dtype"])
        return [torch.cat([x, y], 1)]
    if kind == "massflux":
        v = _ou(seed, 1, rows, 3 * case["atoms"])
        q = _ou(seed, 2, rows, 3, lo=50.0, hi=50.0)
        return [torch.cat([v, q, q], 1), q]
    pos = _positions(seed, 5, rows, case["atoms"])
    if kind == "batched":
        return [_ou(seed, 1, rows, case["n"]), pos, _ou(seed, 3, rows, 9, "f64")]
    if kind == "rhok":
        return [pos]
    both = torch.cat([pos, _ou(seed, 8, rows, 3 * case["atoms"]).reshape(rows, 3, -1)], 1)
    return [both] if kind == "currents" else [both, pos]


def prepare(case, seed):
    frames = _inputs(case, seed)
    groups = _groups(case, seed)
    graph = case["kind"] == "batched"
    tuning = dict(tile_channels=256, chans_per_thread=2, lag_chunk=8, grid_blocks=2048,
                  overlap_producers=1, fold_threads=128) if graph else None
    corr = Correlator(groups, device=0, graph=graph, tuning=tuning)
    state = dict(case=case, corr=corr, frames=frames, at=0)
    if graph:  # steps one by one, as before the stretches that the passes replay
        _push(state, case["fill"])
        state["at"] = 0
    else:
        _push(state, case.get("fill", 0))
    return state


def _push(state, steps):
    corr, frames, rows = state["corr"], state["frames"], state["case"]["rows"]
    for _ in range(steps):
        r = state["at"]
        corr.push([f[r] for f in frames])
        state["at"] = r + 1 if r + 1 < rows else 0


# -------------------------------------------------------------------- the pass
def _kept(group, r):
    """A readout in the precision of the group's sums."""
    cplx = group.dtype in ("cf32", "cf64")
    real, comp = (np.float64, np.complex128) if group.accum == "f64" else (np.float32, np.complex64)
    out = {"t": r["t"], "count": r["count"], "c": r["c"].astype(comp if cplx else real),
           "gk_running": r["gk_running"].astype(real)}
    if "c_per_channel" in r:
        out["c_per_channel"] = r["c_per_channel"].astype(comp if cplx else real)
    return out


def _readouts(case):
    """finalize()'s arguments for every group of a case."""
    kind = case["kind"]
    if kind in ("samples", "cross"):
        kw = {}
        if case["per"]:
            kw["slice_"] = (0, case["per"])
        if case["gk"]:
            kw.update(gk_kind=case["gk"], volume=BOX ** 3, kB=0.831, temperature=90.0)
        return [kw]
    if kind == "massflux":
        return [dict(slice_=(0, 6)), dict(gk_kind=2, volume=BOX ** 3, kB=0.831, temperature=90.0)]
    if kind == "batched":
        return [{}, dict(slice_=(0, case["nk"])), dict(slice_=(0, 9))]
    if kind == "kgap":  # the transverse functions of the whole set are averaged
        return [{}, {}]
    return [dict(slice_=(0, (3 if kind == "currents" else 1) * case["nk"]))]


def run(state):
    case, corr = state["case"], state["corr"]
    if case["kind"] == "batched":
        for _ in range(case["steps"] // case["rows"]):
            corr.push_steps(state["frames"])
    elif case.get("mode") == "replay":
        corr.push_steps(state["frames"])
    else:
        _push(state, case["steps"])
    return [_kept(g, corr.finalize(i, **kw))
            for i, (g, kw) in enumerate(zip(corr.groups, _readouts(case)))]


# -------------------------------------------------------- what a pass must do
def _shape(case):
    """(channels, sample bytes, sum bytes, levels, points, series) of every group."""
    kind = case["kind"]
    if kind in ("samples", "cross"):
        s = 8 if case["dtype"] == "f64" else 4
        return [(case["n"], s, 8, case["levels"], case["points"], 2 if kind == "cross" else 1)]
    if kind == "massflux":
        return [(6, 4, 8, case["levels"], case["points"], 2), (3, 4, 8, case["levels"], case["points"], 1)]
    if kind == "batched":
        return [(case["n"], 4, 8, 10, 16, 1), (case["nk"], 8, 16, 16, 32, 1), (9, 8, 8, 20, 16, 1)]
    lv = 1 if kind == "kgap" else case["levels"]
    sh = [(3 * case["nk"], 8, 16, lv, case["points"], 1), (case["nk"], 8, 16, lv, case["points"], 1)]
    return sh if kind == "kgap" else sh[:1] if kind == "currents" else sh[1:]


def work(case):
    """Each frame read once, the sums and the values that later steps look back
    to read and written once, the readout written once; the lag products, and 14
    (n(k)) or 26 (currents) operations per atom and k-vector."""
    steps, kind = case["steps"], case["kind"]
    nbytes = flops = 0.0
    for n, s, a, lv, p, series in _shape(case):
        half, cplx = p - p // 2, 4 if s == 8 and a == 16 else 1
        got = [steps >> k for k in range(lv)]
        lags = [p if k == 0 else half for k in range(lv)]
        if kind == "kgap":
            lags = [min(p, steps)]
        live = sum(l for l, v in zip(lags, got) if v)
        nbytes += n * (2.0 * a * live + 2.0 * s * series * sum(min(v, p) for v in got))
        if kind in ("samples", "cross") or (kind == "batched" and a != 16):
            nbytes += float(n) * s * series * min(steps, case["rows"])
        flops += 2.0 * cplx * n * sum(l * v for l, v in zip(lags, got))
    atoms, nk, frames = case.get("atoms", 0), case.get("nk", 0), min(steps, case["rows"])
    if kind in ("rhok", "batched"):
        nbytes += 12.0 * atoms * frames
        flops += 14.0 * atoms * nk * steps
    elif kind in ("currents", "kgap"):
        nbytes += 24.0 * atoms * frames
        flops += (26.0 if kind == "currents" else 40.0) * atoms * nk * steps
    elif kind == "massflux":
        nbytes += 13.0 * atoms * frames
        flops += 6.0 * atoms * steps
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------------ the same in 64 bits
def _sequence(case):
    """The frame of every step up to the end of the first pass."""
    rows, fill, steps = case["rows"], case.get("fill", 0), case["steps"]
    before = [i % rows for i in range(fill)]
    start = 0 if case["kind"] == "batched" or case.get("mode") == "replay" else fill
    return before + [(start + i) % rows for i in range(steps)]


def _lags(levels, points, total):
    """The (level, lag, count) of a readout after `total` steps, in its order."""
    out = []
    for k in range(levels):
        got = total >> k
        out += [(k, lag, got - lag) for lag in range(0 if k == 0 else points // 2, points) if got > lag]
    return out


def _sums(x, y, entries):
    """[entry][channel] sums of x(s) conj(y(s - lag)) over the block means."""
    level, out = 0, []
    for k, lag, _ in entries:
        while level < k:
            m = (x.shape[0] // 2) * 2
            x, y = 0.5 * (x[0:m:2] + x[1:m:2]), 0.5 * (y[0:m:2] + y[1:m:2])
            level += 1
        out.append((x[lag:] * y[:x.shape[0] - lag].conj()).sum(0))
    return torch.stack(out)


def _functions(case, g, x, y, seq, norm, kw):
    """One group's readout from its series [row][channel]."""
    entries = _lags(g.levels, g.points, len(seq))
    n, per = x.shape[1], kw.get("slice_", (0, 0))[1]
    at = torch.tensor(seq, device=DEV)
    wide = torch.complex128 if x.is_complex() else torch.float64
    step = max(1, min(n, (1 << 27) // len(seq)))
    total, first = torch.zeros(len(entries), dtype=wide, device=DEV), []
    for c in range(0, n, step):
        xs = x[:, c:c + step].to(wide)[at]
        ys = xs if y is x else y[:, c:c + step].to(wide)[at]
        s = _sums(xs, ys, entries)
        total += s.sum(1)
        if c < per:
            first.append(s[:, :per - c].clone())
    count = np.array([e[2] for e in entries])
    t = np.array([float(lag) * 2.0 ** k * g.update_every * g.dt for k, lag, _ in entries])
    c = total.cpu().numpy() / count / n * norm
    mid = np.concatenate([[0.0], np.cumsum(0.5 * np.diff(t) * (c.real[1:] + c.real[:-1]))])
    scale = 1.0
    if kw.get("gk_kind") == 1:
        scale = kw["volume"] / (kw["kB"] * kw["temperature"])
    elif kw.get("gk_kind") == 2:
        scale = kw["volume"] / (kw["kB"] * kw["temperature"] ** 2)
    out = {"t": t, "count": count.astype(np.int64), "c": c, "gk_running": mid * scale}
    if per:
        out["c_per_channel"] = torch.cat(first, 1).cpu().numpy().T / count[None, :] * norm
    return out


def _waves(frame, kv, velocities):
    """n(k) [nk], or the currents [nk][3 components], of one frame in double."""
    k = torch.tensor(kv, device=DEV)
    pair, row = torch.unique(k[:, :2], dim=0, return_inverse=True)
    z, col = torch.unique(k[:, 2], return_inverse=True)
    nw, atoms = 3 if velocities else 1, frame.shape[1]
    total = torch.zeros(nw, len(pair), len(z), dtype=torch.complex128, device=DEV)
    for a in range(0, atoms, 1 << 16):
        r = frame[:3, a:a + (1 << 16)].double() * (2.0 * math.pi / BOX)
        p = torch.polar(torch.ones((), dtype=torch.float64, device=DEV),
                        pair[:, :1].double() * r[0] + pair[:, 1:].double() * r[1])
        q = torch.polar(torch.ones((), dtype=torch.float64, device=DEV), r[2][:, None] * z.double()[None, :])
        for w in range(nw):
            v = q * frame[3 + w, a:a + (1 << 16)].double()[:, None] if velocities else q
            total[w] += p @ v.contiguous()
    return total[:, row, col]


def _basis(kv):
    """khat and the two transverse directions of every k-vector."""
    k = kv.astype(np.float64)
    kh = k / np.linalg.norm(k, axis=1, keepdims=True)
    e1 = np.eye(3)[np.argmin(np.abs(kh), axis=1)]
    e1 = e1 - (e1 * kh).sum(1, keepdims=True) * kh
    e1 /= np.linalg.norm(e1, axis=1, keepdims=True)
    return np.stack([kh, e1, np.cross(kh, e1)], 1)


def _series(source, frames, case):
    """[row][channel] of a producer's group in double."""
    kv = _kvectors(case["nk"])
    if source == "rhok":
        return torch.stack([_waves(f, kv, False)[0] for f in frames])
    basis = torch.tensor(_basis(kv), device=DEV, dtype=torch.complex128)
    return torch.stack([(basis @ _waves(f, kv, True).T.contiguous()[:, :, None])[:, :, 0].reshape(-1)
                        for f in frames])


def exact(case, seed):
    frames, seq, out = _inputs(case, seed), _sequence(case), []
    for i, (g, kw) in enumerate(zip(_groups(case, seed), _readouts(case))):
        norm = 1.0
        if g.source in ("rhok", "currents"):
            x = y = _series(g.source, frames[i], case)
            norm = 1.0 / case["atoms"]
        elif g.source == "momentum":
            atoms, sp = case["atoms"], torch.tensor(g.species, device=DEV)
            v = frames[i][:, :3 * atoms].reshape(-1, 3, atoms)
            y = torch.stack([torch.stack([torch.stack([f[d][sp == s].double().sum() for d in range(3)])
                                          * (LIF[s] / BOX ** 3) for s in range(2)]).reshape(-1) for f in v])
            x = frames[i][:, 3 * atoms:]
        elif g.pair:
            x, y = frames[i][:, :case["n"]], frames[i][:, case["n"]:]
        else:
            x = y = frames[i]
        out.append(_functions(case, g, x, y, seq, norm, kw))
    return out
