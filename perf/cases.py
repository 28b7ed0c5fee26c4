"""Workloads whose speed is followed: what a user of the sweep library has it do.

A pass of a case is one step of a simulation program's own loop:

  run       n sweeps of every system, then the densities (device) and, where
            `observe` is set, the observables of every system
  coupled   start of a coupled run: chains placed from target concentration
            fields, umbrella on, n sweeps, densities, classes, observables
  save      one checkpoint (raw state and chain classes) or one trajectory
            frame (FP64 positions) to host memory
  resume    a saved state and sweep number set on a context, one sweep,
            density
  analyse   observables, fields and densities of the present configuration
            to host memory

Sizes are those of paper_2606_09356_amd.workloads, of the tests (odd chain
lengths, ragged boxes) and in between.  A context that the program keeps is
made in `prepare`; its seed keys every random number, so another seed is
another trajectory.  The launch shapes are the library's defaults or those
that its autotuner settles on for the workload.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2606_09356_amd import workloads as W
from paper_2606_09356_amd.soma import Soma

DELTA = 0.05        # move half-width, Re
RHO = 128.0         # beads per Re^3
# FP32 and integer operations of one bead move: ten Philox rounds (two
# products and four XORs/adds each), proposal, two cells, field, bond energy
OPS_PER_MOVE = 130


def listed():
    shape = dict(mode=0, tiling=0, waves=0, resident=0, order=0)
    return [
        # the smallest call: a small melt that the program looks at after every sweep
        dict(name="small_monitor", kind="run", systems="plain_small", repr="f32", width=16, **shape,
             reorder=0, sweeps=1, observe=True),
        # a production stretch of the same melt (latency of a sweep is what counts)
        dict(name="small_run", kind="run", systems="plain_small", repr="f32", width=16, mode=1, tiling=0, waves=1,
             resident=8, order=0, reorder=100, sweeps=100, observe=True),
        # odd chain length, ragged box, wide counts, default launch shape
        dict(name="ragged_run", kind="run", systems="one", chains=20011, N=37, arch="ABA", f=0.45, chiN=24.0,
             kappaN=60.0, nx=83, ny=71, nz=63, form=1, smc_A=0.0, repr="f32", width=32, **shape, reorder=50,
             sweeps=20, observe=True),
        # the plain single-system form: 4.2M beads
        dict(name="plain_run", kind="run", systems="plain_large", repr="f32", width=16, mode=2, tiling=0, waves=1,
             resident=0, order=1, reorder=100, sweeps=50, observe=True),
        # one large melt, cell + offset positions and wide counts: 16.8M beads
        dict(name="mixed_run", kind="run", systems="mixed_large", repr="cell", width=32, mode=3, tiling=0, waves=4,
             resident=0, order=1, reorder=100, sweeps=25, observe=True),
        # a parameter study: 64 melts of uneven size in one launch, every one looked at
        dict(name="uneven_batch", kind="run", systems="batched_uneven", n_systems=64, repr="f32", width=16, mode=3,
             tiling=2, waves=4, resident=0, order=1, reorder=100, sweeps=50, observe=True),
        # the largest: 256 systems of every architecture, 124.6M beads
        dict(name="mixed_batch", kind="run", systems="batched_mixed", n_systems=256, repr="cell", width=16, mode=3,
             tiling=2, waves=4, resident=0, order=1, reorder=100, sweeps=20, observe=False),
        # bond-force-biased moves
        dict(name="smart_run", kind="run", systems="plain_large_smc", repr="f32", width=16, mode=3, tiling=0, waves=4,
             resident=0, order=0, reorder=100, sweeps=25, observe=True),
        # particle subdomain of a coupled run: walls, conversion zones, umbrella
        dict(name="coupled_start", kind="coupled", chains=16384, N=32, arch="AB", f=0.5, chiN=20.0, kappaN=50.0,
             nx=64, ny=64, nz=64, form=0, smc_A=0.0, wall=2, zone=4, umbrella=10.0, repr="cell", width=16, **shape,
             reorder=0, sweeps=10),
        # checkpoint of a 4.2M-bead run, and its resumption
        dict(name="checkpoint_save", kind="save", what="state", chains=65536, N=64, arch="AB", f=0.5, chiN=30.0,
             kappaN=50.0, nx=128, ny=128, nz=128, form=0, smc_A=0.0, repr="cell", width=16, **shape, reorder=100),
        dict(name="checkpoint_resume", kind="resume", chains=32768, N=32, arch="AB", f=0.5, chiN=20.0, kappaN=50.0,
             nx=81, ny=81, nz=80, form=0, smc_A=0.0, repr="f32", width=16, **shape, reorder=100),
        # fields, densities and observables of one configuration for a plot or a coupled code
        dict(name="analysis", kind="analyse", chains=65536, N=32, arch="AB", f=0.5, chiN=20.0, kappaN=50.0,
             nx=128, ny=128, nz=64, form=0, smc_A=0.0, repr="f32", width=16, **shape, reorder=0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_one(rng, lo, hi):
    """A single system of lo..hi beads, any chain length, ragged box."""
    N = rng.choice([_log(rng, 2, 128), rng.randint(8, 128), 16, 32, 64])
    beads = _log(rng, lo, hi)
    chains = max(4, beads // N)
    edge = max(4.0, (chains * N / 2.0) ** (1.0 / 3.0))
    nx, ny = (max(4, int(round(edge * rng.uniform(0.7, 1.4)))) for _ in range(2))
    nz = max(6, int(round(chains * N / 2.0 / (nx * ny))))
    return dict(chains=chains, N=N, arch=rng.choice(["AB", "ABA", "blend"]), f=round(rng.uniform(0.3, 0.7), 3),
                chiN=round(rng.uniform(0.0, 50.0), 2), kappaN=round(rng.uniform(25.0, 100.0), 2), nx=nx, ny=ny, nz=nz,
                form=rng.randint(0, 1), smc_A=0.0)


def _draw_shape(rng, modes=(0, 1, 2, 3)):
    tiling = rng.choice([0, 0, 2, 1])
    return dict(repr=rng.choice(["f32", "cell"]), width=rng.choice([16, 16, 32]), mode=rng.choice(list(modes)),
                tiling=tiling, waves=rng.choice([0, 1, 4, 8]), resident=0, order=rng.randint(0, 1),
                reorder=rng.choice([0, 50, 100]))


def draw(rng):
    kind = rng.choice(["run", "run", "run", "batch", "smart", "coupled", "save", "resume", "analyse"])
    if kind == "batch":
        n = _log(rng, 2, 64)
        which = rng.choice(["batched_uneven", "batched_mixed"])
        c = dict(kind="run", systems=which, n_systems=n, table=rng.randint(1, 10 ** 6), **_draw_shape(rng),
                 sweeps=rng.randint(5, 20), observe=n <= 16)
    elif kind in ("run", "smart"):
        one = _draw_one(rng, 2048, 8e6)
        if kind == "smart":
            one["smc_A"] = rng.choice([2e-4, 4e-4])
        c = dict(kind="run", systems="one", **one, **_draw_shape(rng), sweeps=_log(rng, 1, 40), observe=True)
    elif kind == "coupled":
        one = _draw_one(rng, 2e4, 1e6)
        one["nz"] = max(one["nz"], 24)
        zone = rng.choice([0, 3])
        c = dict(kind="coupled", **one, wall=2, zone=zone, umbrella=round(rng.uniform(1.0, 20.0), 2),
                 **_draw_shape(rng, (0, 1)), sweeps=rng.randint(1, 20))
        c["reorder"] = 0
        if zone:
            c["tiling"] = 0
    elif kind == "save":
        c = dict(kind="save", what=rng.choice(["state", "positions"]), **_draw_one(rng, 1e5, 4e6), **_draw_shape(rng))
    elif kind == "resume":
        c = dict(kind="resume", **_draw_one(rng, 1e5, 1.5e6), **_draw_shape(rng))
    else:
        c = dict(kind="analyse", **_draw_one(rng, 1e5, 2e6), **_draw_shape(rng))
        c["reorder"] = 0
    return c


def _patterns(case):
    """Patterns a and b of the case's architecture and how many chains carry a."""
    N, n = case["N"], case["chains"]
    a, b = np.zeros(N, np.uint8), np.ones(N, np.uint8)
    if case["arch"] == "blend":
        return a, b, int(round(case["f"] * n))
    na = min(max(int(math.floor(case["f"] * N + 0.5)), 1), N - 1)
    a[:] = 1
    if case["arch"] == "ABA" and N > 2 and na >= 2:
        a[:na // 2] = 0
        a[N - (na - na // 2):] = 0
    else:
        a[:na] = 0
    return a, a.copy(), n


def _geometry(case):
    """Box and grid at RHO beads per Re^3 with cubic cells."""
    grid = (case["nx"], case["ny"], case["nz"])
    edge = (case["chains"] * case["N"] / RHO / (grid[0] * grid[1] * grid[2])) ** (1.0 / 3.0)
    # a box of the usual two beads per cell keeps the cell edge near Re/4;
    # very small systems on a minimal grid get larger moves' worth of room
    edge = max(edge, 2.5 * DELTA)
    if abs(edge - 0.25) < 1e-6:
        edge = 0.25
    return tuple(edge * g for g in grid), grid


def _one(case):
    pa, pb, n_a = _patterns(case)
    box, grid = _geometry(case)
    s = W.SystemDesc(n_chains=case["chains"], N=case["N"], pattern_a=pa, pattern_b=pb, n_chains_a=n_a,
                     chiN=case["chiN"], kappaN=case["kappaN"], box=box, grid=grid, move_halfwidth=DELTA,
                     ham_form=case["form"], smc_A=case["smc_A"])
    if case.get("wall"):
        s.walls = (case["wall"], grid[2] - case["wall"])
        if case.get("zone"):
            s.zones = (case["zone"], case["zone"])
            s.n_chains_a, s.pattern_b = case["chains"] // 2, (1 - pa).astype(np.uint8)
    return s


def _systems(case):
    which = case.get("systems", "one")
    if which == "one":
        return [_one(case)]
    if which in ("batched_uneven", "batched_mixed"):
        make = W.batched_uneven if which == "batched_uneven" else W.batched_mixed
        return make(n_systems=case["n_systems"], seed=case.get("table"))
    return W.workload(which)


def _context(case, systems, seed, coupling=False):
    return Soma(systems, seed=20260609 + seed, pos_repr=case["repr"], count_width=case["width"], use_graph=True,
                density_mode=case["mode"], packed_tiles=case["tiling"], waves_per_block=case["waves"],
                waves_per_cu=case["resident"], launch_order=case["order"], reorder_every=case["reorder"],
                coupling=coupling)


def _targets(case, grid, seed):
    """Target concentrations of a coupled run: a lamellar profile with noise."""
    rng = np.random.default_rng([seed, 7])
    z = np.arange(grid[2]) / grid[2]
    a = 0.5 + 0.35 * np.sin(2.0 * np.pi * (2.0 * z + rng.uniform()))
    noise = rng.uniform(-0.1, 0.1, size=grid)
    phi = np.stack([a[None, None, :] + noise, 1.0 - a[None, None, :] - noise]).astype(np.float32)
    # nothing outside the slab, with room for a chain to fit in it
    margin = case["wall"] + max(2, grid[2] // 8)
    phi[..., :margin] = 0.0
    phi[..., grid[2] - margin:] = 0.0
    return np.ascontiguousarray(phi.reshape(2, -1))


def _walks(case, seed):
    """Gaussian-walk positions [3, beads] (float64, host) for the analysis."""
    box, _ = _geometry(case)
    rng = np.random.default_rng([seed, 11])
    n, N = case["chains"], case["N"]
    xyz = np.empty((3, n, N))
    sigma = 1.0 / math.sqrt(3.0 * (N - 1))
    for d in range(3):
        b = rng.standard_normal((n, N), dtype=np.float32).astype(np.float64) * sigma
        b[:, 0] = rng.random(n) * box[d]
        np.cumsum(b, axis=1, out=xyz[d])
    return xyz.reshape(3, -1)


def prepare(case, seed):
    kind = case["kind"]
    systems = _systems(case)
    g = _context(case, systems, seed, coupling=kind == "coupled")
    st = dict(case=case, g=g, systems=systems)
    if kind != "save" and kind != "analyse":
        cells = [s.n_cells for s in systems]
        st["counts"] = torch.zeros(2 * sum(cells), dtype=torch.int32, device="cuda")
        st["views"], at = [], 0
        for m in cells:
            st["views"].append(st["counts"][at:at + 2 * m])
            at += 2 * m
    if kind == "coupled":
        st["targets"] = _targets(case, systems[0].grid, seed)
    elif kind == "save":
        g.sweep(2)
    elif kind == "resume":
        g.sweep(3)
        st["saved"] = g.state(0)
        st["sweep"] = g.info()["sweep"]
    elif kind == "analyse":
        g.set_positions(0, _walks(case, seed))
    g.sync()
    return st


def _observables(g, n):
    got = [g.observables(k) for k in range(n)]
    return {k: np.array([o[k] for o in got]) for k in got[0]}


def run(st):
    case, g, kind = st["case"], st["g"], st["case"]["kind"]
    out = {}
    if kind == "run":
        g.sweep(case["sweeps"])
        if case["observe"]:
            out = _observables(g, len(st["systems"]))
    elif kind == "coupled":
        g.place_from_fields(0, st["targets"])
        g.set_umbrella(0, case["umbrella"])
        g.sweep(case["sweeps"])
        out = _observables(g, 1)
        out["classes"] = g.classes(0)
    elif kind == "save":
        if case["what"] == "positions":
            return {"positions": g.positions(0)}
        s = g.state(0)
        out = {"cell": s[1], "offset": s[0]} if case["repr"] == "cell" else {"xyz": s}
        out["classes"] = g.classes(0)
        return out
    elif kind == "resume":
        s = st["saved"]
        if case["repr"] == "cell":
            g.set_state(0, s[0], s[1])
        else:
            g.set_state(0, s)
        g.set_sweep(st["sweep"])
        g.sweep(1)
    else:
        out = _observables(g, 1)
        for k in ("accept_ratio", "n_moves", "n_accepted", "sweep", "converted_to_a", "converted_to_b"):
            del out[k]
        out["fields"] = g.fields(0)
        out["density"] = g.density(0)
        return out
    for k, v in enumerate(st["views"]):
        g.density_device(k, v)
    out["density"] = st["counts"]
    return out


def work(case):
    systems = _systems(case)
    beads = sum(s.n_beads for s in systems)
    cells = sum(s.n_cells for s in systems)
    pos = 12 if case["repr"] == "f32" else 24
    cnt = 4 if case["width"] == 16 else 8
    kind = case["kind"]
    sweeps = case["sweeps"] if kind in ("run", "coupled") else 1 if kind == "resume" else 0
    # a sweep reads and writes every position and every count
    b = sweeps * (2.0 * pos * beads + 2.0 * cnt * cells)
    ops = float(sweeps) * OPS_PER_MOVE * beads
    if kind == "save":
        b += pos * beads + (24 if case["what"] == "positions" else pos) * beads
        ops += beads
    elif kind == "analyse":
        # positions read for the observables, counts read three times
        b += pos * beads + 3.0 * cnt * cells + 16.0 * cells
        ops += 60.0 * beads
    else:
        if kind == "resume":
            b += 2.0 * pos * beads
        if kind == "coupled":
            b += 8.0 * cells + pos * beads
            ops += 200.0 * beads
        if case.get("observe") or kind == "coupled":
            b += pos * beads + cnt * cells
            ops += 30.0 * beads
        b += cnt * cells + 8.0 * cells          # density read, and written as two words per cell
    return {"bytes": float(b), "flops": float(ops)}


def exact(case, seed):
    """The analysis in 64 bits from FP32 positions (a trajectory has no such value:
    a rounding decides an acceptance, and the acceptance all that follows)."""
    if case["kind"] != "analyse" or case["repr"] != "f32":
        return None
    n, N = case["chains"], case["N"]
    box, grid = _geometry(case)
    M, B = grid[0] * grid[1] * grid[2], n * N
    r = _walks(case, seed).astype(np.float32).astype(np.float64).reshape(3, n, N)
    idx = np.zeros((n, N), np.int64)
    for d in range(3):
        e = float(np.float32(box[d] / grid[d]))
        k = np.floor(r[d] / e)
        k -= k * e > r[d]
        k += (k + 1.0) * e <= r[d]
        idx = idx * grid[d] + np.mod(k.astype(np.int64), grid[d])
    pa, pb, n_a = _patterns(case)
    types = np.where((np.arange(n) < n_a)[:, None], pa[None, :], pb[None, :])
    counts = np.stack([np.bincount(idx[types == t], minlength=M) for t in (0, 1)])
    phi = counts * (M / B)
    inc = phi[0] + phi[1] - 1.0
    chiN, kN = case["chiN"], case["kappaN"]
    if case["form"] == 0:
        w = np.stack([kN * inc - 0.5 * chiN * (phi[0] - phi[1]), kN * inc + 0.5 * chiN * (phi[0] - phi[1])]) / N
        h = 0.5 * kN * inc ** 2 - 0.25 * chiN * (phi[0] - phi[1]) ** 2
    else:
        w = np.stack([chiN * phi[1] + kN * inc, chiN * phi[0] + kN * inc]) / N
        h = chiN * phi[0] * phi[1] + 0.5 * kN * inc ** 2
    e2 = ((r[:, :, -1] - r[:, :, 0]) ** 2).sum(0)
    g2 = ((r - r.mean(axis=2, keepdims=True)) ** 2).sum(0).mean(1)
    bonds = ((r[:, :, 1:] - r[:, :, :-1]) ** 2).sum(0).sum(1) * (1.5 * (N - 1))
    err = lambda v: math.sqrt(max((v * v).mean() - v.mean() ** 2, 0.0) / n)  # noqa: E731
    one = lambda v: np.array([float(v)])  # noqa: E731
    return {"Re2": one(e2.mean()), "Re2_err": one(err(e2)), "Rg2": one(g2.mean()), "Rg2_err": one(err(g2)),
            "Ebond_per_chain": one(bonds.mean()), "Enb_per_chain": one((B / M) / N * h.sum() / n), "fields": w,
            "density": counts.astype(np.uint32)}
