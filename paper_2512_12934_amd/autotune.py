"""Autotuner of the node-update launch configuration.

Every configuration of the tuning space (lattice-specific tile shape, sweep
depth, psi source, register policy; see ``csrc/launch.h``) computes exactly
the same arithmetic per node, so the tuner runs each one on a workload,
checks that the state after the timed steps is bitwise equal to that of
configuration 0, and records its pick (see ``pick``) in ``tuning.json`` keyed
by lattice, storage and size class.  ``LBM(..., tile_config="auto")`` reads
that table; a class it does not hold takes the library's own choice, which
knows fewer classes.

    python -m paper_2512_12934_amd.autotune --workload coflow3d --steps 50

    # the table
    python -m paper_2512_12934_amd.autotune --workload table --steps 64 --write
"""
from __future__ import annotations

import argparse
import copy
import functools
import json
import os
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
TABLE = os.path.join(HERE, "tuning.json")


# Upper bounds (box nodes) of the size classes.  The best work item shrinks
# with the domain, from 16 rows or 4 planes where the halo it re-reads is what
# costs, to one pass of a block where too few items would leave CUs idle; the
# classes end where the measured picks of either lattice change.
CLASSES = ((100_000, "100k"), (250_000, "250k"), (450_000, "450k"), (1_000_000, "1M"), (3_000_000, "3M"),
           (5_000_000, "5M"), (16_000_000, "16M"))


def size_class(nodes: int) -> str:
    for limit, name in CLASSES:
        if nodes < limit:
            return name
    return "max"


def key(dim: int, storage: str, nodes: int) -> str:
    return f"d{dim}-{storage}-{size_class(nodes)}"


@functools.lru_cache(maxsize=1)
def _parse(path: str, stamp: tuple) -> dict:
    with open(path) as fh:
        return json.load(fh)


def _table() -> dict:
    # every context that asks for a tuned tile looks it up: the file is parsed
    # once per version of it (0.16 ms, a quarter of what the smallest context
    # takes to create)
    if not os.path.exists(TABLE):
        return {}
    st = os.stat(TABLE)
    return _parse(TABLE, (st.st_mtime_ns, st.st_size, st.st_ino))


def load_table() -> dict:
    return copy.deepcopy(_table())


def lookup(dim: int, storage: str, nodes: int) -> int:
    # both binary16 codecs move the same bytes: the fixed-offset form takes
    # the reference-density form's tuning
    entry = _table().get(key(dim, "f16" if storage == "f16fixed" else storage, nodes))
    return int(entry["best"]) if entry else -1


# Domains whose fluid fills 64-wide tiles badly: the lanes of the 64-wide tiles
# that hold fluid, over those of the 32-wide ones.  From NARROW on (a channel 70
# wide fills half of its second tile) the latter are faster: node updates with
# 64 / 32 columns 97x5000 FP32 28.9 / 26.1 us, 16x200x200 129 / 107, 70x70x70
# binary16 51 / 39; below it, 130x4000 32.6 / 33.2, 130x60x60 56.0 / 55.6.  From
# ONE_TILE on (a single 32-wide tile across) the fused 2-D mode, whose halo
# columns then hold little, beats the two-pass one: 33x8000 14.9 / 16.4, 33x40000
# 55.5 / 65.2; below it, 65x5000 26.1 / 22.8.
NARROW, ONE_TILE = 1.25, 1.75


def lane_ratio(members, layout="caller") -> float:
    """Lanes in 64-wide tiles over lanes in 32-wide tiles, of one domain or of
    a batch (1.0 where there is no fluid)."""
    import numpy as np
    lanes = {32: 0, 64: 0}
    for c in members:
        faces = [c.outlet] if c.outlet is not None else c.inlets
        turned = layout == "face_last" and c.dim == 3 and len(faces) > 0 and faces[0]["axis"] == 0
        x = 1 if turned else 0              # the caller's axis that is contiguous in memory
        nz, ny, nx = (c.n[2] if c.dim == 3 else 1), c.n[1], c.n[0]
        fluid = (np.asarray(c.solid).reshape(nz, ny, nx) == 0).any(axis=tuple(a for a in range(3) if a != 2 - x))
        for w in lanes:
            tiles = np.add.reduceat(fluid, np.arange(0, len(fluid), w)) > 0
            lanes[w] += int(tiles.sum()) * w * (c.N // c.n[x])
    return lanes[64] / lanes[32] if lanes[32] else 1.0


def choose(members, storage: str, layout="caller") -> int:
    """The tile that tile_config="auto" stands for: the class's pick, or for
    narrow domains the class's fastest of at most 32 columns."""
    from .lbm import tile_config_desc, tile_configs
    dim, nodes = members[0].dim, sum(c.N for c in members)
    best = lookup(dim, storage, nodes)
    if best < 0:
        return best
    desc = {c: tile_config_desc(dim, c) for c in range(tile_configs(dim))}
    if desc[best]["tx"] <= 32 and (dim == 3 or desc[best]["psrc"] == 0):
        return best
    ratio = lane_ratio(members, layout)
    if ratio < (NARROW if desc[best]["tx"] > 32 else ONE_TILE):
        return best
    entry = _table()[key(dim, "f16" if storage == "f16fixed" else storage, nodes)]
    fits = lambda d: d["tx"] <= 32 and (dim == 3 or ratio < ONE_TILE or d["psrc"] == 0)
    times = {int(c): t for c, t in entry["ms_per_step"].items() if entry["identical"][c] and fits(desc[int(c)])}
    return min(times, key=times.get) if times else best


def pick(times: dict, identical: dict, prefer=None):
    """The fastest configuration whose state equals that of configuration 0.
    Times within 2% count as equal (what runs of one configuration differ by on
    one device), and of equals ``prefer``, the pick of the next larger size
    class, is kept, so that the picks change with the size only where it gains."""
    good = {c: t for c, t in times.items() if identical[c]}
    best = min(good, key=good.get)
    return prefer if prefer in good and good[prefer] <= 1.02 * good[best] else best


def larger_class(dim: int, storage: str, nodes: int):
    """Key of the next larger size class, or None for the largest."""
    names = [name for _, name in CLASSES] + ["max"]
    i = names.index(size_class(nodes)) + 1
    return f"d{dim}-{storage}-{names[i]}" if i < len(names) else None


def tune(work, storage: str, steps: int, warmup: int, prefer=None, log=print) -> dict:
    """``work``: a case, or a list of them to be stepped as one batch."""
    import numpy as np
    import torch

    from .lbm import LBM, Batch, tile_configs

    batch = isinstance(work, list)
    members = work if batch else [work]
    name = f"batch of {len(work)} {work[0].name.split('_')[0]} members" if batch else f"{work.name} {work.n}"
    times, ok = {}, {}
    ref = None
    for cfg in range(tile_configs(members[0].dim)):
        sim = (Batch if batch else LBM)(work, storage=storage, tile_config=cfg)
        # capture both step graphs before timing, so no configuration's time
        # includes a capture
        sim.set_graph_steps(16)
        sim.step(warmup)
        ms = float("inf")
        for _ in range(3):
            torch.cuda.synchronize()
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record(sim.stream)
            sim.step(steps)
            t1.record(sim.stream)
            torch.cuda.synchronize()
            ms = min(ms, t0.elapsed_time(t1) / steps)
        # the first, middle and last member of a batch; of a large domain the densities
        seen = sorted({0, len(members) // 2, len(members) - 1})
        ctx = [sim.members[i] for i in seen] if batch else [sim]
        state = [s.get_state() if s.N <= 4_000_000 else s.moments()[0] for s in ctx]
        if ref is None:
            ref = state
        ok[cfg] = all(np.array_equal(a, b) for a, b in zip(state, ref))
        times[cfg] = round(ms, 5)
        diff = max(float(np.abs(a - b).max()) for a, b in zip(state, ref))
        log(f"[autotune] {name} {storage} cfg {cfg}: {ms:.4f} ms/step, identical={ok[cfg]} max|diff|={diff:.3e}")
        del sim, ctx
        torch.cuda.empty_cache()
    return {"best": pick(times, ok, prefer), "ms_per_step": times, "identical": ok, "steps": steps, "workload": name,
            "fluid_nodes": sum(c.fluid_nodes for c in members)}


# Workloads by name: a case, or a list of cases for a batch.
WORKLOADS = {
    "taylor": lambda c: c.taylor(5.0, 0.05, nx=320, H=160, R=32.0),
    "tjunction": lambda c: c.tjunction(),
    "tjunction_small": lambda c: c.tjunction(W=32, length=256, x_side=48, side_width=32, side_len=32),
    "droplet_540": lambda c: c.laplace(n=540, R=135.0),
    "droplet_900": lambda c: c.laplace(n=900, R=225.0),
    "tjunction_W256": lambda c: c.sweep_case(256, 0.03, 0.5, 1.0),
    # the sweep geometry at W = 512 (2.4M fluid nodes)
    "tjunction_W512": lambda c: c.sweep_case(512, 0.03, 0.5, 1.0),
    "tjunction_large": lambda c: c.sweep_case(512, 0.01, 0.5, 1.0),
    # the batched sweep, and a quarter of it
    "sweep_64": lambda c: c.sweep(64),
    "sweep_256": lambda c: c.sweep(256),
    "coflow3d_80": lambda c: c.coflow3d(length=80, width=16, inner=4),
    "coflow3d_quarter": lambda c: c.coflow3d_quarter(),
    "coflow3d_200": lambda c: c.coflow3d(length=200, width=40, inner=10),
    "channel3d_250": lambda c: c.channel(250, 51, 0.02, nu=(0.17, 0.17), droplet=(45.0, 26.0, 26.0, 15), dim=3,
                                         major=c.COEX_G09[0], minor=c.COEX_G09[1]),
    "coflow3d_half": lambda c: c.coflow3d(length=300, width=60, inner=15),
    "coflow3d_400": lambda c: c.coflow3d(length=400, width=90, inner=20),
    "coflow3d": lambda c: c.coflow3d(),
}
# The one that stands for each size class of the table, larger classes first
# (a pick depends on the next larger one's).  3-D domains beyond 16M nodes have
# none and take the library's choice.
TABLE_WORKLOADS = ("sweep_256", "sweep_64", "tjunction_W512", "tjunction_W256", "droplet_900", "droplet_540",
                   "tjunction", "taylor", "coflow3d", "coflow3d_400", "coflow3d_half", "channel3d_250", "coflow3d_200",
                   "coflow3d_quarter", "coflow3d_80")


def main(argv=None):
    ap = argparse.ArgumentParser()
    ap.add_argument("--workload", choices=sorted(WORKLOADS) + ["table"], default="coflow3d",
                    help="table: every workload of the table, in place of what it holds")
    ap.add_argument("--storage", choices=["f32", "f16", "both"], default="both")
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--write", action="store_true", help="record the result in tuning.json")
    args = ap.parse_args(argv)
    sys.path.insert(0, os.path.dirname(HERE))
    from . import cases
    whole = args.workload == "table"
    storages = ["f32", "f16"] if args.storage == "both" else [args.storage]
    table = {k: v for k, v in load_table().items() if not (whole and k.split("-")[1] in storages)}
    for name in TABLE_WORKLOADS if whole else [args.workload]:
        work = WORKLOADS[name](cases)
        members = work if isinstance(work, list) else [work]
        dim, nodes = members[0].dim, sum(c.N for c in members)
        for storage in storages:
            above = table.get(larger_class(dim, storage, nodes))
            res = tune(work, storage, args.steps, args.warmup, prefer=above and int(above["best"]),
                       log=lambda m: print(m, flush=True))
            k = key(dim, storage, nodes)
            print(json.dumps({k: res}), flush=True)
            table[k] = res
    if args.write:
        with open(TABLE, "w") as fh:
            json.dump(table, fh, indent=1, sort_keys=True)


if __name__ == "__main__":
    main()
