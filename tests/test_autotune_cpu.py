"""The tuning table: how it is looked up, and that the tuner can make it."""
import json
import os

import numpy as np

from paper_2512_12934_amd import autotune


def test_table_is_parsed_once_per_version(tmp_path, monkeypatch):
    """Lookups read the file again only when it has changed, and what
    load_table returns is the caller's to change."""
    path = tmp_path / "tuning.json"
    monkeypatch.setattr(autotune, "TABLE", str(path))
    assert autotune.lookup(2, "f32", 50) == -1
    k = autotune.key(2, "f32", 50)
    path.write_text(json.dumps({k: {"best": 3}}))
    parsed = []
    load = json.load
    monkeypatch.setattr(autotune.json, "load", lambda fh: parsed.append(1) or load(fh))
    assert [autotune.lookup(2, "f32", 50) for _ in range(5)] == [3] * 5
    assert autotune.lookup(2, "f16fixed", 50) == -1 and len(parsed) == 1
    autotune.load_table()[k]["best"] = 7
    assert autotune.lookup(2, "f32", 50) == 3
    path.write_text(json.dumps({k: {"best": 10}}))
    assert autotune.lookup(2, "f32", 50) == 10 and len(parsed) == 2
    os.remove(path)
    assert autotune.lookup(2, "f32", 50) == -1


def test_workloads_of_earlier_calls_are_accepted(monkeypatch):
    """Every workload name the tuner has taken still runs, on the geometry it
    stood for."""
    from paper_2512_12934_amd import cases
    seen = []
    monkeypatch.setattr(autotune, "tune", lambda work, storage, steps, warmup, **kw: seen.append(work) or {"best": 0})
    want = {"tjunction": cases.tjunction(), "coflow3d_quarter": cases.coflow3d_quarter(),
            "tjunction_small": cases.tjunction(W=32, length=256, x_side=48, side_width=32, side_len=32),
            "tjunction_large": cases.sweep_case(512, 0.01, 0.5, 1.0)}
    for name, c in want.items():
        autotune.main(["--workload", name, "--storage", "f32"])
        got = seen.pop()
        assert got.n == c.n and got.nu == c.nu and (got.solid == c.solid).all(), name


def test_table_is_what_the_tuner_makes():
    """Every entry of the committed table belongs to one workload of the
    tuner, holds a time of every configuration, all of them with the bits of
    configuration 0, and its pick is the tuner's rule applied to its times."""
    from paper_2512_12934_amd import cases
    sources = open(os.path.join(autotune.HERE, "csrc", "launch.h")).read()
    n_cfg = {d: sources[sources.index(f"constexpr TileCfg CFG{d}[]"):].split("};")[0].count("\n    {") for d in (2, 3)}
    assert n_cfg[2] >= 12 and n_cfg[3] >= 12
    table = autotune.load_table()
    stood_for = {}
    for name in autotune.TABLE_WORKLOADS:
        work = autotune.WORKLOADS[name](cases)
        members = work if isinstance(work, list) else [work]
        for storage in ("f32", "f16"):
            nodes = sum(c.N for c in members)
            k = autotune.key(members[0].dim, storage, nodes)
            assert k not in stood_for, (name, stood_for[k])
            stood_for[k] = name
            e = table[k]
            times = {int(c): t for c, t in e["ms_per_step"].items()}
            same = {int(c): v for c, v in e["identical"].items()}
            assert sorted(times) == list(range(n_cfg[members[0].dim])) and all(same[c] for c in times), k
            above = table.get(autotune.larger_class(members[0].dim, storage, nodes))
            assert e["best"] == autotune.pick(times, same, above and above["best"]), k
            assert e["fluid_nodes"] == sum(c.fluid_nodes for c in members), k
    assert sorted(stood_for) == sorted(table)


def test_pick():
    """The fastest, unless the larger class's pick is within 2%; never one
    whose state differs."""
    t, ok = {0: 1.0, 1: 0.50, 2: 0.505, 3: 0.4}, {0: True, 1: True, 2: True, 3: False}
    assert autotune.pick(t, ok) == 1
    assert autotune.pick(t, ok, prefer=2) == 2
    assert autotune.pick(t, ok, prefer=0) == 1
    assert autotune.pick(t, ok, prefer=3) == 1


def test_narrow_domains_take_narrow_tiles():
    """A 64-wide pick gives way to the class's fastest tile of at most 32
    columns where the fluid fills 64-wide tiles badly, counted along the axis
    that is contiguous in memory and over all members of a batch; a 2-D domain
    of one such tile across takes the fused one."""
    from paper_2512_12934_amd import cases
    from paper_2512_12934_amd.lbm import tile_config_desc

    def box(shape, walls):
        return cases.random_box(shape, seed=3, dim=2 if shape[2] == 1 else 3, periodic=(not walls,) * 3, walls=walls)

    for shape, walls, ratio in [((97, 8000, 1), True, 4 / 3), ((97, 8000, 1), False, 1.0),
                                ((65, 12000, 1), False, 4 / 3), ((65, 12000, 1), True, 1.0),
                                ((33, 40000, 1), True, 2.0), ((128, 6000, 1), False, 1.0),
                                ((130, 6000, 1), False, 1.2), ((16, 200, 200), True, 2.0),
                                ((70, 90, 90), False, 4 / 3), ((130, 60, 90), False, 1.2),
                                ((200, 60, 60), True, 8 / 7), ((33, 8000, 1), True, 2.0), ((40, 8000, 1), True, 1.0)]:
        c = box(shape, walls)
        assert abs(autotune.lane_ratio([c]) - ratio) < 1e-12, (shape, walls)
        for st in ("f32", "f16", "f16fixed"):
            picked = autotune.lookup(c.dim, st, c.N)
            was = tile_config_desc(c.dim, picked)
            now = tile_config_desc(c.dim, autotune.choose([c], st))
            if ratio < autotune.NARROW:
                assert now == was
            else:
                assert now["tx"] == 32 and (was["tx"] == 64 or now == was or ratio >= autotune.ONE_TILE)
            if c.dim == 2 and ratio >= autotune.ONE_TILE:
                assert now["psrc"] == 0
    assert autotune.lane_ratio([box((20, 30, 1), False).copy(solid=np.ones(600, np.uint8))]) == 1.0
    # a wide member and a narrow one, by the rows of each
    few, many = box((33, 40, 40), True), box((33, 400, 100), True)
    assert autotune.lane_ratio([box((64, 400, 100), False), few]) < autotune.NARROW
    assert autotune.lane_ratio([box((64, 20, 20), False), many]) > autotune.NARROW
    # the caller's x leaves the front where the open faces go last
    c = cases.coflow3d(length=200, width=68, inner=16)
    assert autotune.lane_ratio([c]) < autotune.NARROW <= autotune.lane_ratio([c], "face_last")
