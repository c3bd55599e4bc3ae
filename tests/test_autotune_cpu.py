"""The tuning table: how it is looked up, and that the tuner can make it."""
import json
import os

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
