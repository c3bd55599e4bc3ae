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
