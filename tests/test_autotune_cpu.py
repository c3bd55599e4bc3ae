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
