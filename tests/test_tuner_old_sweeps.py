"""Saved tuner sweeps of other tile configurations are refused, not half used."""

import json

import pytest

from paper_1511_07658_amd import tune


def test_a_sweep_of_other_configurations_is_refused(tmp_path, monkeypatch):
    old, both = "256x128x32R3", "128x128x32R2P"   # one that is gone, and a name that is still there
    assert old not in tune.CONFIG_NAMES and both in tune.CONFIG_NAMES
    sweep = {"1024": {"best": 23, "us": {old: 120.0, both: 134.0}}}
    with pytest.raises(ValueError, match=old):
        tune.merge_sweeps([sweep])
    # from the command line: nothing is written
    saved = tmp_path / "old.json"
    saved.write_text(json.dumps(sweep))
    monkeypatch.setattr(tune, "write_table", lambda *a, **k: pytest.fail("a table was written"))
    with pytest.raises(ValueError):
        tune.main(["--from-json", str(saved)])
