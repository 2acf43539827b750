"""The line bench.py prints holds the contract's keys and is short enough to survive where
only the end of a run's output is kept; the whole record goes to a file."""
import json
import os

import pytest

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("name", ["bench_turb256", "bench_dns840", "bench_channel256", "bench_channel_dns", "bench_channel_vk"])
def test_line_of_a_recorded_run(name, tmp_path, capsys):
    record = json.load(open(os.path.join(ROOT, "profiles", name + ".json")))
    path = tmp_path / "record.json"
    bench.report(record, str(path))
    out = capsys.readouterr().out
    assert out.count("\n") == 1 and len(out) < 2000
    line = json.loads(out)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
              "vs_baseline", "dtype", "data", "config"):
        assert line[k] == record[k]
    assert line["mcell_per_s"] == {m: r["mcell_per_s"] for m, r in record["modes"].items()}
    assert json.load(open(path)) == record
