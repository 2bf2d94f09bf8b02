"""The benchmark's last line is the headline: JSON with the contract's keys, and short whatever the
other workloads report (readers keep the last few thousand characters)."""
import json

import bench


def test_headline_is_the_last_line(capsys):
    result = {"metric": "m", "value": 1.0, "unit": "u", "n_gpus": 1, "config": {"workload": "w"}}
    legs = {"one": {"rows": list(range(3000))}, "two": {"ms": 2.0}}
    bench.emit(result, legs)
    lines = capsys.readouterr().out.splitlines()
    last = json.loads(lines[-1])
    assert last["metric"] == "m" and last["value"] == 1.0 and last["legs"] == ["one", "two"]
    assert len(lines[-1]) < 500
    assert [line.split(":")[0] for line in lines[:-1]] == ["leg one", "leg two"]
    assert json.loads(lines[0].split(": ", 1)[1]) == legs["one"]
