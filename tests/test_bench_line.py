"""bench.py's one line on stdout: the contract's keys, without the secondary
measurements, which go to stderr a line each."""
import json
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_secondary_measurements_stay_out_of_the_line(capsys):
    sys.path.insert(0, ROOT)
    import bench
    line = {"metric": "m", "value": 1.0, "config": {"code": "toric2d:32"}}
    extras = {f"leg{k}": {"rows": list(range(1500))} for k in range(4)}
    bench.emit(line, extras)
    out, err = capsys.readouterr()
    assert out.count("\n") == 1 and json.loads(out) == line
    rows = [json.loads(x[len("[bench] "):]) for x in err.strip().split("\n")]
    assert rows == [{k: v} for k, v in extras.items()]
    bench.emit(dict(line, long="x" * bench.LINE_LIMIT), {})  # printed all the same, with a word about it
    out, err = capsys.readouterr()
    assert json.loads(out)["value"] == 1.0 and "characters" in err


def test_the_line_holds_the_contract_and_no_extras():
    src = open(os.path.join(ROOT, "bench.py")).read()
    body = src[src.index('    line = {\n        "metric"'):src.index("    emit(line, extras)")]
    keys = re.findall(r'^        "([a-z0-9_]+)":', body, re.M)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
              "vs_baseline", "dtype", "data", "config", "roofline", "cpu_baseline"):
        assert k in keys, k
    assert "extras" not in keys
