"""The bench's command line on the CPU: more than one GPU is refused with a
message and exit status 2, before anything touches a device."""
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 2
    msg = json.loads(r.stdout.strip().splitlines()[-1])
    assert "one GPU" in msg["error"]


def test_the_result_is_one_short_line(capsys):
    """Whatever the sections hold, stdout is one JSON line that a log's last 8000 characters
    keep whole; the sections' details are on stderr."""
    sys.path.insert(0, ROOT)
    import bench
    head = {"metric": bench.METRIC, "value": 1.0, "ms_per_step": 0.25, "hbm_frac": 0.17, "n_gpus": 1}
    long = {"densities": {str(k): {"hbm_frac": 0.5, "rows": list(range(2000))} for k in range(5)}}
    bench.print_result(dict(head), [("batched", lambda: {"batched_ms": 2.0, "rows": list(range(5000))}), ("c2", lambda: long)])
    out, err = capsys.readouterr()
    assert len(out.splitlines()) == 1 and len(out) < 4000
    line = json.loads(out)
    assert {k: line[k] for k in head} == head
    assert line["summary"]["c1_ms_per_iter"] == 0.25 and line["summary"]["c3_batched_ms"] == 2.0
    assert line["summary"]["c2_hbm_frac"] == {str(k): 0.5 for k in range(5)}
    assert [list(json.loads(x)) for x in err.splitlines()] == [["batched"], ["c2"]]
