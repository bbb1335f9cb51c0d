"""bench.py's memory-optimised workload prints its line, with a time for every GEMM launch of a step."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_line():
    r = subprocess.run([sys.executable, "bench.py", "--workload", "memopt", "--config", "3", "--steps", "2", "--warmup", "1", "--no-cpu-baseline"],
                       cwd=ROOT, capture_output=True, text=True, timeout=110)
    assert r.returncode == 0, r.stderr[-2000:]
    launches = json.loads(r.stdout.strip().splitlines()[-1])["roofline"]["launches"]
    assert len(launches) == 8 and all(v["ms"] > 0 for v in launches.values())
    assert sum(len(v["MxNxK"]) for v in launches.values()) == 12
