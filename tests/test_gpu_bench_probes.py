"""bench.py's row-gather probe at the smallest workload, whose update is one launch (no fixup)."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_row_gather_probe_without_a_fixup_launch():
    r = subprocess.run(
        [sys.executable, os.path.join(ROOT, "bench.py"), "--config", "1", "--steps", "20",
         "--warmup", "10", "--no-cpu-baseline", "--no-extra-configs", "--no-ceilings",
         "--row-gather-probe"], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    probe = json.loads(r.stdout.strip().splitlines()[-1])["row_gather_probe"]
    for n in (0, 8, 32):
        rec = probe["head_rows_removed_%d" % n]
        assert rec["apply_us"] > 0 and rec["fixup_us"] == 0
