"""The instrumented library counts the node boxes and points that a wave reads for one ball in
the counts of small launches (in a process of its own: it cannot share one with the
product library)."""
import json
import subprocess
import sys

import pytest

from tests.gpu_util import dev, say

pytestmark = pytest.mark.gpu

COUNT = """
import json, torch
from paper_2609_18316_amd import kdt, workloads
kdt.load(kdt.LIB_COUNTS_PATH)
x = torch.from_numpy(workloads.uniform(20000, 3, 5)).cuda()
q = torch.from_numpy(workloads.uniform(1000, 3, 6)).cuda()
t = kdt.build(x, leaf_size=16)
out = []
for call in (lambda: t.range(q, 0.0), lambda: t.range(q, 0.05), lambda: t.range(q, 2.0)):
    kdt.visits(reset=True)
    call()
    c = kdt.visits(reset=True)
    out.append((int(c["wave_nodes"]), int(c["wave_points"])))
print(json.dumps(out))
"""


def test_a_ball_per_wave_is_counted():
    dev()
    r = subprocess.run([sys.executable, "-c", COUNT], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    empty, some, everything = json.loads(r.stdout.strip().splitlines()[-1])
    say(f"boxes and points by a wave per ball: {empty} {some} {everything}")
    assert everything == [1000, 0]  # the root's box, held whole
    assert empty[0] > 1000 and some[0] > empty[0]
    assert some[1] > 1000
