"""Float64 kNN at scales whose squared distances leave float32's range on either side:
the rows are the oracle's, and a search is as long as in the unit box.  A power of two
scales every float64 operation exactly, so the boxes and points that the instrumented library
counts have to be the same to the last one (counted in a process of its own: it
cannot share one with the product library)."""
import json
import subprocess
import sys

import numpy as np
import pytest

import oracle
from paper_2609_18316_amd import kdt, workloads
from tests.gpu_util import dev, say, to_dev, to_host

pytestmark = pytest.mark.gpu

COUNT = """
import json, numpy as np, torch
from paper_2609_18316_amd import kdt, workloads
kdt.load(kdt.LIB_COUNTS_PATH)
x = torch.from_numpy(workloads.uniform(20000, {d}, 5)).double().cuda()
q = torch.from_numpy(workloads.uniform(1000, {d}, 6)).double().cuda()
out = []
for e in (0, 75, -90):
    s = 2.0 ** e
    t = kdt.build_f64(x * s, leaf_size=16)
    for k in (8, 32):
        kdt.visits(reset=True)
        t.knn((q * s).contiguous(), k)
        c = kdt.visits(reset=True)
        out.append((e, k, int(c["lane_nodes"]), int(c["lane_points"])))
print(json.dumps(out))
"""


@pytest.mark.parametrize("scale", (1e22, 1e-26, 1e150, 1e-150))
@pytest.mark.parametrize("d", (2, 3, 8))
def test_rows_at_any_scale(d, scale):
    dev()
    x = workloads.uniform(4000, d, 5).astype(np.float64) * scale
    q = np.concatenate([workloads.uniform(300, d, 6).astype(np.float64) * scale, x[:100]])
    t = kdt.build_f64(to_dev(x), leaf_size=16)
    for k in (1, 8, 32, 64):
        say(f"float64 kNN d={d} scale={scale} k={k}")
        oi, od = oracle.knn_brute_f64(x, q, k)
        gi, gd = t.knn(to_dev(q), k)
        np.testing.assert_array_equal(to_host(gi), oi)
        np.testing.assert_array_equal(to_host(gd), od)
    t.close()


@pytest.mark.parametrize("d", (2, 3))
def test_a_search_is_as_long_at_any_scale(d):
    dev()
    r = subprocess.run([sys.executable, "-c", COUNT.format(d=d)], capture_output=True, text=True,
                       timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    rows = json.loads(r.stdout.strip().splitlines()[-1])
    say(f"visits d={d}: {rows}")
    for e, k, nodes, points in rows:
        assert nodes > 0 and points > 0
        assert [nodes, points] == next([a, b] for e0, k0, a, b in rows if (e0, k0) == (0, k)), e
