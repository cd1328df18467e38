"""Float64 ball counts of queries in input order, around the number of queries and the size
of the tree from which waves of queries that lie apart are answered one query per lane:
the counts are the oracle's for queries in order, in none, partly in order, at one point and
not finite; and the wave-shared traversal leaves out the waves that lie apart, no others
(counted by the instrumented library in a process of its own)."""
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
import json, torch
from paper_2609_18316_amd import kdt, workloads
kdt.load(kdt.LIB_COUNTS_PATH)
x = torch.from_numpy(workloads.uniform(20000, 3, 5)).cuda()
q = torch.from_numpy(workloads.uniform(1 << 17, 3, 6)).cuda()  # whole waves
order = kdt.build(x, leaf_size=16).query_order(q)
t = kdt.build_f64(x.double(), leaf_size=16)
mixed = q[order.long()].double()
mixed[1 << 16:] = q[1 << 16:].double()
out = []
for queries, given in ((q.double(), order), (q[order.long()].double().contiguous(), None),
                       (mixed, None), (q.double(), None)):
    kdt.visits(reset=True)
    t.range(queries, 0.05, sort_queries=False, order=given)
    out.append(int(kdt.visits(reset=True)["wave_nodes"]))
print(json.dumps(out))
"""


@pytest.mark.parametrize("d,n", [(2, (1 << 13) - 1), (2, 1 << 13), (3, 9000), (4, 1 << 13),
                                 (8, 1 << 13)])
def test_counts_in_input_order(d, n):
    dev()
    x = workloads.uniform(n, d, 5).astype(np.float64)
    q = workloads.uniform((1 << 15) + 1, d, 6).astype(np.float64)
    r = 0.6 * (20 / n) ** (1 / d)
    t = kdt.build_f64(to_dev(x), leaf_size=16)
    some = np.concatenate([np.arange(0, len(q), 331), [40, 41, len(q) - 1]])
    for kind in ("none", "ordered", "partly", "one point", "not finite"):
        p = q.copy()
        if kind in ("ordered", "partly"):
            p = p[np.lexsort((p[:, 0], np.floor(p[:, 1] * 200)))]
        if kind == "partly":
            p[5000:9000] = q[5000:9000]
        if kind == "one point":
            p[:] = x[0]
        if kind == "not finite":
            p[40] = np.nan
            p[41, 0] = np.inf
        for nq in (1 << 15, (1 << 15) + 1):
            say(f"float64 counts in input order d={d} n={n} nq={nq} {kind}")
            got = to_host(t.range(to_dev(p[:nq]), r, sort_queries=False))
            row = some[some < nq]
            finite = np.isfinite(p[row]).all(axis=1)
            np.testing.assert_array_equal(got[row[finite]],
                                          oracle.range_brute_f64(x, p[row[finite]], r))
            assert (got[row[~finite]] == 0).all()
            np.testing.assert_array_equal(got, to_host(t.range(to_dev(p[:nq]), r)))
    t.close()


def test_waves_that_lie_apart_are_left_out():
    dev()
    r = subprocess.run([sys.executable, "-c", COUNT], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    given, ordered, mixed, none = json.loads(r.stdout.strip().splitlines()[-1])
    say(f"nodes visited by waves: {given}, {ordered} in order, {mixed} half in order, {none} in none")
    assert ordered == given and 0 < mixed < given and none == 0
