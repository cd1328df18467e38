"""Ball counts and lists whose traversals are handed on: budgets on both sides of the
largest one that is walked widest first, launches on both sides of the wave
count where the default budget changes, trees of one leaf and of two, balls that hold
everything, nothing or the surface of a dense cluster, float32 and float64 -- equal
to the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_18316_amd import kdt
from tests.gpu_util import dev, say, to_dev, to_host

pytestmark = pytest.mark.gpu


def cluster(n, nq, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    x = (0.5 + 0.01 * rng.standard_normal((n, 3))).astype(np.float32)
    q = (0.5 + 0.03 * (rng.random((nq, 3)) - 0.5)).astype(np.float32)
    q[: nq // 16] = 9.0  # far from every point
    return x, q


@pytest.mark.parametrize("n,leaf", [(5, 8), (9, 8), (40000, 8), (40000, 64)])
@pytest.mark.parametrize("budget", (0, 1, 2, 23, 24, 25, 64))
def test_handed_on_by_budget(n, leaf, budget):
    dev()
    x, q = cluster(n, 700, n + leaf)
    t, ot = kdt.build(to_dev(x), leaf_size=leaf), oracle.Tree(x, leaf)
    t64 = kdt.build_f64(torch.from_numpy(x.astype(np.float64)).to(dev()), leaf_size=leaf)
    q64 = torch.from_numpy(q.astype(np.float64)).to(dev())
    for r in (0.003, 0.02, 0.5):
        say(f"handed on n={n} leaf={leaf} budget={budget} r={r}")
        oc, ooff, olst = ot.range(q, r, lists=True)
        c, off, lst = t.range(to_dev(q), r, lists=True, traversal=2, split_budget=budget)
        np.testing.assert_array_equal(to_host(c), oc)
        np.testing.assert_array_equal(to_host(off), ooff)
        np.testing.assert_array_equal(to_host(lst), olst)
        if budget == 0:
            oc = oracle.range_brute_f64(x.astype(np.float64), q.astype(np.float64), r)
            np.testing.assert_array_equal(to_host(t64.range(q64, r)), oc)


@pytest.mark.parametrize("nq", (131072, 131073))
def test_handed_on_by_launch_size(nq):
    dev()
    x, q = cluster(60000, nq, nq)
    t, ot = kdt.build(to_dev(x), leaf_size=16), oracle.Tree(x, 16)
    say(f"handed on nq={nq}")
    np.testing.assert_array_equal(to_host(t.range(to_dev(q), 0.004)), ot.range(q, 0.004))
