"""Float64 ball counts and lists around the limits of the wave-shared route: leaves
of 64 points and beyond, 16 dimensions (whose leaves outgrow the LDS first),
trees of one leaf, self rows in input and in tree order -- equal to the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_18316_amd import kdt
from tests.gpu_util import dev, say, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,leaf", [(1, 32), (65, 64), (1000, 2), (1500, 64), (1500, 65),
                                    (1501, 256)])
@pytest.mark.parametrize("d", (2, 3, 4, 8, 16))
def test_balls_f64_by_leaf(n, leaf, d):
    dev()
    rng = np.random.Generator(np.random.PCG64(n + leaf + d))
    x = rng.random((n, d))
    q = rng.random((130, d)) * 1.2 - 0.1
    q[5] = x[0]
    t = kdt.build_f64(torch.from_numpy(x).to(dev()), leaf_size=leaf)
    qt = torch.from_numpy(q).to(dev())
    perm = t.export()["perm"]
    for r in (0.0, 0.15 * d, 0.4 * d, np.inf):
        say(f"f64 balls n={n} leaf={leaf} d={d} r={r}")
        oc, ooff, oidx = oracle.range_brute_f64(x, q, r, lists=True)
        gc, goff, gidx = t.range(qt, r, lists=True)
        np.testing.assert_array_equal(to_host(gc), oc)
        np.testing.assert_array_equal(to_host(goff), ooff)
        np.testing.assert_array_equal(to_host(gidx), oidx)
        own = oracle.range_brute_f64(x, x, r)
        np.testing.assert_array_equal(to_host(t.range(None, r)), own)
        np.testing.assert_array_equal(to_host(t.range(None, r, tree_rows=True)), own[perm])
