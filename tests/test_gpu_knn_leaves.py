"""Per-lane kNN over leaves of every size that one tree can have, in the dimensions whose
lists insert, and around the size of the tree from which 4-dimensional lists of 32 do --
bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2609_18316_amd import kdt
from tests import cases
from tests.gpu_util import dev, say, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,leaf", [(3, 2), (127, 4), (1000, 16), (1023, 33), (2047, 64), (900, 200)])
@pytest.mark.parametrize("d", (4, 8))
def test_leaves_of_two_sizes(n, leaf, d):
    dev()
    x = cases.points("uniform", n, d, seed=n + leaf)
    q = np.concatenate([x[: min(n, 100)], cases.points("normal", 100, d, seed=n)])
    t, ot = kdt.build(to_dev(x), leaf_size=leaf), oracle.Tree(x, leaf)
    for k in (1, 8, 16, 32, 33, 64):
        say(f"kNN by leaves n={n} leaf={leaf} d={d} k={k}")
        oi, od = ot.knn(q, k)
        idx, d2 = t.knn(to_dev(q), k, traversal=1)
        np.testing.assert_array_equal(to_host(idx), oi)
        np.testing.assert_array_equal(to_host(d2), od)


@pytest.mark.parametrize("n", ((1 << 18) - 1, 1 << 18))
@pytest.mark.parametrize("leaf", (16, 17, 32, 64))
def test_four_dimensions_by_tree(n, leaf):
    dev()
    x = cases.points("uniform", n, 4, seed=leaf)
    x[1000:1400] = x[7]  # equal distances
    q = np.concatenate([x[:200], cases.points("uniform", 200, 4, seed=n)])
    t, ot = kdt.build(to_dev(x), leaf_size=leaf), oracle.Tree(x, leaf)
    for k in (17, 32):
        say(f"kNN d=4 n={n} leaf={leaf} k={k}")
        oi, od = ot.knn(q, k)
        for sort in (True, False):
            idx, d2 = t.knn(to_dev(q), k, traversal=1, sort_queries=sort)
            np.testing.assert_array_equal(to_host(idx), oi)
            np.testing.assert_array_equal(to_host(d2), od)
