"""GPU parity of the per-lane kNN where its batches, leaves and votes can go
wrong: trees around the batch of 16 points, leaves that are not a multiple of it,
list lengths around 32, ties, and distances that overflow float32 -- bit-exact
against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2609_18316_amd import kdt
from tests import cases
from tests.gpu_util import dev, say, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,leaf", [(1, 32), (15, 32), (16, 32), (17, 32), (31, 2), (33, 16),
                                    (500, 9), (777, 17), (1000, 20), (1003, 25), (2049, 64),
                                    (3001, 200)])
@pytest.mark.parametrize("d", (2, 3, 4))
@pytest.mark.parametrize("kind", ("uniform", "duplicates"))
def test_lane_knn_matches_oracle(n, leaf, d, kind):
    dev()
    x = cases.points(kind, n, d, seed=n + leaf)
    q = np.concatenate([x[: min(n, 100)], 3.0 * cases.points("normal", 157, d, seed=n)])
    q[-1] = 3e38  # squared distances overflow to +inf
    t, ot = kdt.build(to_dev(x), leaf_size=leaf), oracle.Tree(x, leaf)
    for k in (1, 16, 17, 24, 32, 33):
        say(f"lane kNN n={n} leaf={leaf} d={d} {kind} k={k}")
        oi, od = ot.knn(q, k)
        for sort in (True, False):
            idx, d2 = t.knn(to_dev(q), k, traversal=1, sort_queries=sort)
            np.testing.assert_array_equal(to_host(idx), oi)
            np.testing.assert_array_equal(to_host(d2), od)
        kth = to_host(t.knn(to_dev(q), k, traversal=1, kth_only=1))
        np.testing.assert_array_equal(kth, od[:, k - 1])
        self_d2 = to_host(t.knn(None, k, traversal=1, kth_only=1))
        np.testing.assert_array_equal(self_d2, ot.knn(x, k)[1][:, k - 1])


@pytest.mark.parametrize("n,leaf", [(1, 8), (15, 16), (16, 16), (500, 9), (1000, 20)])
def test_lane_knn_torus_matches_oracle(n, leaf):
    dev()
    x = cases.points("uniform", n, 3, seed=n)
    q = cases.points("uniform", 200, 3, seed=n + 1)
    t = kdt.build(to_dev(x), leaf_size=leaf)
    for k in (17, 32):
        say(f"lane kNN torus n={n} leaf={leaf} k={k}")
        oi, od = oracle.knn_brute(x, q, k, period=1.0)
        idx, d2 = t.knn(to_dev(q), k, period=1.0)
        np.testing.assert_array_equal(to_host(idx), oi)
        np.testing.assert_array_equal(to_host(d2), od)
        kth = to_host(t.knn(to_dev(q), k, period=1.0, kth_only=1))
        np.testing.assert_array_equal(kth, od[:, k - 1])


def test_lane_knn_nan_queries_find_nothing():
    """A NaN coordinate (of either sign) is at no distance from any point."""
    dev()
    x = cases.points("uniform", 1000, 3, seed=5)
    q = cases.points("uniform", 70, 3, seed=6)
    q[3] = np.nan
    q[64, 1] = -np.nan
    good = ~np.isnan(q).any(axis=1)
    t, ot = kdt.build(to_dev(x), leaf_size=16), oracle.Tree(x, 16)
    for k in (8, 32, 64):
        oi, od = ot.knn(q[good], k)
        idx, d2 = (to_host(a) for a in t.knn(to_dev(q), k, traversal=1))
        np.testing.assert_array_equal(idx[good], oi)
        np.testing.assert_array_equal(d2[good], od)
        assert (idx[~good] == -1).all() and np.isinf(d2[~good]).all()
        kth = to_host(t.knn(to_dev(q), k, traversal=1, kth_only=1))
        np.testing.assert_array_equal(kth[good], od[:, k - 1])
        assert np.isinf(kth[~good]).all()
