"""kNN with k above the register lists where a wave searches one ball: leaves below, at and
above the width of a leaf scan (and beyond a wave), trees of one leaf, runs of whole
nodes, duplicated points, balls that hold everything, 2 to 16 dimensions, the torus, and
launches on both sides of the number of balls that are counted by a wave each --
equal to the oracle."""
import numpy as np
import pytest

import oracle
from paper_2609_18316_amd import kdt
from tests.gpu_util import dev, say, to_dev, to_host

pytestmark = pytest.mark.gpu


def points(n, d, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    x = rng.random((n, d))
    x[: n // 3] = 0.4 + 0.01 * rng.random((n // 3, d))  # a dense clump
    x[n // 3: n // 3 + n // 8] = x[0]  # many duplicates
    return x.astype(np.float32), rng.random((90, d)).astype(np.float32)


@pytest.mark.parametrize("leaf", (2, 5, 16, 64, 65, 256))
@pytest.mark.parametrize("d", (2, 3, 4, 8, 16))
def test_large_k_by_leaf(d, leaf):
    dev()
    for n, k in ((70, 65), (70, 70), (3000, 65), (3000, 700), (3000, 2999)):
        x, q = points(n, d, n + k + d)
        t = kdt.build(to_dev(x), leaf_size=leaf)
        say(f"wave balls d={d} leaf={leaf} n={n} k={k}")
        idx, d2 = t.knn(to_dev(q), k)
        oi, od = oracle.knn_brute(x, q, k)
        np.testing.assert_array_equal(to_host(idx), oi)
        np.testing.assert_array_equal(to_host(d2), od)


@pytest.mark.parametrize("leaf", (8, 64, 100))
@pytest.mark.parametrize("k", (65, 500, 3000))
def test_large_k_torus(leaf, k):
    dev()
    x, q = points(5000, 3, k)
    t = kdt.build(to_dev(x), leaf_size=leaf)
    say(f"wave balls torus leaf={leaf} k={k}")
    idx, d2 = t.knn(to_dev(q), k, period=1.0)
    oi, od = oracle.knn_brute(x, q, k, period=1.0)
    np.testing.assert_array_equal(to_host(idx), oi)
    np.testing.assert_array_equal(to_host(d2), od)


@pytest.mark.parametrize("nq", (1 << 18, (1 << 18) + 1))
def test_large_k_by_launch_size(nq):
    dev()
    rng = np.random.Generator(np.random.PCG64(nq))
    x, _ = points(9000, 3, 1)
    q = rng.random((nq, 3)).astype(np.float32)
    t = kdt.build(to_dev(x), leaf_size=8)
    say(f"wave balls nq={nq}")
    idx, d2 = (to_host(a) for a in t.knn(to_dev(q), 65))
    some = np.concatenate([[0, nq - 1], rng.integers(0, nq, 400)])
    oi, od = oracle.knn_brute(x, q[some], 65)
    np.testing.assert_array_equal(idx[some], oi)
    np.testing.assert_array_equal(d2[some], od)


@pytest.mark.parametrize("leaf", (2, 16, 64))
@pytest.mark.parametrize("d", (2, 3, 4, 8, 16))
def test_counts_by_wave(d, leaf):
    dev()
    for n in (1, 3, 70, 3000):
        x, q = points(n, d, n + d)
        t = kdt.build(to_dev(x), leaf_size=leaf)
        ot = oracle.Tree(x, leaf)
        for r in (0.0, 0.1, 0.5, 5.0):
            say(f"wave counts d={d} leaf={leaf} n={n} r={r}")
            oc = ot.range(q, r)
            np.testing.assert_array_equal(to_host(t.range(to_dev(q), r)), oc)
            np.testing.assert_array_equal(to_host(t.range(to_dev(q), r, split_budget=7)), oc)
            np.testing.assert_array_equal(to_host(t.range(None, r)), ot.range(x, r))


@pytest.mark.parametrize("nq", (1 << 17, (1 << 17) + 1))
def test_counts_by_launch_size(nq):
    dev()
    x, _ = points(20000, 3, 1)
    q = np.random.Generator(np.random.PCG64(nq)).random((nq, 3)).astype(np.float32)
    t, ot = kdt.build(to_dev(x), leaf_size=16), oracle.Tree(x, 16)
    say(f"wave counts nq={nq}")
    np.testing.assert_array_equal(to_host(t.range(to_dev(q), 0.03)), ot.range(q, 0.03))
