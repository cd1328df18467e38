"""Float64 kNN where distances are equal once rounded to float32, or exactly:
trees around the batch of 16 points, k around the list of 32, and points that
float32 cannot tell apart -- equal to the oracle, order included."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_18316_amd import kdt
from tests.gpu_util import dev, say, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ("uniform", "lattice", "close", "mixed"))
@pytest.mark.parametrize("n", (15, 16, 17, 40, 3000))
def test_knn_f64_ties(kind, n):
    dev()
    rng = np.random.Generator(np.random.PCG64(n))
    x = rng.random((n, 3))
    if kind in ("lattice", "mixed"):
        x = np.round(x * 8) / 8
    if kind == "close":  # distances that differ by parts in 10^10
        x = np.round(x * 4) / 4 + rng.random((n, 3)) * 1e-10
    if kind == "mixed":  # half of them moved off the lattice, below float32's resolution
        x[::2] += rng.random((len(x[::2]), 3)) * 1e-12
    q = np.concatenate([x[: min(n, 60)], np.round(rng.random((70, 3)) * 8) / 8])
    t = kdt.build_f64(torch.from_numpy(x).to(dev()), leaf_size=9)
    for k in (1, 8, 16, 17, 31, 32, 33):
        say(f"f64 ties {kind} n={n} k={k}")
        oi, od = oracle.knn_brute_f64(x, q, k)
        gi, gd = t.knn(torch.from_numpy(q).to(dev()), k)
        np.testing.assert_array_equal(to_host(gd), od)
        np.testing.assert_array_equal(to_host(gi), oi)
