"""GPU parity of friends-of-friends in every dimension: nodes tested two at a time up to
8 dimensions and one at a time in 16, leaves of every size up to the wave's 64 points and
beyond, open and periodic -- labels equal to the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2609_18316_amd import kdt
from tests import cases
from tests.gpu_util import dev, say, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", (1, 65, 700, 2500))
@pytest.mark.parametrize("leaf", (2, 17, 32, 64, 100))
@pytest.mark.parametrize("d", (2, 4, 8, 16))
def test_fof_by_dimension(n, leaf, d):
    dev()
    x = cases.points("uniform", n, d, seed=n)
    x[n // 2: n // 2 + n // 8] = x[0]  # a clique
    t = kdt.build(to_dev(x), leaf_size=leaf)
    for b in (0.0, 0.3, 0.8):
        l = float(np.float32(b * n ** (-1.0 / d)))
        say(f"fof n={n} leaf={leaf} d={d} b={b}")
        np.testing.assert_array_equal(to_host(t.fof(l)), oracle.fof_brute(x, l))
        np.testing.assert_array_equal(to_host(t.fof(l, period=1.0)),
                                      oracle.fof_brute(x, l, period=1.0))
