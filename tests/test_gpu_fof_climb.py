"""GPU parity of friends-of-friends where the wave-shared search starts and climbs:
point counts around the 64 points of a wave, trees of one leaf, every leaf size up
to the wave's 64 points and one beyond, open and periodic -- labels equal to
the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2609_18316_amd import kdt, workloads
from tests import cases
from tests.gpu_util import dev, say, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", (1, 63, 64, 65, 129, 1000, 4097))
@pytest.mark.parametrize("leaf", (2, 9, 32, 64, 65))
@pytest.mark.parametrize("kind", ("uniform", "clustered", "identical"))
def test_fof_climb_matches_oracle(n, leaf, kind):
    dev()
    x = workloads.clustered(n, n) if kind == "clustered" else cases.points(kind, n, 3, seed=n)
    t = kdt.build(to_dev(x), leaf_size=leaf)
    for b in (0.0, 0.2, 0.7, 3.0):
        l = float(np.float32(b * n ** (-1.0 / 3.0)))
        say(f"fof climb n={n} leaf={leaf} {kind} b={b}")
        np.testing.assert_array_equal(to_host(t.fof(l)), oracle.fof_brute(x, l))
        np.testing.assert_array_equal(to_host(t.fof(l, period=1.0)),
                                      oracle.fof_brute(x, l, period=1.0))
