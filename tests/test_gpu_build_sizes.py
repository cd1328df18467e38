"""Tree invariants at the sizes where the build's schedule changes: nodes of one
subtree workgroup and one point more, nodes of one chunk and one row more,
chunk counts around the widths of the passes, few and many subtrees."""
import pytest

from paper_2609_18316_amd import kdt
from tests import cases
from tests.gpu_util import dev, say, to_dev
from tests.test_gpu_core import check_tree_invariants

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", (64, 65, 2048, 2049, 4096, 4097, 8193, 65537, 300007))
@pytest.mark.parametrize("d", (2, 3, 8))
@pytest.mark.parametrize("kind", ("uniform", "duplicates"))
def test_build_schedule_sizes(n, d, kind):
    dev()
    leaf = 24 if n < 100_000 else 200
    say(f"build schedule n={n} d={d} {kind} leaf={leaf}")
    x = cases.points(kind, n, d, seed=n + d)
    check_tree_invariants(kdt.build(to_dev(x), leaf_size=leaf), x)


@pytest.mark.parametrize("n", (1_100_003, 2_200_001))
def test_build_many_subtrees(n):
    """More than 512 subtrees in 3-D (four waves each)."""
    dev()
    x = cases.points("normal", n, 3, seed=n)
    check_tree_invariants(kdt.build(to_dev(x), leaf_size=256), x)
