"""Deposits on both sides of the sizes where the first pass changes its lanes and where the
work items of a tile change: around 2^13 particles with supports, and meshes of few and of
many tiles with one that holds most particles (ordered and not, single items and split ones) --
against the float64 oracle.  Dense meshes are held to the deposit's tolerance, 1e-5 of the
larger of the value and the mean per cell.  With about one particle per cell and supports that
only just reach it, one ulp of the positions alone moves a cell by 6e-5, so there each
particle's weights w are held to what float32 can give, m (ew / S + w sum(ew) / S^2), with the
errors ew of the weights as the adjoint's test derives them (U = 2^-24; offsets off by
4.5 U along an axis)."""
import numpy as np
import pytest

import oracle
from paper_2609_18316_amd import kdt, workloads
from tests.gpu_util import dev, say, to_dev, to_host

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


def weight_bound(x, m, h, cells, periodic):
    """Per cell, what the float32 errors of every particle's weights can add up to."""
    out = np.zeros((cells,) * 3)
    for p, mp, hp in zip(x.astype(np.float64), m.astype(np.float64), h):
        H = max(float(hp), float(np.float32(1.0 / cells)))
        span = int(np.ceil(H * cells)) + 1
        ax = [np.arange(int(p[a] * cells) - span, int(p[a] * cells) + span + 1) for a in range(3)]
        if not periodic:
            ax = [i[(i >= 0) & (i < cells)] for i in ax]
        r2 = sum(np.meshgrid(*[(p[a] - (ax[a] + 0.5) / cells) ** 2 for a in range(3)],
                             indexing="ij", sparse=True))
        q = 2 / H * np.sqrt(r2)
        dq = 2 / H * np.sqrt(3) * 4.5 * U + 4 * U * 2
        near = q < 2 + dq
        q = np.minimum(q, 2.0)
        w = np.where(q < 1, 1 - 1.5 * q ** 2 + 0.75 * q ** 3, 0.25 * (2 - q) ** 3)
        dw = np.where(q < 1, 3 * q - 2.25 * q ** 2, 0.75 * (2 - q) ** 2)
        ew = np.where(near, dw * dq + 1.5 * dq ** 2 + 8 * U, 0.0)
        S, e = w.sum(), ew.sum()
        low = max(S - e, 1e-300)
        np.add.at(out, np.ix_(*[i % cells for i in ax]), mp * (ew / low + w * e / (S * low)))
    return out


@pytest.mark.parametrize("n", (1 << 13, (1 << 13) + 1))
@pytest.mark.parametrize("cells,periodic", [(20, False), (40, True)])
def test_supports_by_particles(n, cells, periodic):
    dev()
    rng = np.random.Generator(np.random.PCG64(n))
    x = workloads.uniform(n, 3, n)
    m = workloads.masses(n, n + 1)
    h = (rng.uniform(0.3, 3.0, n) / cells).astype(np.float32)
    h[:20] = 0.45
    say(f"supports n={n} cells={cells} periodic={periodic}")
    g = to_host(kdt.p2m(to_dev(x), to_dev(m), to_dev(h), (0, 0, 0), 1 / cells, (cells,) * 3,
                        periodic=periodic)).astype(np.float64)
    o = oracle.p2m(x, m, h, (0, 0, 0), 1 / cells, (cells,) * 3, periodic=periodic)
    bound = weight_bound(x, m, h, cells, periodic) + 2 * U * np.abs(o)
    assert (np.abs(g - o) <= bound).all()
    # and the bound is not loose: a thousandth of the mean at its median
    assert np.median(bound) <= 1e-3 * m.astype(np.float64).sum() / o.size
    assert abs(g.sum() - m.astype(np.float64).sum()) <= 1e-5 * m.astype(np.float64).sum()


@pytest.mark.parametrize("scheme", ("ngp", "cic", "tsc", "sph"))
@pytest.mark.parametrize("cells", (16, 32, 128))
@pytest.mark.parametrize("dense", (16383, 16384, 80000))
def test_one_tile_of_most(scheme, cells, dense):
    dev()
    sph = scheme == "sph"
    if sph and dense > 16384:
        pytest.skip("the bound is a loop over the particles")
    n = dense + 3000
    x = workloads.uniform(n, 3, dense)
    x[:dense] *= np.float32(8 / cells)  # inside the first tile
    m = workloads.masses(n, cells)
    t = kdt.build(to_dev(x))
    h = np.full(n, 1.5 / cells, np.float32) if sph else None
    mt, ht = t.gather(to_dev(m)), to_dev(h) if sph else None
    lo, shape, total = (0, 0, 0), (cells,) * 3, m.astype(np.float64).sum()
    say(f"one tile of most {scheme} cells={cells} dense={dense}")
    if sph:
        o = oracle.p2m(x, m, h, lo, 1 / cells, shape)
        own = kdt.p2m(to_dev(x), to_dev(m), ht, lo, 1 / cells, shape)
        bound = weight_bound(x, m, h, cells, False) + 2 * U * np.abs(o)
    else:
        o = oracle.p2m_cloud(x, m, lo, 1 / cells, shape, scheme)
        own = kdt.p2m_cloud(to_dev(x), to_dev(m), lo, 1 / cells, shape, scheme)
        bound = 1e-5 * np.maximum(np.abs(o), total / o.size)
    tree = kdt.p2m_tree(t, mt, ht, lo, 1 / cells, shape, scheme=scheme)
    for g in (own, tree):
        g = to_host(g).astype(np.float64)
        assert (np.abs(g - o) <= bound).all()
        assert abs(g.sum() - total) <= 1e-5 * total
    t.close()
