"""The SPH deposit and its adjoint on both sides of the sizes where the number of
lanes per particle changes, with few tiles (many work items each), particles
on nodes of the mesh, at cell centres (r = 0) and with supports of one cell and
of half the mesh.

The deposit is held to 1e-5 of the larger of the value and the mean per cell.  A
particle whose support only just reaches its cells is ill-conditioned in float32
positions, so the gradients are held per particle to what float32 can give: with
u = 2^-24, the mesh within 1.5 of the origin (images included) and three roundings
on the way (the cell size, the cell's centre, the difference) an offset along an
axis is off by delta = 3 * 1.5 u, the distance by sqrt(3) delta + 2 u r, and q = 2 r / H
by dq = (2 / H) sqrt(3) delta + 4 u q.  |w'| <= 1, so each weight is off by |w'(q)| dq +
1.5 dq^2 + 8 u; each gradient weight, with |w''| and |w' / q| <= 3, by
(2 / H) (6 dq + 8 u).  Over all particles the position gradients agree to 1e-4 in
relative L2 norm."""
import numpy as np
import pytest

import oracle
from paper_2609_18316_amd import kdt, workloads
from tests.gpu_util import dev, say, to_dev, to_host

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


def adjoint_of(x, m, h, cells, g, periodic):
    """One particle's gradients in float64 and their float32 bounds."""
    x = x.astype(np.float64)
    H = max(float(h), float(np.float32(1.0 / cells)))
    span = int(np.ceil(H * cells)) + 1
    ax = [np.arange(int(x[a] * cells) - span, int(x[a] * cells) + span + 1) for a in range(3)]
    if not periodic:
        ax = [i[(i >= 0) & (i < cells)] for i in ax]
    d = np.stack(np.meshgrid(*[x[a] - (ax[a] + 0.5) / cells for a in range(3)], indexing="ij"), -1)
    gc = g[np.ix_(*[i % cells for i in ax])].astype(np.float64)
    r = np.sqrt((d ** 2).sum(-1))
    dq = 2 / H * np.sqrt(3) * 4.5 * U + 4 * U * 2
    q = 2 * r / H
    near = q < 2 + dq
    d, gc, r, q = d[near], gc[near], r[near], np.minimum(q[near], 2.0)
    inner = q < 1
    w = np.where(inner, 1 - 1.5 * q ** 2 + 0.75 * q ** 3, 0.25 * (2 - q) ** 3)
    dw = np.where(inner, -3 * q + 2.25 * q ** 2, -0.75 * (2 - q) ** 2)
    k = (dw / np.maximum(r, 1e-300) * (2 / H))[:, None] * d
    ew = np.abs(dw) * dq + 1.5 * dq ** 2 + 8 * U
    ek = 2 / H * (6 * dq + 8 * U)
    S = w.sum()
    gm = (w * gc).sum() / S
    gx = m / S * ((gc - gm)[:, None] * k).sum(0)
    em = (np.abs(gc - gm) * ew).sum() / (S - ew.sum()) + 2 * U * abs(gm)
    ex = m / (S - ew.sum()) * (np.abs(gc - gm).sum() * ek + em * (np.abs(k).sum(0) + len(q) * ek))
    return gm, gx, em, ex + np.abs(gx) * (ew.sum() / S + 4 * U)


@pytest.mark.parametrize("n,cells", [(1, 8), (7, 20), (300, 17), (65535, 33), (65536, 33),
                                     (1048575, 64), (1048576, 64)])
@pytest.mark.parametrize("periodic", (False, True))
def test_deposit_by_group_size(n, cells, periodic):
    dev()
    rng = np.random.Generator(np.random.PCG64(n))
    x = workloads.uniform(n, 3, n)
    x[: n // 8] = (np.floor(x[: n // 8] * cells) + 0.5) / cells  # cell centres
    x[n // 8: n // 6] = np.floor(x[n // 8: n // 6] * cells) / cells  # mesh nodes
    x = np.minimum(x, np.float32(1) - np.float32(2) ** -24).astype(np.float32)
    m = workloads.masses(n, n + 1)
    # mostly two to three cells, some below one cell, a few of nearly half the mesh
    h = (rng.uniform(0.3, 3.0, n) / cells).astype(np.float32)
    h[: min(n, 20)] = 0.45
    shape, cell = (cells,) * 3, 1.0 / cells
    say(f"deposit groups n={n} cells={cells} periodic={periodic}")
    xt, mt, ht = to_dev(x), to_dev(m), to_dev(h)
    rho = to_host(kdt.p2m(xt, mt, ht, (0, 0, 0), cell, shape, periodic=periodic))
    ref = oracle.p2m(x, m, h, (0, 0, 0), cell, shape, periodic=periodic)
    mean = m.astype(np.float64).sum() / ref.size
    assert (np.abs(rho - ref) <= 1e-5 * np.maximum(np.abs(ref), mean)).all()
    g = rng.standard_normal(shape).astype(np.float32)
    gm, gx = (to_host(a) for a in kdt.p2m_backward(xt, mt, ht, (0, 0, 0), cell, shape, to_dev(g),
                                                   periodic=periodic))
    assert np.isfinite(gm).all()
    ref = oracle.p2m_backward(x, m, h, (0, 0, 0), cell, shape, g, periodic=periodic)[1]
    assert np.linalg.norm(gx - ref) <= 1e-4 * np.linalg.norm(ref)
    some = np.unique(np.concatenate([np.arange(min(n, 40)), rng.integers(0, n, 400),
                                     rng.integers(n // 8, max(n // 6, 1), 200), [n - 1]]))
    for i in some:
        om, ox, em, ex = adjoint_of(x[i], float(m[i]), h[i], cells, g, periodic)
        assert abs(gm[i] - om) <= em, i
        assert (np.abs(gx[i] - ox) <= ex).all(), i
