"""The SPH deposit and its adjoint on a mesh of small units: cells of 2^-60, so that the
squares of distances below an eighth of a cell are subnormal float32 values.
A power of two changes no rounding of the positions, so the bounds are those of the other
deposit tests: 1e-5 of the larger of the value and the mean per cell, and 1e-4 in
relative L2 norm for the gradients.  (A square's own rounding, 2^-150, moves a weight
by 2e-8 at most.)"""
import numpy as np
import pytest

import oracle
from paper_2609_18316_amd import kdt, workloads
from tests.gpu_util import dev, say, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("exponent", (0, -60))
@pytest.mark.parametrize("n", (400, 70000))
def test_deposit_in_small_units(n, exponent):
    dev()
    cells, cell = 14, 2.0 ** exponent
    rng = np.random.Generator(np.random.PCG64(n))
    x = workloads.uniform(n, 3, n) * np.float32(cells)
    x[: n // 4] = np.floor(x[: n // 4]) + np.float32(0.5)  # near the centres of cells
    x[: n // 4] += rng.uniform(-0.1, 0.1, (n // 4, 3)).astype(np.float32)
    x = (np.minimum(x, np.float32(cells) - np.float32(1e-5)) * np.float32(cell)).astype(np.float32)
    h = (rng.uniform(0.3, 2.5, n) * cell).astype(np.float32)
    m = workloads.masses(n, n + 1)
    shape = (cells,) * 3
    say(f"deposit of {n} with cells of 2^{exponent}")
    xt, mt, ht = to_dev(x), to_dev(m), to_dev(h)
    rho = to_host(kdt.p2m(xt, mt, ht, (0, 0, 0), cell, shape))
    ref = oracle.p2m(x, m, h, (0, 0, 0), cell, shape)
    mean = m.astype(np.float64).sum() / ref.size
    assert (np.abs(rho - ref) <= 1e-5 * np.maximum(np.abs(ref), mean)).all()
    g = rng.standard_normal(shape).astype(np.float32)
    got = [to_host(a) for a in kdt.p2m_backward(xt, mt, ht, (0, 0, 0), cell, shape, to_dev(g))]
    for a, b in zip(got, oracle.p2m_backward(x, m, h, (0, 0, 0), cell, shape, g)):
        assert np.linalg.norm((a - b) * cell) <= 1e-4 * np.linalg.norm(b * cell)
