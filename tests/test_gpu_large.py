"""More elements than one launch of 256 threads each holds (GPU)."""
import numpy as np
import pytest

import workloads
from paper_2012_13487_amd import binding

pytestmark = pytest.mark.gpu


def test_moments_of_more_than_two_to_the_24_elements():
    """4097 x 4096 elements, p = 1, 9 velocities, FP32 storage (604 million
    values): the moments of an equilibrium state are the fields it was made of,
    but for the rounding of nine deviations of at most 0.5 to FP32 (3e-8 each,
    times velocities within 1.8: below 1e-6)."""
    print("[gpu] moments of 4097 x 4096 elements", flush=True)
    spec = workloads.periodic_box(nx=4097, ny=4096, p=1, velset=("gh", 3))
    g = binding.Solver.from_spec(spec, precision=binding.FP32)
    n = np.arange(g.K * g.Np)
    rho = 1.0 + 0.1 * (n % 8191) / 8191.0   # (a period that no element, row or launch shares)
    ux = 0.05 * (n % 8179) / 8179.0
    uy = -0.05 * (n % 8171) / 8171.0
    g.init_moments(rho, ux, uy)
    print("[gpu] state set", flush=True)
    r, x, y = (v.reshape(-1) for v in g.moments())
    for got, want in ((r, rho), (x, ux), (y, uy)):
        assert np.max(np.abs(got - want)) < 1e-6
    g.close()
