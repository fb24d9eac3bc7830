"""Node moments (GPU): one work-group per element, a few velocities at a time,
at the node counts and velocity counts where that split has remainders, against
sums of the state that is read out.  Both sum the same FP64 values in another
order: at most (q + H) eps of sum |e f|, below 1e-12 of the largest density for
velocities within 3 and up to 513 of them."""
import numpy as np
import pytest

import workloads
from paper_2012_13487_amd import binding
from test_gpu_rows import _spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [binding.FP64, binding.FP32, binding.FP32_REF], ids=["fp64", "fp32", "fp32_ref"])
@pytest.mark.parametrize("p,q", [(1, 5), (1, 65), (2, 9), (2, 28), (2, 29), (3, 16), (3, 513), (4, 10), (4, 257)])
def test_moments_are_the_sums_of_the_state(p, q, prec):
    spec = _spec(p, q, 5, 3, "cavity")
    print(f"[gpu] moments {spec.name} precision {prec}", flush=True)
    g = binding.Solver.from_spec(spec, precision=prec)
    g.set_state(workloads.perturbed_state(13 + q, g.w, g.K, g.Np, amp=0.1))
    g.step(3, g.stable_dt(0.2))
    if prec == binding.FP32_REF and q % 2:
        g.fold()
        g.step(2, g.stable_dt(0.2))
    f = g.get_state().reshape(q, g.K, g.Np)
    rho = f.sum(axis=0)
    m = [np.tensordot(e, f, axes=1) for e in (g.ex, g.ey)]
    got = [np.asarray(v).reshape(rho.shape) for v in g.moments()]
    top = np.max(rho)
    assert np.max(np.abs(got[0] - rho)) < 1e-12 * top
    for u, mu in zip(got[1:], m):
        assert np.max(np.abs(u * rho - mu)) < 1e-12 * top
