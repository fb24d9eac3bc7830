"""Implicit steps that fail (GPU): nothing of the call is left running when it
returns, although products are enqueued ahead of the projections the host reads
(the allocation-free entry point's workspace belongs to the next caller)."""
import numpy as np
import pytest

import workloads
from paper_2012_13487_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("noalloc", [False, True], ids=["own", "static"])
@pytest.mark.parametrize("p,m,n", [(3, 12, 16), (2, 6, 24)])
def test_a_failed_step_leaves_nothing_running(p, m, n, noalloc):
    """A uniform state of 1e160 without walls: its residual is rounding (1e144 or
    so) and finite in the 2-norm, |y|^2 is not, and with the difference step
    neither is the first Krylov vector."""
    import torch
    print(f"[gpu] failing implicit step p{p} m{m} {n}x{n} noalloc {noalloc}", flush=True)
    side = torch.cuda.Stream()
    g = binding.Solver.from_spec(workloads.periodic_box(nx=n, ny=n, p=p, velset=("nc", m, 4.0)), stream=side.cuda_stream)
    dt = g.stable_dt(0.2)
    opt = dict(restart=4)
    g.init_equilibrium()
    g.implicit_step(1, dt, "backward_euler", **opt)  # (the pinned memory that products ahead need)
    g.init_equilibrium(1e160)
    f = g.get_state()
    with pytest.raises(binding.DgbgkError) as e:
        g.implicit_step(1, dt, "backward_euler", noalloc=noalloc, **opt)
    idle = side.query()
    assert e.value.code == binding.ENONFINITE and "Krylov" in str(e.value)
    assert idle
    assert np.array_equal(g.get_state(), f)
    g.init_equilibrium()
    assert g.implicit_step(1, dt, "backward_euler", noalloc=noalloc, **opt)["converged"] == 1
    g.set_stream(None)
