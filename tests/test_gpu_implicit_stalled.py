"""Implicit steps whose GMRES cycles are too short to converge (GPU): row
kernels and block kernels stop after the same iterations in the same state.
Their products differ by the rounding of L over the difference step, 1e-16 /
1e-6 = 1e-10 of the transport terms; a factor of 1e3 for the conditioning of
the solves at 100 explicit steps and as much again for their restarts and the
Newton steps gives the bar of 1e-4 of the step's change."""
import numpy as np
import pytest

import workloads
from paper_2012_13487_amd import binding
from test_gpu_rows import _spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp32_basis", [False, True], ids=["basis64", "basis32"])
@pytest.mark.parametrize("p,q,nx,ny,restart", [(2, 9, 3, 1, 5), (1, 65, 3, 3, 1)])
def test_stalled_step_matches_block_kernels(p, q, nx, ny, restart, fp32_basis):
    spec = _spec(p, q, nx, ny, "cavity")
    print(f"[gpu] stalled implicit step {spec.name} restart {restart} fp32 basis {fp32_basis}", flush=True)
    g, b = (binding.Solver.from_spec(spec) for _ in range(2))
    b.set_block_elements(1)
    assert g.step_form()["form"] != 0 and b.step_form()["form"] == 0
    f = workloads.perturbed_state(5 + q, g.w, g.K, g.Np, amp=0.15)
    dt = 100 * g.stable_dt(0.2)
    opt = dict(newton_rtol=1e-13, newton_atol=1e-17, max_newton=4, krylov_rtol=1e-5 if fp32_basis else 1e-8,
               max_krylov=1000, restart=restart, krylov_fp32=fp32_basis)
    rep = []
    for s in (g, b):
        s.set_state(f)
        rep.append(s.implicit_step(1, dt, "backward_euler", **opt))
    assert rep[0]["converged"] == rep[1]["converged"] == 0
    assert abs(rep[0]["max_final_residual"] - rep[1]["max_final_residual"]) < 1e-4 * rep[1]["max_final_residual"]
    y = b.get_state()
    assert np.max(np.abs(g.get_state() - y)) < 1e-4 * np.max(np.abs(y - f))
