"""FP32 storage: the device memory a solver asks for (host only), and calls that
move a state through the FP64 transfer buffer, where row plans of several
velocity tiles, and those of orders 2 and 4, keep the moment sums handed from
one step to the next (GPU): they leave the steps as they are, bit for bit."""
import numpy as np
import pytest

import workloads
from paper_2012_13487_amd import binding
from test_gpu_rows import TOL, _errors, _spec

PRECISIONS = pytest.mark.parametrize("prec", [binding.FP32, binding.FP32_REF], ids=["fp32", "fp32_ref"])


def _layout(K, p, Q, ref):
    """Four FP32 registers, the FP64 transfer buffer, the tables, the reference
    (FP64 state, its FP32 rate, its moments), and two slots of seven moments per
    node for the orders whose one-element blocks hand them on."""
    Nfp, Np = p + 1, (p + 1) ** 2
    n, up = K * Np * Q, lambda b: (b + 255) // 256 * 256  # noqa: E731
    total = 4 * up(4 * n) + up(8 * n) + up(24 * Q) + up(32 * Q) + up(128 * Q) + up(24 * K * Np) + up(32 * K * Nfp)
    total += up(64) + up((2 * Np + 15) // 16 * 16 * 32 * 2)
    if ref:
        total += up(8 * n) + up(4 * n) + up(24 * K * Np)
    return total + (2 * up(56 * K * Np) if p in (1, 3) else 0)


@PRECISIONS
@pytest.mark.parametrize("p,m,n", [(2, 9, 5), (4, 24, 128), (3, 16, 64), (3, 24, 7), (1, 9, 1), (2, 31, 1)])
def test_required_bytes_have_no_part_for_the_row_plans(p, m, n, prec):
    spec = workloads.cavity(n=n, p=p, m=m)
    vel = binding.velocity_set(spec.velset)
    got = binding.required_bytes(n, n, p, vel, 0.8, spec.bc, spec.wall_u, precision=prec)
    assert got == _layout(n * n, p, m * m, prec == binding.FP32_REF)


@pytest.mark.gpu
@PRECISIONS
@pytest.mark.parametrize("p,q,nx,ny", [(2, 62, 1, 1), (2, 81, 5, 3), (4, 65, 3, 2), (4, 321, 3, 2), (2, 1021, 2, 2),
                                       (3, 100, 4, 3), (3, 513, 3, 2), (1, 257, 5, 4)])
def test_calls_between_steps_leave_the_steps_as_they_are(p, q, nx, ny, prec):
    spec = _spec(p, q, nx, ny, "cavity")
    print(f"[gpu] transfers between steps {spec.name} precision {prec}", flush=True)
    a, b = (binding.Solver.from_spec(spec, precision=prec) for _ in range(2))
    assert a.step_form()["form"] == 1
    f = workloads.perturbed_state(5 + q, a.w, a.K, a.Np, amp=0.05)
    dt = a.stable_dt(0.2)
    for s in (a, b):
        s.set_state(f)
        s.step(3, dt)
    between = [a.get_state, lambda: a.rhs(f), a.residual, a.moments]
    if prec != binding.FP32_REF:
        between.append(lambda: a.wall_density(f))
    for graph in (0, 2):
        for s in (a, b):
            s.set_graph(graph)
        for call in between:
            call()
            a.step(4, dt)
            b.step(4, dt)
        assert np.array_equal(a.get_state(), b.get_state())
        assert a.residual() == b.residual()


@pytest.mark.gpu
@PRECISIONS
@pytest.mark.parametrize("p,q", [(3, 513), (1, 257)])
def test_one_element_blocks_share_the_buffer(oracle_mod, p, q, prec):
    """The block kernels of such velocity counts hand their moments on in the
    same place: steps with transfers between them against the oracle."""
    spec = _spec(p, q, 3, 2, "cavity")
    print(f"[gpu] transfers between steps of blocks {spec.name} precision {prec}", flush=True)
    g, o = binding.Solver.from_spec(spec, precision=prec), oracle_mod.Oracle.from_spec(spec)
    g.set_block_elements(1)
    assert g.step_form()["form"] == 0
    f = workloads.perturbed_state(9 + q, g.w, g.K, g.Np, amp=0.05)
    dt = o.stable_dt(0.2)
    for s in (g, o):
        s.set_state(f)
    for call in (g.get_state, lambda: g.rhs(f), g.residual):
        g.step(3, dt)
        o.rk4(3, dt)
        call()
    r, _ = o.residual()
    assert abs(g.residual() - r) < TOL[prec] * r
    er, eu = _errors(g.moments(), o.moments())
    assert er < TOL[prec] and eu < TOL[prec], (er, eu)
