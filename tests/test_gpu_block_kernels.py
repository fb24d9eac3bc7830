"""The block kernels (GPU), which the steps run where a caller sets the elements
per work-group: one to sixteen elements at every order up to 4, partial last
blocks, strip order, odd Q Np (4-byte accesses in FP32), alone against the
oracle and in a batch against the same solvers alone; and one-element blocks
whose once-read streams move with non-temporal hints."""
import numpy as np
import pytest

import workloads
from paper_2012_13487_amd import binding
from test_gpu_rows import PRECISIONS, TOL, _errors, _spec

pytestmark = pytest.mark.gpu

# (p, velocities, nx, ny, walls, elements per work-group)
BLOCKS = [
    (2, 16, 8, 5, "couette", 1), (2, 16, 9, 7, "cavity", 4), (2, 25, 5, 3, "cavity", 2), (2, 13, 33, 4, "couette", 16),
    (4, 25, 5, 3, "cavity", 1), (4, 25, 5, 4, "cavity", 4), (4, 36, 6, 5, "box", 2), (4, 144, 5, 4, "cavity", 1),
    (1, 9, 7, 6, "cavity", 8), (3, 9, 5, 4, "box", 4),
    # strips of 16 columns and a narrower last one; blocks of two
    (2, 256, 20, 3, "cavity", 1), (3, 100, 40, 2, "cavity", 2),
]
IDS = [f"{c[4]}_{c[2]}x{c[3]}_p{c[0]}_q{c[1]}_E{c[5]}" for c in BLOCKS]
PREC = pytest.mark.parametrize("prec", PRECISIONS, ids=["fp64", "fp32", "fp32_ref"])


def _solver(case, prec):
    g = binding.Solver.from_spec(_spec(*case[:5]), precision=prec)
    g.set_block_elements(case[5])
    assert g.step_form()["form"] == 0 and g.tiling()["fused"] and g.tiling()["elems_per_group"] == case[5]
    return g


def _state(g, seed):
    return workloads.perturbed_state(seed, g.w, g.K, g.Np, amp=0.05)


@PREC
@pytest.mark.parametrize("case", BLOCKS, ids=IDS)
def test_steps_match_oracle(oracle_mod, case, prec):
    print(f"[gpu] blocks {case} precision {prec}", flush=True)
    g, o = _solver(case, prec), oracle_mod.Oracle.from_spec(_spec(*case[:5]))
    f = _state(g, 41 + case[1])
    dt = o.stable_dt(0.2)
    for s in (g, o):
        s.set_state(f)
    g.step(8, dt)
    o.rk4(8, dt)
    r, rc = o.residual()
    assert rc == 0 and abs(g.residual() - r) < TOL[prec] * r
    er, eu = _errors(g.moments(), o.moments())
    assert er < TOL[prec] and eu < TOL[prec], (er, eu)
    fo = o.get_state()
    assert np.max(np.abs(g.get_state() - fo)) < TOL[prec] * np.max(np.abs(fo))


@PREC
def test_batch_members_match_solo(prec):
    for graph in (0, 2):
        print(f"[gpu] blocks in a batch, precision {prec}, graph {graph}", flush=True)
        both = [[_solver(c, prec) for c in BLOCKS] for _ in range(2)]
        for sv in both:
            for i, g in enumerate(sv):
                g.set_state(_state(g, 17 + i))
        dts = np.array([g.stable_dt(0.2) for g in both[0]])
        b = binding.Batch(both[0], graph=graph)
        b.step(5, dts)
        r = b.residuals()
        for x, y, dt, rx in zip(both[0], both[1], dts, r):
            y.step(5, dt)
            assert np.array_equal(x.get_state(), y.get_state()) and rx == y.residual()
        b.close()


def test_one_element_blocks_and_tiles_agree():
    print("[gpu] one-element blocks vs tiles", flush=True)
    a, b = (binding.Solver.from_spec(workloads.cavity(n=8, p=3, m=12, lid=0.1)) for _ in range(2))
    a.set_block_elements(1)
    b.set_tiling(2, 40)
    assert a.step_form()["form"] == 0 and b.step_form()["form"] == 0
    for s in (a, b):
        s.init_equilibrium()
        s.step(30, s.stable_dt(0.2))
    fa = a.get_state()
    assert np.max(np.abs(b.get_state() - fa)) < 1e-13 * np.max(np.abs(fa))


def test_streaming_hints_of_one_element_blocks():
    """96x96, p = 3, 256 velocities (604 MB per FP32 state set): the blocks move
    their once-read streams with non-temporal hints; 50 steps against the FP64
    row kernels at the FP32 bar."""
    print("[gpu] blocks with streaming hints: 96x96 p3 nc16", flush=True)
    spec = workloads.cavity(n=96, p=3, m=16, lid=0.1)
    res = {}
    for prec in PRECISIONS:
        g = binding.Solver.from_spec(spec, precision=prec, stream="torch", torch_memory=True)
        if prec != binding.FP64:
            g.set_block_elements(1)
        assert g.step_form()["form"] == (1 if prec == binding.FP64 else 0)
        g.set_state(workloads.perturbed_state(79, g.w, g.K, g.Np, amp=0.05))
        g.step(50, g.stable_dt(spec.cfl))
        res[prec] = g.moments()
        g.close()
    for prec in (binding.FP32, binding.FP32_REF):
        er, eu = _errors(res[prec], res[binding.FP64])
        assert er < TOL[prec] and eu < TOL[prec], (prec, er, eu)
