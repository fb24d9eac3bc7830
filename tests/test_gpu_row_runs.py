"""Row kernels with several whole elements in a wavefront (GPU): two to four of
them, with and without rows of the element before (odd velocity counts start
off a 16-byte boundary), mesh rows that the wavefronts tile and rows that they
wrap around, a partial last wavefront, and launches large enough to be ordered
in strips (whole, narrower last, and none because the rows wrap) -- from states
that differ in every element, against the oracle, at the bars of each
precision; the residual; and members of a batch against the same solvers alone."""
import numpy as np
import pytest

import workloads
from paper_2012_13487_amd import binding
from test_gpu_rows import PRECISIONS, TOL, _errors, _spec

# (p, velocities, nx, ny, walls, elements per wavefront in FP64 and in FP32 storage)
RUNS = [
    (2, 16, 96, 24, "cavity", 4, 4),    # 576 wavefronts tile the rows
    (2, 16, 47, 47, "couette", 4, 4),   # rows wrap, the last wavefront has one element
    (2, 21, 48, 64, "cavity", 3, 2),    # odd rows with a lead; FP64: 1024 wavefronts in strips of 5, the last of 1
    (3, 20, 50, 33, "cavity", 3, 3),    # rows wrap
    (4, 30, 33, 32, "box", 2, 2),       # rows wrap
    (4, 31, 33, 32, "cavity", 2, 1),    # odd rows of 25 values
    (1, 8, 64, 64, "cavity", 4, 4),     # 1024 wavefronts in strips of 4
    (1, 13, 68, 64, "couette", 4, 4),   # the last strip of 1
    (2, 16, 128, 40, "box", 4, 4),      # 1280 wavefronts, eight strips
    (1, 15, 70, 60, "cavity", 4, 4),    # 1050 wavefronts, rows wrap: no strips
]
IDS = [f"{c[4]}_{c[2]}x{c[3]}_p{c[0]}_q{c[1]}" for c in RUNS]
PREC = pytest.mark.parametrize("prec", PRECISIONS, ids=["fp64", "fp32", "fp32_ref"])


def _solver(case, prec):
    g = binding.Solver.from_spec(_spec(*case[:5]), precision=prec)
    ew = case[5] if prec == binding.FP64 else case[6]
    assert g.step_form() == {"form": 2, "wavefronts": 1, "velocity_tiles": 1, "elems_per_wavefront": ew}
    return g


def _state(g, seed):
    return workloads.perturbed_state(seed, g.w, g.K, g.Np, amp=0.05)


@PREC
@pytest.mark.parametrize("case", RUNS, ids=IDS)
def test_plans(case, prec):
    _solver(case, prec)


@pytest.mark.gpu
@PREC
@pytest.mark.parametrize("case", RUNS, ids=IDS)
def test_runs_of_elements_match_oracle(oracle_mod, case, prec):
    print(f"[gpu] row runs {case} precision {prec}", flush=True)
    g, o = _solver(case, prec), oracle_mod.Oracle.from_spec(_spec(*case[:5]))
    f = _state(g, 31 + case[1])
    dt = o.stable_dt(0.2)
    for s in (g, o):
        s.set_state(f)
    g.step(5, dt)
    o.rk4(5, dt)
    r, rc = o.residual()
    assert rc == 0 and abs(g.residual() - r) < TOL[prec] * r
    er, eu = _errors(g.moments(), o.moments())
    assert er < TOL[prec] and eu < TOL[prec], (er, eu)
    fo, mid = o.get_state(), g.get_state()
    assert np.max(np.abs(mid - fo)) < TOL[prec] * np.max(np.abs(fo))
    if prec == binding.FP64:
        g.step(3, dt)
        h = _solver(case, prec)
        h.set_state(mid)
        h.step(3, dt)
        assert np.array_equal(h.get_state(), g.get_state())


@pytest.mark.gpu
@PREC
def test_runs_of_elements_in_a_batch_match_solo(prec):
    for graph in (0, 2):
        print(f"[gpu] row runs in a batch, precision {prec}, graph {graph}", flush=True)
        both = [[_solver(c, prec) for c in RUNS] for _ in range(2)]
        for sv in both:
            for i, g in enumerate(sv):
                g.set_state(_state(g, 7 + i))
        dts = np.array([g.stable_dt(0.2) for g in both[0]])
        b = binding.Batch(both[0], graph=graph)
        b.step(5, dts)
        r = b.residuals()
        for x, y, dt, rx in zip(both[0], both[1], dts, r):
            y.step(5, dt)
            assert np.array_equal(x.get_state(), y.get_state()) and rx == y.residual()
        b.close()
