"""Row kernels (GPU): the RK stages by wavefronts of 64 velocity rows, at the
sizes where their splits change -- the smallest velocity count, whole elements
in a wavefront with and without rows of the element before (odd counts start
off a 16-byte boundary), the last count that fits a wavefront and the first
that does not, partial and full last wavefronts, one to four velocity tiles,
meshes narrower than, equal to and wider than the strips the work-groups are
ordered in -- against the oracle, at the bars of each precision; and the parts
that share state: a state read out and set again continues bit for bit, batch
members equal the same solvers alone."""
import numpy as np
import pytest

import workloads
from paper_2012_13487_amd import binding

pytestmark = pytest.mark.gpu

TOL = {binding.FP64: 1e-12, binding.FP32: 1e-5, binding.FP32_REF: 1e-5}
PRECISIONS = [binding.FP64, binding.FP32, binding.FP32_REF]


def _velocities(q):
    """q seeded velocities on [-3, 3]^2, a few of them parallel to a face, with
    positive weights summing to one."""
    rng = np.random.default_rng(q)
    ex, ey = rng.uniform(-3.0, 3.0, q), rng.uniform(-3.0, 3.0, q)
    ex[q // 3] = 0.0
    ey[q // 2] = 0.0
    w = rng.uniform(0.5, 1.5, q)
    return "custom", ex, ey, w / w.sum(), 1.0


def _spec(p, q, nx, ny, walls):
    bc = {"cavity": (1, 1, 1, 1), "couette": (1, 0, 1, 0), "box": (0, 0, 0, 0)}[walls]
    wall_u = ((0.0, 0.0), (0.0, 0.0), (0.1, 0.0), (0.0, 0.0))
    return workloads.ProblemSpec(name=f"{walls}_{nx}x{ny}_p{p}_q{q}", nx=nx, ny=ny, p=p, velset=_velocities(q),
                                 kn=0.8, bc=bc, wall_u=wall_u)


CASES = [
    # whole elements in a wavefront
    (1, 8, 5, 3, "cavity"), (2, 9, 7, 5, "cavity"), (2, 16, 33, 16, "couette"), (3, 15, 6, 7, "box"),
    (4, 13, 5, 4, "cavity"), (2, 21, 9, 4, "couette"), (4, 31, 3, 5, "cavity"), (1, 64, 4, 4, "cavity"),
    (2, 61, 3, 5, "cavity"), (2, 64, 5, 3, "box"), (3, 64, 3, 3, "couette"), (4, 64, 3, 2, "cavity"),
    # an element over several wavefronts and velocity tiles
    (1, 65, 34, 31, "cavity"), (2, 62, 3, 3, "cavity"), (2, 63, 3, 5, "couette"), (2, 65, 5, 3, "cavity"),
    (3, 65, 4, 3, "cavity"), (4, 65, 3, 3, "box"), (2, 127, 3, 3, "cavity"), (4, 129, 3, 3, "couette"),
    (3, 256, 32, 33, "box"), (2, 257, 3, 2, "cavity"), (4, 321, 2, 3, "cavity"), (3, 513, 2, 2, "cavity"),
    (2, 1021, 2, 1, "couette"), (4, 1023, 1, 2, "cavity"), (1, 1024, 2, 2, "box"),
]


def _errors(got, want):
    er = np.max(np.abs(got[0] - want[0])) / np.max(np.abs(want[0]))
    u = np.stack(want[1:])
    return er, np.max(np.abs(np.stack(got[1:]) - u)) / np.max(np.abs(u))


@pytest.mark.parametrize("prec", PRECISIONS, ids=["fp64", "fp32", "fp32_ref"])
@pytest.mark.parametrize("p,q,nx,ny,walls", CASES, ids=[f"{c[4]}_{c[2]}x{c[3]}_p{c[0]}_q{c[1]}" for c in CASES])
def test_row_kernels_match_oracle(oracle_mod, p, q, nx, ny, walls, prec):
    """Five steps of a perturbed state, the residual, then three more from the
    state read out and set again."""
    spec = _spec(p, q, nx, ny, walls)
    print(f"[gpu] rows {spec.name} precision {prec}", flush=True)
    g, o = binding.Solver.from_spec(spec, precision=prec), oracle_mod.Oracle.from_spec(spec)
    f = workloads.perturbed_state(97 + q, o.w, o.K, o.Np, amp=0.05)
    dt = o.stable_dt(0.2)
    for s in (g, o):
        s.set_state(f)
    g.step(5, dt)
    o.rk4(5, dt)
    r, rc = o.residual()
    assert rc == 0 and abs(g.residual() - r) < TOL[prec] * r
    er, eu = _errors(g.moments(), o.moments())
    assert er < TOL[prec] and eu < TOL[prec], (er, eu)
    if prec == binding.FP64:
        fo, mid = o.get_state(), g.get_state()
        assert np.max(np.abs(mid - fo)) < TOL[prec] * np.max(np.abs(fo))
        g.step(3, dt)
        h = binding.Solver.from_spec(spec)
        h.set_state(mid)
        h.step(3, dt)
        assert np.array_equal(h.get_state(), g.get_state())


@pytest.mark.parametrize("prec", PRECISIONS, ids=["fp64", "fp32", "fp32_ref"])
def test_row_kernels_in_a_batch_match_solo(prec):
    """Members of both plans and of every order, eager and from a graph."""
    specs = [_spec(*c) for c in CASES if c[1] in (8, 9, 16, 31, 61, 64, 65, 129, 513)]
    for graph in (0, 2):
        print(f"[gpu] rows in a batch, precision {prec}, graph {graph}", flush=True)
        both = []
        for _ in range(2):
            sv = [binding.Solver.from_spec(s, precision=prec) for s in specs]
            for i, g in enumerate(sv):
                g.set_state(workloads.perturbed_state(7 + i, g.w, g.K, g.Np, amp=0.05))
            both.append(sv)
        dts = np.array([g.stable_dt(0.2) for g in both[0]])
        b = binding.Batch(both[0], graph=graph)
        b.step(5, dts)
        r = b.residuals()
        for x, y, dt, rx in zip(both[0], both[1], dts, r):
            y.step(5, dt)
            assert np.array_equal(x.get_state(), y.get_state()) and rx == y.residual()
        b.close()


@pytest.mark.parametrize("prec", PRECISIONS, ids=["fp64", "fp32", "fp32_ref"])
@pytest.mark.parametrize("p,q", [(1, 8), (2, 9), (3, 15), (4, 31), (2, 62), (3, 65), (4, 129), (4, 321), (2, 1021)])
def test_residual_matches_the_rates_block_kernels_write(p, q, prec):
    """The residual reduced inside the row kernels (whole elements in a
    wavefront, one to four velocity tiles) against the block kernels' rates
    reduced by a pass of its own; twice the same number; a value that is NaN is reported."""
    spec = _spec(p, q, 5, 3, "cavity")
    print(f"[gpu] residual {spec.name} precision {prec}", flush=True)
    g = binding.Solver.from_spec(spec, precision=prec)
    f = workloads.perturbed_state(11 + q, g.w, g.K, g.Np, amp=0.05)
    g.set_state(f)
    r = [g.residual(), g.residual()]
    before = g.get_state()
    g.set_block_elements(1)
    want = g.residual()
    assert r[0] == r[1] and abs(r[0] - want) < TOL[prec] * want
    assert np.array_equal(g.get_state(), before)
    if prec != binding.FP32_REF:
        g.set_block_elements(0)
        f.reshape(-1)[f.size // 2] = np.nan
        g.set_state(f)
        with pytest.raises(binding.DgbgkError) as e:
            g.residual()
        assert e.value.code == binding.ENONFINITE


@pytest.mark.parametrize("fp32_basis", [False, True], ids=["basis64", "basis32"])
@pytest.mark.parametrize("p,q,nx,ny,walls,mult,restart",
                         [(1, 9, 1, 1, "box", 10, 30), (2, 9, 3, 1, "cavity", 100, 5), (3, 15, 5, 3, "couette", 10, 30),
                          (4, 31, 3, 3, "cavity", 30, 64), (1, 65, 3, 3, "cavity", 100, 1), (2, 62, 3, 3, "cavity", 10, 30),
                          (2, 257, 3, 2, "couette", 30, 12), (3, 65, 2, 3, "box", 10, 30), (4, 321, 2, 2, "cavity", 10, 30)])
def test_implicit_step_by_row_kernels_solves_its_equation(oracle_mod, p, q, nx, ny, walls, mult, restart, fp32_basis):
    """A backward-Euler step with its products by the row kernels (odd lengths,
    one to several velocity tiles, second Gram-Schmidt passes, short and long
    cycles): y - f - dt L(y) with the oracle's L.  Newton stops at 1e-13 of the
    first residual in the 2-norm, at most 1e-13 sqrt(n) < 2e-11 in the maximum
    norm; the bar leaves the rest to the rounding of L."""
    spec = _spec(p, q, nx, ny, walls)
    print(f"[gpu] implicit rows {spec.name} x{mult} restart {restart} fp32 basis {fp32_basis}", flush=True)
    g, o = binding.Solver.from_spec(spec), oracle_mod.Oracle.from_spec(spec)
    f = workloads.perturbed_state(5 + q, o.w, o.K, o.Np, amp=0.15)
    dt = mult * o.stable_dt(0.2)
    g.set_state(f)
    r0 = g.residual()
    opt = dict(newton_rtol=1e-13, newton_atol=1e-17, max_newton=4 if mult == 100 else 60,
               krylov_rtol=1e-5 if fp32_basis else 1e-8, max_krylov=1000, restart=restart, krylov_fp32=fp32_basis)
    rep = g.implicit_step(1, dt, "backward_euler", **opt)
    y = g.get_state()
    if mult == 100:  # (cycles this short stagnate at this step, with the block kernels' products as well)
        b = binding.Solver.from_spec(spec)
        b.set_block_elements(1)
        b.set_state(f)
        blocks = b.implicit_step(1, dt, "backward_euler", **opt)
        for name in ("converged", "newton_iterations", "krylov_iterations", "rhs_evaluations"):
            assert rep[name] == blocks[name], (rep, blocks)
    else:
        assert rep["converged"] == 1, rep
        F = y - f - dt * o.rhs(y)
        assert np.max(np.abs(F)) < 1e-10 * np.max(np.abs(dt * o.rhs(f)))
    h = binding.Solver.from_spec(spec)  # (the sums of f_n that a residual left behind are not the new state's)
    h.set_state(y)
    assert h.residual() == g.residual() and r0 > 0


def test_block_elements_and_tiles_choose_the_block_kernels(oracle_mod):
    """A block size or a velocity tile set by the caller keeps the block kernels
    (rounding apart from the automatic row kernels), back to automatic the row
    kernels continue; a change in between keeps the state."""
    spec = _spec(2, 169, 5, 4, "cavity")
    o = oracle_mod.Oracle.from_spec(spec)
    g = binding.Solver.from_spec(spec)
    f = workloads.perturbed_state(3, o.w, o.K, o.Np, amp=0.05)
    for s in (g, o):
        s.set_state(f)
    dt = o.stable_dt(0.2)
    for change in (lambda: None, lambda: g.set_block_elements(1), lambda: g.set_block_elements(0),
                   lambda: g.set_tiling(2, 50), lambda: g.set_tiling(0), lambda: g.set_graph(2)):
        change()
        g.step(4, dt)
        o.rk4(4, dt)
        fo = o.get_state()
        assert np.max(np.abs(g.get_state() - fo)) < 1e-12 * np.max(np.abs(fo))
