"""Calls recorded into a caller's HIP graph (GPU).  A replay finds the state
that is there then, which may have been set, folded or stepped since the
capture: steps, residuals and folds of a replay, and ordinary calls after it,
equal the same calls made one after the other on a solver of its own, bit for
bit.  (One-element block kernels sum the moments of a state in another order
than those of a stage's output; the solver that is called directly is made to
reduce them at the start of each call too.)  Sizes: moments handed between stages (one tile, several), in the
wavefront, and by the block kernels."""
import numpy as np
import pytest

import workloads
from paper_2012_13487_amd import binding
from test_gpu_rows import _spec

pytestmark = pytest.mark.gpu

SIZES = [(2, 81, 0), (4, 65, 0), (3, 100, 0), (2, 300, 0), (2, 16, 0), (3, 16, 1), (2, 81, 1)]
IDS = [f"p{p}_q{q}" + ("_blocks" if e else "") for p, q, e in SIZES]
PRECISIONS = pytest.mark.parametrize("prec", [binding.FP64, binding.FP32, binding.FP32_REF],
                                     ids=["fp64", "fp32", "fp32_ref"])


def _pair(spec, prec, blocks, stream):
    out = []
    for st in (stream, None):
        g = binding.Solver.from_spec(spec, precision=prec, stream=st)
        if blocks:
            g.set_block_elements(blocks)
        out.append(g)
    return out


def _reduces(h, blocks):
    """Make the next call of h reduce the moments of its state."""
    if blocks:
        h.set_block_elements(blocks)
    return h


def _state(g, seed):
    return workloads.perturbed_state(seed, g.w, g.K, g.Np, amp=0.05)


@PRECISIONS
@pytest.mark.parametrize("p,q,blocks", SIZES, ids=IDS)
def test_replayed_steps_follow_the_state_that_is_there(p, q, blocks, prec):
    import torch
    spec = _spec(p, q, 5, 4, "cavity")
    print(f"[gpu] captured steps {spec.name} precision {prec} blocks {blocks}", flush=True)
    side = torch.cuda.Stream()
    g, h = _pair(spec, prec, blocks, side.cuda_stream)
    dt = g.stable_dt(0.2)
    for s in (g, h):
        s.set_state(_state(g, 1))
        s.step(2, dt)  # (the tables are on the device, the moments of the state at hand)
    g.synchronize()
    out = torch.zeros(1, dtype=torch.float64, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        g.step(3, dt)
        g.residual_async(out.data_ptr())
        if prec == binding.FP32_REF:
            g.fold()
    torch.cuda.synchronize()

    def check(replays):
        for _ in range(replays):
            with torch.cuda.stream(side):
                graph.replay()
            torch.cuda.synchronize()
            _reduces(h, blocks).step(3, dt)
            assert out.item() == _reduces(h, blocks).residual()
            if prec == binding.FP32_REF:
                h.fold()
        assert np.array_equal(g.get_state(), h.get_state())

    check(2)                                   # the state as the capture left it
    for s in (g, h):
        s.set_state(_state(g, 2))              # another state, then replays only
    check(2)
    for s in (g, _reduces(h, blocks)):         # ordinary calls between replays
        s.step(2, dt)
    assert g.residual() == _reduces(h, blocks).residual()
    check(1)
    for s in (g, h):
        s.init_equilibrium(1.2, 0.01, 0.02)
    check(1)
    assert g.residual() == _reduces(h, blocks).residual()
    for s in (g, _reduces(h, blocks)):         # and the library's own graph after them
        s.set_graph(2)
        s.step(5, dt)
    check(1)
    for s in (g, _reduces(h, blocks)):
        s.step(4, dt)
    assert np.array_equal(g.get_state(), h.get_state())
    g.set_stream(None)


@PRECISIONS
def test_replayed_batch_steps_follow_the_states_that_are_there(prec):
    import torch
    print(f"[gpu] captured batch steps, precision {prec}", flush=True)
    side = torch.cuda.Stream()
    pairs = [_pair(_spec(p, q, 5, 4, "cavity"), prec, e, side.cuda_stream) for p, q, e in SIZES]
    dts = np.array([g.stable_dt(0.2) for g, _ in pairs])
    for i, (g, h) in enumerate(pairs):
        for s in (g, h):
            s.set_state(_state(g, 10 + i))
    a, b = binding.Batch([g for g, _ in pairs], stream=side.cuda_stream), binding.Batch([h for _, h in pairs])
    for x in (a, b):
        x.step(2, dts)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        a.step(2, dts)
    torch.cuda.synchronize()
    for seed in (20, 30):
        for i, (g, h) in enumerate(pairs):
            for s in (g, h):
                s.set_state(_state(g, seed + i))
        for _ in range(2):
            with torch.cuda.stream(side):
                graph.replay()
            torch.cuda.synchronize()
            for (_, h), (_, _, e) in zip(pairs, SIZES):
                _reduces(h, e)
            b.step(2, dts)
        for (_, h), (_, _, e) in zip(pairs, SIZES):
            _reduces(h, e)
        assert np.array_equal(a.residuals(), b.residuals())
        for g, h in pairs:
            assert np.array_equal(g.get_state(), h.get_state())
    a.close()
    b.close()
    for g, _ in pairs:
        g.set_stream(None)


def _failed_capture():
    """A batch of one solver whose call of three steps took one and could not
    capture the graph of the rest: the stream is being captured already."""
    import torch
    side = torch.cuda.Stream()
    g = binding.Solver.from_spec(_spec(2, 16, 5, 4, "cavity"), stream=side.cuda_stream)
    g.set_state(_state(g, 3))
    b = binding.Batch([g], stream=side.cuda_stream)
    dt = [g.stable_dt(0.2)]
    b.step(1, dt)
    b.set_graph(2)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        with pytest.raises(binding.DgbgkError) as e:
            b.step(3, dt)
    assert e.value.code == binding.EDEVICE
    torch.cuda.synchronize()
    return g, b, dt


def test_an_error_is_reported_once():
    """The calls after a reported HIP error work: its last-error slot is empty."""
    print("[gpu] calls after a failed capture", flush=True)
    g, b, dt = _failed_capture()
    h = binding.Solver.from_spec(_spec(2, 16, 5, 4, "cavity"))
    for s in (g, h):
        s.set_state(_state(g, 4))
    b.step(4, dt)
    h.step(4, dt[0])
    assert np.array_equal(g.get_state(), h.get_state())
    b.close()
    g.set_stream(None)


def test_a_batch_counts_the_steps_it_enqueued_before_a_failure():
    print("[gpu] batch: steps counted before a failed capture", flush=True)
    g, b, dt = _failed_capture()
    assert g.steps_taken() == 2  # (one before, one in the failed call)
    b.step(5, dt)                # (an eager one and two replays)
    assert g.steps_taken() == 7
    b.close()
    g.set_stream(None)
