"""Which kernels the steps of a solver run (host only): the row kernels' plans,
and the choices of a caller that select the block kernels instead."""
import pytest

import workloads
from paper_2012_13487_amd import binding

BLOCKS = {"form": 0, "wavefronts": 0, "velocity_tiles": 0, "elems_per_wavefront": 0}


def _form(spec, precision=binding.FP64):
    f = binding.Solver.from_spec(spec, precision=precision).step_form()
    return f["form"], f["wavefronts"], f["velocity_tiles"], f["elems_per_wavefront"]


@pytest.mark.parametrize("prec", [binding.FP64, binding.FP32, binding.FP32_REF], ids=["fp64", "fp32", "fp32_ref"])
def test_row_plans(prec):
    # few elements: one per wavefront; many: as many as 64 rows hold, up to four
    assert _form(workloads.couette(nx=8, ny=8, p=2), prec) == (2, 1, 1, 1)
    assert _form(workloads.couette(nx=96, ny=96, p=2), prec) == (2, 1, 1, 4)
    assert _form(workloads.couette(nx=40, ny=40, p=3), prec) == (2, 1, 1, 2)
    # 256 velocities: four wavefronts; 576: three tiles of three
    assert _form(workloads.CAVITY_64x64_P3_NC16, prec) == (1, 4, 1, 1)
    assert _form(workloads.CAVITY_128x128_P4_NC24_KN8, prec) == (1, 3, 3, 1)


def test_choices_that_run_the_block_kernels():
    s = binding.Solver.from_spec(workloads.CAVITY_64x64_P3_NC16)
    rows = s.step_form()
    assert rows["form"] == 1
    for choose in (lambda: s.set_block_elements(1), lambda: s.set_tiling(2, 48), lambda: s.set_tiling(4)):
        choose()
        assert s.step_form() == BLOCKS
        s.set_block_elements(0)
        s.set_tiling(0)
        assert s.step_form() == rows
    for mode in (1, 3):  # these name the form of the block kernels where they run
        s.set_tiling(mode)
        assert s.step_form() == rows
    for spec, prec in ((workloads.cavity(n=2, p=5, m=4), binding.FP64),
                       (workloads.periodic_box(velset=("gh", 2)), binding.FP64),
                       (workloads.cavity(n=4, p=3, m=40), binding.FP64),
                       (workloads.cavity(n=4, p=2, m=8), binding.FP32_BF16MMA)):
        assert binding.Solver.from_spec(spec, precision=prec).step_form() == BLOCKS


def test_meshes_beyond_one_launch_of_the_row_kernels_run_the_block_kernels():
    """A launch holds fewer than 2^32 threads along x: 256 per element of 196
    velocities, 64 per element of 36, 128 per element of 81."""
    box = lambda nx, ny, n: workloads.periodic_box(nx=nx, ny=ny, p=1, velset=("gh", n))  # noqa: E731
    assert _form(box(4095, 4096, 14)) == (1, 4, 1, 1) and _form(box(4096, 4096, 14))[0] == 0
    assert _form(box(8191, 8192, 6)) == (2, 1, 1, 1) and _form(box(8192, 8192, 6))[0] == 0
    assert _form(box(4096, 8191, 9)) == (1, 2, 1, 1) and _form(box(4096, 8192, 9))[0] == 0
    t = binding.Solver.from_spec(box(4096, 8192, 9)).tiling()  # (several elements per work-group of 256)
    assert t["fused"] and t["elems_per_group"] >= 2
