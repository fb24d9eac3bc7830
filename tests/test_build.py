"""The build refuses row kernels that use scratch memory (host only: hipcc
compiles for the GPU without one)."""
import pytest

from paper_2012_13487_amd import build

KERNEL = """
#include <hip/hip_runtime.h>
// 64 values per lane, all live across a barrier
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu({waves}, {waves})))
void many_values(const float *in, float *out) {{
  float v[64];
#pragma unroll
  for (int i = 0; i < 64; ++i) v[i] = in[i * 256 + threadIdx.x];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 64; ++i) out[(63 - i) * 256 + threadIdx.x] = v[i] * v[(i + 31) % 64] + v[(i * 7 + 5) % 64];
}}
"""


@pytest.mark.parametrize("waves,fits", [(2, True), (8, False)])
def test_scratch_in_a_row_kernel_fails_the_build(tmp_path, waves, fits):
    src = build.NO_SCRATCH[0]
    (tmp_path / src).write_text(KERNEL.format(waves=waves))
    if fits:
        assert build.compile_sources([src], str(tmp_path), str(tmp_path)) == [str(tmp_path / (src + ".o"))]
        return
    with pytest.raises(RuntimeError, match="scratch memory.*many_values"):
        build.compile_sources([src], str(tmp_path), str(tmp_path))


def test_sources_that_are_not_checked_may_use_scratch(tmp_path):
    src = "kernels.hip"  # (the block kernels of p >= 5 do)
    assert src not in build.NO_SCRATCH
    (tmp_path / src).write_text(KERNEL.format(waves=8))
    build.compile_sources([src], str(tmp_path), str(tmp_path))


def test_remarks_that_are_missing_are_an_error():
    with pytest.raises(RuntimeError, match="no kernel resource remarks"):
        build.scratch_users("warning: something else\n")
    with pytest.raises(RuntimeError, match="incomplete"):
        build.scratch_users("x.hip:1:1: remark: Function Name: k [-R]\nx.hip:1:1: remark:     VGPRs: 8 [-R]\n")
