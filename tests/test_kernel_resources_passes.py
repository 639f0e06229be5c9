"""Register budget of the passes that grids take by default (CPU), beside the
kernels of test_kernel_resources.py: three steps a pass, the tile passes, user
coefficients and sources.  Read from the built library's code objects."""
import pytest

from test_kernel_resources import kernels  # noqa: F401  (fixture)

# kernel (demangled prefix): most registers of a wavefront, most spilled
BUDGET = {
    "lw_step3_kernel<true, false,": (256, 0),
    "lw_batch3_kernel": (256, 0),
    "lw_step_kernel<true, true,": (256, 0),
    "lw_step_kernel<false,": (256, 0),
    "lw_step2_kernel<true, true,": (256, 0),
    "lw_step2_kernel<false,": (256, 0),
    "lw_step3_kernel<true, true,": (512, 8),  # one wavefront to a SIMD
    # workgroups of up to 1024 threads (four wavefronts to a SIMD), 512 (two)
    "lw_tile_kernel<16, 1, 1024,": (128, 0),
    "lw_tile_kernel<32, 1, 1024,": (128, 0),
    "lw_tile_kernel<64, 1, 1024,": (128, 0),
    "lw_tile_kernel<32, 2, 512,": (256, 0),
    "lw_tile_kernel<64, 2, 512,": (256, 0),
    "lw_tile_kernel<64, 3, 512,": (256, 0),
    "lw_adjoint_tile_kernel<16, 1, 1024,": (128, 0),
    "lw_adjoint_tile_kernel<32, 1, 1024,": (128, 0),
    "lw_adjoint_tile_kernel<64, 1, 1024,": (128, 0),
    "lw_adjoint_tile_kernel<32, 2, 512,": (256, 0),
    "lw_adjoint_tile_kernel<64, 2, 512,": (256, 0),
    "lw_adjoint_tile_kernel<64, 3, 512,": (256, 0),
}


@pytest.mark.parametrize("prefix", list(BUDGET))
def test_registers(kernels, prefix):  # noqa: F811
    most, spills = BUDGET[prefix]
    found = [n for n in kernels if n.startswith(prefix)]
    assert found
    for name in found:
        md = kernels[name]
        # vgpr_count is of the whole register file, accumulation registers included
        assert int(md.get("vgpr_count", 0)) <= most, (name, md["vgpr_count"])
        assert int(md.get("vgpr_spill_count", 0)) <= spills, (name, md["vgpr_spill_count"])
