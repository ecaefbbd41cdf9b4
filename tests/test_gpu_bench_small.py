"""The bench's small batches: what it reports as whole sub-grids and as planned are
different kernels (one sub-grid in parts takes about a tenth of the whole one's time)."""
import pytest

from paper_2304_11002_amd import fmm

from _gpu_helpers import ensure_library
from _profile import kernels_of

pytestmark = pytest.mark.gpu


def test_small_batches_are_measured_both_ways():
    import torch
    import bench
    ensure_library()
    res = {}
    with fmm.Context(0) as ctx:
        names = kernels_of(torch, lambda: res.update(bench.bench_small(torch, fmm, ctx, 3, 1)))
        assert ctx.get_option(fmm.FMM_OPT_ROUND_SPLIT) == -1
    assert any("m2l_fwd_whole_kernel" in k for k in names) and any("m2l_fwd_part_kernel" in k for k in names)
    one, small = res["single_subgrid"], res["small_uneven_batch"]
    assert one["whole_subgrid_step_ms_median"] > 2 * one["step_ms_median"] > 0
    assert small["whole_subgrids_m2l_ms"] > small["m2l_ms"] > 0 and small["autotuned_m2l_ms"] > 0
