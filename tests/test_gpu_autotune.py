"""fmm_autotune chooses between whole sub-grids and parts of them by timing both, as it
chooses the configuration; the results are the same bits either way."""
import numpy as np
import pytest

import synth
from paper_2304_11002_amd import fmm

from _gpu_helpers import ensure_library
from _profile import kernels_of

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


@pytest.mark.parametrize("prec", [fmm.FMM_FP64, fmm.FMM_FP64_HARMONIC])
@pytest.mark.parametrize("n", [1, 90, 256, 300])
def test_autotune_times_whole_subgrids_and_parts(torch, prec, n):
    ensure_library()
    rng = np.random.default_rng([81, n])
    desc, m_el, l_el = fmm.make_descriptors(rng.integers(2, 5, n), np.zeros(n, int),
                                            [synth.random_mask(rng) for _ in range(n)])
    M = torch.randn(m_el, dtype=torch.float64, device="cuda")
    outs = [torch.full((l_el,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(4)]
    with fmm.Context(0) as ctx:
        ctx.m2l(desc, M, outs[0], prec)
        timed = kernels_of(torch, lambda: ctx.autotune(desc, M, outs[1], prec))
        assert sum("m2l_fwd_whole_kernel" in k for k in timed) == 4        # a warm-up and three
        assert sum("m2l_fwd_part_kernel" in k for k in timed) == 4
        # the choice holds for -1 only
        used = kernels_of(torch, lambda: ctx.m2l(desc, M, outs[2], prec))
        ctx.set_option(fmm.FMM_OPT_ROUND_SPLIT, 0)
        whole = kernels_of(torch, lambda: ctx.m2l(desc, M, outs[3], prec))
    # one sub-grid, and 44 in a second turn of the compute units, are twice as fast in parts
    # and more; per-wave kernels, over whole sub-grids, cannot be the fastest there
    assert len(used) == 1 and "m2l_fwd_" in used[0]
    if n in (1, 300):
        assert "m2l_fwd_part_kernel" in used[0]
    if "m2l_fwd_part_kernel" in used[0]:
        assert len(whole) == 1 and "m2l_fwd_whole_kernel" in whole[0]
    for got in outs[1:]:
        assert torch.equal(got, outs[0])
