"""fmm_m2l_noalloc depends on nothing that an earlier call left in its static device
array: calls that overlapped may leave any value in the work counter, and only
those calls may be wrong. Here the whole array is overwritten before the call."""
import ctypes
import subprocess

import numpy as np
import pytest

import synth
from paper_2304_11002_amd import fmm

from _gpu_helpers import ensure_library

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


def _fill_static_array(lib, byte):
    # the array's host-side name is a local symbol: found in the symbol table, at
    # its distance from an exported function
    at = {}
    for line in subprocess.check_output(["nm", "-S", fmm.LIB_PATH], text=True).splitlines():
        f = line.split()
        if f[-1] in ("_ZL7scratch", "fmm_create"):
            at[f[-1]] = (int(f[0], 16), int(f[1], 16))
    base = ctypes.cast(lib.fmm_create, ctypes.c_void_p).value - at["fmm_create"][0]
    host, size = at["_ZL7scratch"]
    dev = ctypes.c_void_p()
    assert lib.hipGetSymbolAddress(ctypes.byref(dev), ctypes.c_void_p(base + host)) == 0
    assert size >= 40 * fmm.NOALLOC_MAX_SUBGRIDS
    assert lib.hipMemset(dev, ctypes.c_int(byte), ctypes.c_size_t(size)) == 0
    assert lib.hipDeviceSynchronize() == 0


def _batch(torch, n):
    rng = np.random.default_rng([61, n])
    desc, m_el, l_el = fmm.make_descriptors(rng.integers(2, 5, n), rng.integers(0, 3, n),
                                            [synth.random_mask(rng) for _ in range(n)])
    return desc, torch.from_numpy(rng.standard_normal(m_el)).to("cuda"), l_el


# 1 sub-grid: parts without the counter; 150: parts with it; 600: whole sub-grids
@pytest.mark.parametrize("n", [1, 150, 600])
@pytest.mark.parametrize("prec,cfg", [(fmm.FMM_FP64_HARMONIC, -1), (fmm.FMM_FP64, -1), (fmm.FMM_FP64, 3),
                                      (fmm.FMM_SPLIT_FP32, -1)])
def test_noalloc_after_any_contents_of_the_static_array(torch, prec, cfg, n):
    lib = ensure_library()
    desc, M, l_el = _batch(torch, n)
    want = torch.full((l_el,), float("nan"), dtype=torch.float64, device="cuda")
    with fmm.Context(0) as ctx:
        ctx.set_option(fmm.FMM_OPT_TILE_CONFIG, cfg)
        ctx.m2l(desc, M, want, prec)
        _fill_static_array(lib, 1)     # a counter far past any work list
        got = torch.full_like(want, float("nan"))
        ctx.m2l_noalloc(desc, M, got, prec)
        torch.cuda.synchronize()
    assert bool(torch.isfinite(want).all())
    assert torch.equal(got, want)


def test_noalloc_streamed_after_per_wave_calls(torch):
    # the per-wave configurations leave the counter at the numbers they drew
    ensure_library()
    desc, M, l_el = _batch(torch, 300)
    outs = []
    with fmm.Context(0) as ctx:
        for cfg in (3, -1, 5, -1):
            ctx.set_option(fmm.FMM_OPT_TILE_CONFIG, cfg)
            outs.append(torch.full((l_el,), float("nan"), dtype=torch.float64, device="cuda"))
            ctx.m2l_noalloc(desc, M, outs[-1])
        torch.cuda.synchronize()
    assert bool(torch.isfinite(outs[0]).all())
    for got in outs[1:]:
        assert torch.equal(got, outs[0])
