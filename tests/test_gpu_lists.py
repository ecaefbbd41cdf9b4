"""Work lists of a descriptor set: made by the first M2L or adjoint of a form, not by
calls that need none, and in time for a call under stream capture."""
import json

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


def _batch(torch, seed, n):
    rng = np.random.default_rng([71, seed, n])
    desc, m_el, l_el = fmm.make_descriptors(rng.integers(2, 5, n), rng.integers(0, 3, n),
                                            [synth.random_mask(rng) for _ in range(n)])
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return desc, torch.randn(m_el, dtype=torch.float64, device="cuda", generator=g), l_el


def _uploaded(torch, path, call):
    """Bytes copied to the device during call()."""
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    prof.export_chrome_trace(str(path))
    copies = [e for e in json.loads(path.read_text())["traceEvents"]
              if "memcpy" in str(e.get("cat", "")).lower() and "HtoD" in e.get("name", "").replace("HostToDevice", "HtoD")]
    assert copies and all("bytes" in e["args"] for e in copies), copies
    return sum(int(e["args"]["bytes"]) for e in copies)


def test_calls_without_lists_upload_descriptors_only(torch, tmp_path):
    # a new set's P2M, P2M adjoint and evaluation need its descriptors and the ids per
    # order: 44 bytes a sub-grid, and up to 256 of padding for each of four sections.
    # (The lists of 640 mixed sub-grids are several times that.)
    ensure_library()
    n = 640
    M = torch.zeros(35 * 13824 * n, dtype=torch.float64, device="cuda")
    L = torch.zeros(35 * 512 * n, dtype=torch.float64, device="cuda")
    pos = torch.rand(3 * n * 13824, dtype=torch.float64, device="cuda")
    mass = torch.rand(n * 13824, dtype=torch.float64, device="cuda")
    out = torch.empty(n * 4 * 512, dtype=torch.float64, device="cuda")
    with fmm.Context(0) as ctx:
        calls = [lambda d: ctx.p2m(d, pos, mass, 1, M), lambda d: ctx.p2m_backward(d, pos, 1, M, mass),
                 lambda d: ctx.evaluate(d, pos, mass, 1, L, out)]
        for i, call in enumerate(calls):
            rng = np.random.default_rng([72, i])
            desc, _, _ = fmm.make_descriptors(rng.integers(2, 5, n), rng.integers(0, 3, n),
                                              [synth.random_mask(rng) for _ in range(n)], 1)
            assert _uploaded(torch, tmp_path / ("t%d.json" % i), lambda: call(desc)) <= 44 * n + 4 * 256


@pytest.mark.parametrize("mode", ["thread_local", "global"])
@pytest.mark.parametrize("n", [3, 150, 600, 1100])       # (above 1024 the lists are allocated then)
def test_first_m2l_and_adjoint_of_a_set_under_capture(torch, n, mode):
    # the set is known from another call; its lists are made during the capture
    ensure_library()
    desc, M, l_el = _batch(torch, 1, n)
    dL = torch.randn(l_el, dtype=torch.float64, device="cuda")
    for prec, form in ((fmm.FMM_FP64, 0), (fmm.FMM_FP64_HARMONIC, 1)):
        with fmm.Context(0) as ref:
            ref.set_option(fmm.FMM_OPT_ADJOINT_FORM, form)
            L0, G0 = torch.empty(l_el, dtype=torch.float64, device="cuda"), torch.empty_like(M)
            ref.m2l(desc, M, L0, prec)
            ref.m2l_backward(desc, dL, G0)
            torch.cuda.synchronize()
        with fmm.Context(0) as ctx:
            ctx.set_option(fmm.FMM_OPT_ADJOINT_FORM, form)
            ctx.set_option(fmm.FMM_OPT_M2L_KERNEL, 1)
            L, G = torch.empty_like(L0), torch.empty_like(M)
            ctx.m2l(desc, M, L)                        # the reference kernel: no lists
            ctx.set_option(fmm.FMM_OPT_M2L_KERNEL, 0)
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, capture_error_mode=mode):
                ctx.m2l(desc, M, L, prec)
                ctx.m2l_backward(desc, dL, G)
            # an eager call before the first replay finds the lists on the device
            L1 = torch.full_like(L0, float("nan"))
            ctx.m2l(desc, M, L1, prec)
            torch.cuda.synchronize()
            assert torch.equal(L1, L0)
            for rep in range(3):
                L.fill_(float("nan"))
                G.fill_(float("nan"))
                graph.replay()
                torch.cuda.synchronize()
                assert torch.equal(L, L0) and torch.equal(G, G0), rep
                assert torch.ones(1000, device="cuda").sum().item() == 1000   # eager work between replays
            del graph
