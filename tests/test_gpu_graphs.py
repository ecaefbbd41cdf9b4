"""The cached graphs (FMM_FP64, per-wave tile configurations), and the options that
earlier tests compare at their defaults: whole sub-grids against parts."""
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


def _batch(torch, seed, n):
    rng = np.random.default_rng([83, seed, n])
    desc, m_el, l_el = fmm.make_descriptors(rng.integers(2, 5, n), rng.integers(0, 3, n),
                                            [synth.random_mask(rng) for _ in range(n)])
    return desc, torch.from_numpy(rng.standard_normal(m_el)).to("cuda"), l_el


def _plain(torch, batch, cfg):
    desc, M, l_el = batch
    L = torch.full((l_el,), float("nan"), dtype=torch.float64, device="cuda")
    with fmm.Context(0) as ref:
        ref.set_option(fmm.FMM_OPT_USE_GRAPH, 0)
        ref.set_option(fmm.FMM_OPT_TILE_CONFIG, cfg)
        ref.m2l(desc, M, L)
        torch.cuda.synchronize()
    assert bool(torch.isfinite(L).all())
    return L


@pytest.mark.parametrize("cfg", [2, 3, 4, 5])
def test_graph_replays_of_per_wave_configurations(torch, cfg):
    ensure_library()
    batch = _batch(torch, 1, 5)
    desc, M, l_el = batch
    want = _plain(torch, batch, cfg)
    L = torch.empty_like(want)
    with fmm.Context(0) as ctx:
        ctx.set_option(fmm.FMM_OPT_TILE_CONFIG, cfg)
        for rep in range(4):
            L.fill_(float("nan"))
            ctx.m2l(desc, M, L)                         # captured at the first call, replayed then
            x = torch.ones(1000, device="cuda").sum()   # eager work between replays
            torch.cuda.synchronize()
            assert torch.equal(L, want), rep
            assert x.item() == 1000
        names = kernels_of(torch, lambda: ctx.m2l(desc, M, L))
    assert any("m2l_fwd_kernel" in k for k in names) and any("reset_counter_kernel" in k for k in names), names


def test_graph_and_set_eviction_over_two_streams(torch):
    # 12 descriptor sets (more than the 8 a context holds) and 24 graphs (more than the
    # 16 it keeps), enqueued alternately on two streams without host synchronisation:
    # evicting a set drops only its own graphs, and a released graph has finished
    ensure_library()
    sets = [_batch(torch, 10 + i, 3) for i in range(12)]
    want = [_plain(torch, b, 3) for b in sets]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [[torch.full_like(w, float("nan")) for w in want] for _ in range(2)]
    torch.cuda.synchronize()
    with fmm.Context(0) as ctx:
        ctx.set_option(fmm.FMM_OPT_TILE_CONFIG, 3)
        for r in range(2):
            for i, (desc, M, _) in enumerate(sets):
                ctx.m2l(desc, M, outs[r][i], stream=streams[(i + r) % 2])
        torch.cuda.synchronize()
        for r in range(2):
            for i in range(12):
                assert torch.equal(outs[r][i], want[i]), (r, i)
        # 18 graphs of 6 held sets on both streams: the least recently used are released
        extra = [[torch.full_like(w, float("nan")) for w in want[:6]] for _ in range(3)]
        for r in range(3):
            for i in range(6):
                ctx.m2l(sets[i][0], sets[i][1], extra[r][i], stream=streams[(i + r) % 2])
        torch.cuda.synchronize()
        for r in range(3):
            for i in range(6):
                assert torch.equal(extra[r][i], want[i]), (r, i)


@pytest.mark.parametrize("n", [9, 200, 257])
@pytest.mark.parametrize("prec", [fmm.FMM_FP64, fmm.FMM_FP64_HARMONIC])
def test_round_split_option_selects_the_kernel(torch, prec, n):
    # 0: whole sub-grids at any size; 1: parts, of at most 256; the same bits
    ensure_library()
    desc, M, l_el = _batch(torch, 40, n)
    L = {}
    with fmm.Context(0) as ctx:
        for opt, kernel in ((0, "m2l_fwd_whole_kernel"), (1, "m2l_fwd_part_kernel")):
            ctx.set_option(fmm.FMM_OPT_ROUND_SPLIT, opt)
            L[opt] = torch.full((l_el,), float("nan"), dtype=torch.float64, device="cuda")
            ctx.m2l(desc, M, L[opt], prec)               # (the first call also uploads)
            names = kernels_of(torch, lambda: ctx.m2l(desc, M, L[opt], prec))
            assert len(names) == 1
            if opt == 0 or n <= 256:
                assert kernel in names[0], (opt, names)
    assert bool(torch.isfinite(L[0]).all()) and torch.equal(L[0], L[1])


@pytest.mark.parametrize("rest", [1, 7])
def test_exact_slices_of_an_uneven_batch_with_a_short_last_turn(torch, rest):
    # whole sub-grids over full turns of the compute units, a few of the smallest in
    # halves: the bits of the same sub-grids in a batch that ends on a full turn
    ensure_library()
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    n = 2 * ncu + rest
    rng = np.random.default_rng([85, rest])
    desc, m_el, l_el = fmm.make_descriptors(rng.integers(2, 4, n), rng.integers(0, 3, n),
                                            [synth.random_mask(rng) for _ in range(n)])
    g = torch.Generator(device="cuda")
    g.manual_seed(rest)
    M = torch.randn(m_el, dtype=torch.float64, device="cuda", generator=g)
    L, Lw = (torch.full((l_el,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(2))
    with fmm.Context(0) as ctx:
        for rep in range(2):
            ctx.m2l(desc, M, L, fmm.FMM_EXACT_SLICE)
        ctx.m2l(desc[:2 * ncu], M, Lw, fmm.FMM_EXACT_SLICE)
        ctx.m2l(desc[rest:], M, Lw, fmm.FMM_EXACT_SLICE)     # (the rest of them, and the others again)
        torch.cuda.synchronize()
    assert bool(torch.isfinite(L).all()) and torch.equal(L, Lw)
