"""The one-launch step (P2M and M2L) and the one-launch adjoints, on batches whose plan
takes them: every test asserts that the single kernel ran. Against the two launches bit
for bit, and sampled sub-grids against the oracle."""
import numpy as np
import pytest

import oracle as O
import synth
from paper_2304_11002_amd import fmm

from _gpu_helpers import ensure_library, moment_abs_scale, split_views
from _plans import adjoint_plan, stream_plan
from _profile import kernels_of

pytestmark = pytest.mark.gpu
TOL = 1e-12
PPC = 8
ROWS = np.zeros((24, 24, 24), bool)          # [z][y][x]: rows (y, z) in [2, 22)^2, every x
ROWS[2:22, 2:22, :] = True

# two of one order for every compute unit, all full or half of them with absent blocks;
# and orders, spacings and masks mixed, so that the next sub-grid differs from this one
CASES = [(2, False), (3, False), (4, False), (2, True), (3, True), (4, True), (0, True)]


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


@pytest.fixture(scope="module")
def ctx(torch):
    ensure_library()
    c = fmm.Context(0)
    yield c
    c.close()


def _batch(torch, p, uneven):
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    n = 2 * ncu if p else ncu * 1100 // 256
    rng = np.random.default_rng([n, p, 1, 5])
    ps = np.full(n, p) if p else rng.integers(2, 5, n)
    masks = [synth.random_mask(rng) if uneven and (not p or b % 2) else fmm.FULL_MASK for b in range(n)]
    lh = rng.integers(0, 3, n) if uneven else np.zeros(n, int)
    desc, m_el, l_el = fmm.make_descriptors(ps, lh, masks, PPC)
    g = torch.Generator(device="cuda")
    g.manual_seed(17 + p)
    cell = torch.arange(fmm.NCELL, device="cuda")
    corner = torch.stack((cell % 24, cell // 24 % 24, cell // 576), 1).double().repeat_interleave(PPC, 0)
    pos = torch.empty(n, fmm.NCELL * PPC, 3, dtype=torch.float64, device="cuda")
    for b in range(n):
        pos[b] = (corner + torch.rand(corner.shape, dtype=torch.float64, device="cuda", generator=g)) * 2.0 ** -int(lh[b])
    mass = torch.rand(n, fmm.NCELL, PPC, dtype=torch.float64, device="cuda", generator=g)
    return desc, m_el, l_el, pos, mass, ncu


def _picks(desc):
    return sorted({int(np.flatnonzero(desc["p"] == p)[k]) for p in set(desc["p"].tolist()) for k in (0, -1)})


def _host(pos, mass, b):
    return pos[b].reshape(fmm.NCELL, PPC, 3).cpu().numpy(), mass[b].cpu().numpy()


def _args(desc, b):
    return int(desc["p"][b]), 2.0 ** -int(desc["log2_inv_h"][b]), int(desc["mask"][b])


@pytest.mark.parametrize("p,uneven", CASES)
@pytest.mark.parametrize("prec", [fmm.FMM_FP64, fmm.FMM_FP64_HARMONIC])
def test_one_launch_step(ctx, torch, prec, p, uneven):
    desc, m_el, l_el, pos, mass, ncu = _batch(torch, p, uneven)
    harm = prec == fmm.FMM_FP64_HARMONIC
    assert stream_plan(desc, harm, ncu)[1]
    nan = lambda n: torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")
    M1, L1, M2, L2 = nan(m_el), nan(l_el), nan(m_el), nan(l_el)
    ctx.set_option(fmm.FMM_OPT_P2M_WINDOW, 1)
    ctx.p2m(desc, pos, mass, PPC, M1)
    ctx.set_option(fmm.FMM_OPT_P2M_WINDOW, 0)
    ctx.m2l(desc, M1, L1, prec)
    names = kernels_of(torch, lambda: ctx.p2m_m2l(desc, pos, mass, PPC, M2, L2, prec))
    assert len(names) == 1 and "m2l_fwd_whole_kernel<%s, true>" % str(harm).lower() in names[0], names
    assert bool(torch.isfinite(L2).all()) and torch.equal(L1, L2)
    # the moments' bits, and nothing written outside the rows (NaN as it was)
    assert torch.equal(M1.view(torch.int64), M2.view(torch.int64))
    L3 = nan(l_el)
    ctx.p2m_m2l(desc, pos, mass, PPC, M2, L3, prec)   # the counter as the first launch left it
    assert torch.equal(L3, L2)
    Lh = L2.cpu().numpy()
    for b in _picks(desc):
        q, h, mask = _args(desc, b)
        hp, hm = _host(pos, mass, b)
        Mo = O.p2m(hp, hm, q, h, mask)
        Lb = split_views(Lh, desc[b:b + 1], "L")[0]
        assert (np.abs(Lb - O.m2l(Mo, q, h, mask)) <= TOL * O.m2l_abs(Mo, q, h, mask)).all(), b
        o = int(desc["m_off"][b])
        Mb = M2[o:o + Mo.size].cpu().numpy().reshape(Mo.shape)
        assert (np.abs(Mb - Mo)[:, ROWS] <= 1e-13 * moment_abs_scale(hp, hm, q, h, mask)[:, ROWS]).all(), b
        assert np.isnan(Mb[:, ~ROWS]).all()


@pytest.mark.parametrize("p,uneven", CASES)
@pytest.mark.parametrize("form", [0, 1])
def test_one_launch_adjoints(ctx, torch, form, p, uneven):
    desc, m_el, l_el, pos, mass, ncu = _batch(torch, p, uneven)
    assert adjoint_plan(desc, bool(form), ncu)[1]
    g = torch.Generator(device="cuda")
    g.manual_seed(23)
    dL = torch.randn(l_el, dtype=torch.float64, device="cuda", generator=g)
    nan = lambda t: torch.full_like(t, float("nan"))
    M1 = torch.full((m_el,), float("nan"), dtype=torch.float64, device="cuda")
    M2, d1, d2, d3 = nan(M1), nan(mass), nan(mass), nan(mass)
    ctx.set_option(fmm.FMM_OPT_ADJOINT_FORM, form)
    try:
        ctx.m2l_backward(desc, dL, M1)
        ctx.p2m_backward(desc, pos, PPC, M1, d1)
        names = kernels_of(torch, lambda: ctx.m2l_p2m_backward(desc, pos, PPC, dL, M2, d2))
        assert torch.equal(M1, M2) and torch.equal(d1, d2)
        ctx.m2l_p2m_backward(desc, pos, PPC, dL, M2, d3)
        torch.cuda.synchronize()
    finally:
        ctx.set_option(fmm.FMM_OPT_ADJOINT_FORM, 0)
    assert len(names) == 1 and "m2l_bwd_kernel<%s, true>" % ("true" if form else "false") in names[0], names
    assert torch.equal(d3, d2)
    dLh = dL.cpu().numpy()
    for b in _picks(desc):
        q, h, mask = _args(desc, b)
        hp, _ = _host(pos, mass, b)
        W = split_views(dLh, desc[b:b + 1], "L")[0]
        Go, Ga = O.m2l_adjoint(W, q, h, mask), O.m2l_adjoint_abs(W, q, h, mask)
        o = int(desc["m_off"][b])
        assert (np.abs(M2[o:o + Go.size].cpu().numpy().reshape(Go.shape) - Go) <= TOL * Ga).all(), b
        go = O.p2m_adjoint(hp, Go, q, h, mask)
        c = O.cell_centres(h)[:, None, :]
        assert (np.abs(d2[b].cpu().numpy() - go) <= TOL * O.p2m_adjoint(c + np.abs(hp - c), Ga, q, h, mask)).all(), b
