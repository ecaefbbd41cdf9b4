"""Plans of batches with absent blocks (host only): a sub-grid's time depends little on
its mask, so a batch of one order that fits the compute units is not thought uneven."""
import os

import numpy as np
import pytest

import synth
from paper_2304_11002_amd import fmm

if not os.path.exists(fmm.LIB_PATH):
    pytest.skip("libfmm.so is not built", allow_module_level=True)

from _plans import adjoint_plan, sorted_items, stream_plan

CENTRE = 1 << 13


def _batch(n, p, uneven=True):
    # seven of ten with random blocks absent, the others full, as timed
    rng = np.random.default_rng([n, p, 1])
    masks = [synth.random_mask(rng) if uneven and rng.random() < 0.7 else fmm.FULL_MASK for _ in range(n)]
    return fmm.make_descriptors(np.full(n, p), np.zeros(n, int), masks)[0]


@pytest.mark.parametrize("n", [208, 224, 240, 250, 256])
def test_uneven_forward_of_second_order_runs_whole(n):
    # harmonic p = 2, whole and in parts: 520 to 526 us and 547 to 565
    assert not stream_plan(_batch(n, 2), True)[0]


@pytest.mark.parametrize("p,n", [(3, 240), (3, 250), (3, 256), (4, 240), (4, 250), (4, 256)])
def test_uneven_harmonic_adjoint_runs_whole(p, n):
    # whole and by rounds: p = 3 1412 to 1427 us and 1456 to 1464, p = 4 3331 to 3342 and 3636 to 3761
    assert not adjoint_plan(_batch(n, p), True)[0]


@pytest.mark.parametrize("p", [2, 3, 4])
@pytest.mark.parametrize("harmonic", [False, True])
def test_few_and_badly_dividing_batches_are_cut(p, harmonic):
    # one, and a second turn of the compute units for 44: parts and rounds (twice as fast and more)
    for n, uneven in ((1, False), (300, False), (300, True)):
        assert stream_plan(_batch(n, p, uneven), harmonic)[0], n
        assert adjoint_plan(_batch(n, p, uneven), harmonic)[0], n


def test_costs_follow_measured_times():
    for harmonic in (False, True):
        d = fmm.make_descriptors([3, 3, 4, 2], [0] * 4, [fmm.FULL_MASK, CENTRE, CENTRE, fmm.FULL_MASK])[0]
        for adjoint in (False, True):
            it = sorted_items(d, harmonic, adjoint)
            cost = dict(zip(it["sub"].tolist(), it["part"].tolist()))
            assert it["part"].tolist() == sorted(it["part"].tolist(), reverse=True)
            # the centre block alone: 0.75 of the forward's time, 1.1 of the adjoint's
            lo, hi = (1.05, 1.2) if adjoint else (0.6, 0.8)
            assert lo <= cost[1] / cost[0] <= hi
            assert cost[2] > cost[0] > cost[3]
