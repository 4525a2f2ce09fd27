"""One wavefront per cell as a setting of its own (neighbour-build lanes 64): every
lane count that the autotuner reports can be set on a context again, and the forced
kernel's exact lists equal the brute-force oracle, also for the sims that it leaves
to the lanes-per-particle kernel (a periodic axis with too few cells, a grid with
more cells than particles)."""
import math

import numpy as np
import pytest

import oracle as O
from paper_1904_00861_amd import dtsph as D
from paper_1904_00861_amd import inputs as I

from gpu_helpers import banner

pytestmark = pytest.mark.gpu


def short_axis(prob, div):
    """Does a periodic axis have fewer than 2 div + 3 cells (so that the cell kernel
    does not take the sim)?"""
    p = prob.params
    kh = p["kappa"] * p["h"]
    span = [p["hi"][a] - p["lo"][a] for a in range(p["dim"]) if p["periodic"][a]]
    skin = min([(0.25 if p["shift"] else 0.3) * p["h"]] + [0.5 * (0.5 * s - kh) for s in span])
    cells = [math.floor(s / ((kh + skin) / div * (1 + 1e-6))) for s in span]
    return any(n < 2 * div + 3 for n in cells)


CASES = {
    "tgv2d_30": (lambda: I.tgv2d(30, seed=3, jitter=0.3), False),
    "tgv3d_12": (lambda: I.tgv3d(12, seed=4, jitter=0.3), False),
    "tgv3d_8": (lambda: I.tgv3d(8, seed=4, jitter=0.3), True),
    "dam_0.05": (lambda: I.dam_break(0.05), False),
}


@pytest.mark.parametrize("case", list(CASES))
def test_forced_cell_kernel_lists(case):
    make, short = CASES[case]
    prob = make()
    banner(f"one wavefront per cell, forced: lists {case}")
    assert short_axis(prob, 2) == short
    ob, ib = O.neighbors(prob.params, prob.n_fluid, prob.n_wall, prob.x, "brute")
    sim = D.Sim(prob, precision=D.FP32)
    sim.set_option(D.OPT_NBR_LANES, 64)
    off, idx = sim.neighbor_list()
    sim.close()
    assert np.array_equal(off, ob) and np.array_equal(idx, ib)


@pytest.mark.parametrize("make", [lambda: I.tgv3d(14, seed=2), lambda: I.cavity(24), lambda: I.dam_break(0.04)])
def test_tuned_shape_can_be_set_again(make):
    prob = make()
    banner(f"tuned shape set again {prob.name}")
    a = D.Sim(prob, precision=D.FP32)
    rep = a.autotune(repeats=1)
    a.close()
    b = D.Sim(prob, precision=D.FP32)
    b.set_option(D.OPT_LANES, rep["lanes"])
    b.set_option(D.OPT_BLOCK, rep["block"])
    b.set_option(D.OPT_CELL_DIV, rep["cell_div"])
    b.set_option(D.OPT_NBR_LANES, rep["nbr_lanes"])
    b.set_option(D.OPT_NBR_LANES, 64)  # which of them it reports is a matter of timing
    b.set_option(D.OPT_NBR_TILES, rep["nbr_tiles"])
    b.set_option(D.OPT_FILTER_LANES, rep["filter_lanes"])
    st, _ = b.step(2)
    for bad in (16, 32, 65, 128):
        with pytest.raises(D.DtsphError):
            b.set_option(D.OPT_NBR_LANES, bad)
    b.close()
    assert st >= 0
