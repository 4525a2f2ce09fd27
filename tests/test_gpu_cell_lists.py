"""The neighbour kernel with one wavefront per cell (the automatic choice in 3D and
for small 2D contexts): exact lists equal the brute-force oracle bit for bit where it can go
wrong (cells with more particles than one batch of 8, lists longer than its LDS rows,
candidates in many chunks of 64, walls, particles beyond the grid, periodic images in
every axis, a batch that mixes it with sims whose axes are too short for it), and the
order of the lists is that of the lanes-per-particle kernel: steps agree bit for bit.
The choice is the library's own here: sims with too few cells on a periodic axis at a
subdivision (the vortices at most) or more cells than particles (`beyond`) take the
lanes-per-particle kernel; test_gpu_cell_order.py forces the kernel on sims it takes."""
import numpy as np
import pytest

import oracle as O
from paper_1904_00861_amd import dtsph as D
from paper_1904_00861_amd import inputs as I

from gpu_helpers import banner

pytestmark = pytest.mark.gpu


def _dense(dim):
    # a patch with tens of particles per cell in a lattice that has a few
    prob = I.tgv2d(30, seed=5) if dim == 2 else I.tgv3d(12, seed=5)
    k = np.arange(prob.n // 3)
    d = prob.params["dim"]
    box = 0.25
    prob.x[k, :d] = 0.4 + box * (prob.x[k, :d] - prob.x[k, :d].min(axis=0)) / np.ptp(prob.x[k, :d], axis=0).max()
    prob.params["max_neighbors"] = 1200
    return prob


def _beyond():
    prob = I.dam_break(0.06)
    prob.x[0, :2] = [4.7, 1.0]
    prob.x[1, :2] = [4.75, 1.02]
    prob.x[2, :2] = [-0.7, 1.5]
    prob.x[3, :2] = [2.0, 4.4]
    return prob


CASES = {
    "dense_2d": lambda: _dense(2),
    "dense_3d": lambda: _dense(3),
    "beyond": _beyond,
    "tgv2d_11": lambda: I.tgv2d(11, seed=3, jitter=0.3),
    "tgv3d_9": lambda: I.tgv3d(9, seed=4, jitter=0.3),
    "channel": lambda: I.poiseuille(ny=12, nx=16),
    "cavity_13": lambda: I.cavity(13),
}


@pytest.mark.parametrize("div", [1, 2, 3])
@pytest.mark.parametrize("case", list(CASES))
def test_cell_kernel_lists(case, div):
    prob = CASES[case]()
    banner(f"one wavefront per cell: lists {case} cell subdivision {div}")
    ob, ib = O.neighbors(prob.params, prob.n_fluid, prob.n_wall, prob.x, "brute")
    sim = D.Sim(prob, precision=D.FP64)
    sim.set_option(D.OPT_CELL_DIV, div)
    sim.set_option(D.OPT_NBR_LANES, 0)
    off, idx = sim.neighbor_list()
    sim.close()
    assert np.array_equal(off, ob) and np.array_equal(idx, ib)


def test_cell_kernel_in_a_batch_with_short_axes():
    # the 7 x 7 vortex has fewer cells per axis than a block needs: the general kernel takes it
    probs = [I.tgv2d(20, seed=1), I.tgv2d(7, seed=2, jitter=0.2), I.cavity(9), I.tgv2d(24, seed=3)]
    banner("one wavefront per cell: batch with a short-axis member")
    sim = D.Sim(probs, precision=D.FP32)
    for s, prob in enumerate(probs):
        ob, ib = O.neighbors(prob.params, prob.n_fluid, prob.n_wall, prob.x, "brute")
        off, idx = sim.neighbor_list(s)
        assert np.array_equal(off, ob) and np.array_equal(idx, ib), s
    sim.close()


def test_cell_kernel_reports_overflow():
    banner("one wavefront per cell: capacity overflow")
    prob = _dense(2)
    prob.params["max_neighbors"] = 40
    sim = D.Sim(prob, precision=D.FP32)
    with pytest.raises(D.DtsphError) as e:
        sim.neighbor_list()
    sim.close()
    assert e.value.status == D.EOVERFLOW


@pytest.mark.parametrize("case", ["tgv2d_11", "tgv3d_9", "cavity_13", "beyond"])
def test_cell_kernel_keeps_list_order(case):
    prob = CASES[case]()
    banner(f"one wavefront per cell against lanes per particle, FP32 steps, {case}")
    out = []
    for lanes in (0, 2):
        sim = D.Sim(prob, precision=D.FP32)
        sim.set_option(D.OPT_NBR_LANES, lanes)
        sim.step(3)
        out.append(sim.get_state())
        sim.close()
    for k in out[0]:
        assert np.array_equal(out[0][k], out[1][k]), k
