"""Order of the neighbour lists of the kernel with one wavefront per cell, forced
(neighbour-build lanes 64) on sims that it takes itself: FP32 sums follow the list
order, so steps agree bit for bit with the lanes-per-particle kernel. 2D and 3D,
periodic images across every axis, walls, particles beyond the grid, cells with
more particles than one batch and lists longer than the kernel's LDS rows, and a
batch that mixes them with a sim left to the other kernel."""
import numpy as np
import pytest

from paper_1904_00861_amd import dtsph as D
from paper_1904_00861_amd import inputs as I

from gpu_helpers import banner
from test_gpu_nbr_cell_option import short_axis

pytestmark = pytest.mark.gpu


def _walled_3d(n):
    # the 3D vortex in a closed box: three layers of wall particles on every side
    prob = I.tgv3d(n, seed=9, jitter=0.2)
    dx = 1.0 / n
    k = (np.arange(n + 6) - 2.5) * dx
    g = np.stack(np.meshgrid(k, k, k, indexing="ij"), axis=-1).reshape(-1, 3)
    wall = g[((g < 0) | (g > 1)).any(axis=1)]
    prob.params.update(periodic=(0, 0, 0), lo=(-3 * dx,) * 3, hi=(1 + 3 * dx,) * 3)
    zero = np.zeros((len(wall), 3))
    prob.x = np.concatenate([prob.x, wall])
    prob.v = np.concatenate([prob.v, zero])
    prob.v_prev = np.concatenate([prob.v_prev, zero])
    prob.p = np.concatenate([prob.p, np.zeros(len(wall))])
    prob.n_wall = len(wall)
    return prob


def _dense(prob, share, at, box):
    # a share of the particles squeezed into a box: tens of them per cell
    d = prob.params["dim"]
    k = np.arange(int(prob.n * share))
    x = prob.x[k, :d]
    prob.x[k, :d] = at + box * (x - x.min(axis=0)) / np.ptp(x, axis=0).max()
    prob.params.update(max_neighbors=1600, dt=prob.params["dt"] * 1e-3, max_iter=4)
    return prob


def _beyond(prob):
    prob.x[0, :2] = [1.3, 0.5]  # the grid ends at -0.25 and 1.25
    prob.x[1, :2] = [1.31, 0.51]
    prob.x[2, :2] = [-0.3, 0.5]
    prob.x[3, :2] = [0.5, 1.4]
    prob.x[4, :2] = [1.4, 1.4]
    return prob


CASES = {
    "tgv2d_30": lambda: I.tgv2d(30, seed=3, jitter=0.3),
    "tgv3d_18": lambda: I.tgv3d(18, seed=4, jitter=0.3),
    "walled_3d_10": lambda: _walled_3d(10),
    "channel": lambda: I.poiseuille(ny=20, nx=24),
    "cavity_24": lambda: I.cavity(24),
    "beyond": lambda: _beyond(I.cavity(24)),
    "dense_2d": lambda: _dense(I.tgv2d(30, seed=5), 0.4, 0.4, 0.2),
    "dense_3d": lambda: _dense(I.tgv3d(18, seed=5), 0.15, 0.4, 0.15),
}


def _steps(probs, lanes, div):
    sim = D.Sim(probs, precision=D.FP32)
    try:
        sim.set_option(D.OPT_CELL_DIV, div)
        sim.set_option(D.OPT_NBR_TILES, 0)
        sim.set_option(D.OPT_NBR_LANES, lanes)
        sim.predict()
        _, reps = sim.pseudo_iterate(4)
        first = sim.get_state(loop=True)
        sim.correct()
        sim.step(2)
        return reps, first, sim.get_state()
    finally:
        sim.close()


def _agree(a, b):
    assert a[0] == b[0]
    for ga, gb in zip(a[1:], b[1:]):
        for k in ga:
            assert np.array_equal(ga[k], gb[k], equal_nan=True), k
            assert np.isfinite(ga[k]).all(), k


@pytest.mark.parametrize("div", [1, 2, 3])
@pytest.mark.parametrize("case", list(CASES))
def test_order_of_the_cell_kernel(case, div):
    prob = CASES[case]()
    banner(f"list order, one wavefront per cell: {case} cell subdivision {div}")
    assert not short_axis(prob, div)  # the sim is the cell kernel's
    _agree(_steps(prob, 64, div), _steps(prob, 1, div))


def test_order_in_a_batch_with_a_short_axis():
    banner("list order, one wavefront per cell: batch with a short-axis member")
    probs = [I.tgv2d(30, seed=1), I.tgv2d(7, seed=2, jitter=0.2), I.cavity(16), I.tgv2d(24, seed=3)]
    assert [short_axis(p, 2) for p in probs] == [False, True, False, False]
    _agree(_steps(probs, 64, 2), _steps(probs, 2, 2))
