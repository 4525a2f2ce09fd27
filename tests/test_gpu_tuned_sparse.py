"""A tuned launch shape is kept per process and applied to later contexts of the same
kind, but one wavefront per cell is only taken where cells hold particles: a filled
3D box is tuned, then a context of the same size in a mostly empty domain builds its
lists in the time of the automatic choice (mostly empty wavefronts take several
times as long)."""
import numpy as np
import pytest

from paper_1904_00861_amd import dtsph as D
from paper_1904_00861_amd import inputs as I

from gpu_helpers import banner

pytestmark = pytest.mark.gpu

N = 36


def _sparse():
    # the same particles in the middle of a box of 5 x 5 x 5 their volume, not periodic
    prob = I.tgv3d(N, seed=3)
    prob.params.update(periodic=(0, 0, 0), lo=(-2.0,) * 3, hi=(3.0,) * 3)
    return prob


def _build_ms(sim):
    best = np.inf
    for _ in range(4):
        sim.set_option(D.OPT_RESET_TIMING, 0)
        for _ in range(5):
            sim.set_state_from_problems()
            sim.build_cells()
        t = sim.timing()
        best = min(best, t["build_ms"] / t["build_launches"])
    return best


def test_sparse_context_after_a_tuned_filled_one():
    banner("tuned 3D box, then a sparse domain of the same size")
    a = D.Sim(I.tgv3d(N, seed=3), precision=D.FP32)
    rep = a.autotune(repeats=3)
    a.close()
    sim = D.Sim(_sparse(), precision=D.FP32)
    assert sim.info["n_cells"] > 2 * sim.info["n"]
    sim.set_option(D.OPT_TIMING, 1)
    tuned = _build_ms(sim)
    sim.set_option(D.OPT_NBR_LANES, 0)
    auto = _build_ms(sim)
    sim.set_option(D.OPT_NBR_LANES, 64)
    cells = _build_ms(sim)
    sim.close()
    print(f"[gpu-time] tuned nbr_lanes {rep['nbr_lanes']}: full build {1e3 * tuned:.1f} us as created, "
          f"{1e3 * auto:.1f} us automatic, {1e3 * cells:.1f} us one wavefront per cell", flush=True)
    # as created: the automatic choice or lanes that were tuned, never wavefronts per cell
    assert tuned < 0.5 * (auto + cells)
