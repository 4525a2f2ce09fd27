"""Timed launches while two groups of iterations are in flight: every iteration that
a loop's reports count is booked once with its pairs, launches past a loop's stop are
not, and timing changes no result. Chunked loops count the same."""
import numpy as np
import pytest

from paper_1904_00861_amd import dtsph as D
from paper_1904_00861_amd import inputs as I

from gpu_helpers import banner

pytestmark = pytest.mark.gpu

CASES = {
    "tgv2d_30": lambda: I.tgv2d(30, seed=5),
    "cavity_20": lambda: I.cavity(20),
    "steady_16": lambda: I.cavity(16, steady=True),
}


@pytest.mark.parametrize("chunk", [0, 3])
@pytest.mark.parametrize("case", list(CASES))
def test_every_iteration_is_booked_once(case, chunk):
    banner(f"timed launches {case} chunk {chunk}")
    prob = CASES[case]()
    prob.params.update(max_iter=40)
    out = []
    for timed in (0, 1):
        sim = D.Sim(prob, precision=D.FP32)
        sim.set_option(D.OPT_CHUNK, chunk)
        sim.set_option(D.OPT_TIMING, timed)
        sim.set_option(D.OPT_RESET_TIMING, 0)
        _, reps = sim.step(5)
        sim.predict()
        _, fixed = sim.pseudo_iterate(150)  # groups of 64
        sim.correct()
        t = sim.timing()
        out.append((reps, fixed, sim.get_state()))
        sim.close()
        loops = [r[0] for r in reps] + fixed
        if timed:
            assert t["pass_launches"] == sum(r["iters"] for r in loops)
            assert t["pass_pairs"] == sum(r["iters"] * r["pairs"] for r in loops)
            assert t["pass_particles"] == prob.n_fluid * t["pass_launches"]
            assert t["build_launches"] == t["full_builds"] and t["pass_ms"] > 0
        else:
            assert t["pass_launches"] == 0
    assert out[0][:2] == out[1][:2]
    for k in out[0][2]:
        assert np.array_equal(out[0][2][k], out[1][2][k]), k


def test_timed_loops_do_not_keep_events():
    # many loops with launches past their stops: counts stay exact to the end
    banner("timed launches over many loops")
    sim = D.Sim(I.tgv2d(16, seed=2), precision=D.FP32)
    sim.set_option(D.OPT_TIMING, 1)
    total = 0
    for _ in range(40):
        _, reps = sim.step(5)
        total += sum(r[0]["iters"] for r in reps)
    t = sim.timing()
    sim.close()
    assert t["pass_launches"] == total
