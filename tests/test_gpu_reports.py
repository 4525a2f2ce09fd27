"""Reports of the pseudo-time loops as the host takes them: every loop of a long
run of small sims ends with each sim stopped (a report, or its stop flag, taken
before all of it has arrived in host memory would end a loop early), and the
counts repeat from run to run. Single sims, batches with and without the tail
launch, and the chunked loop."""
import pytest

from paper_1904_00861_amd import dtsph as D
from paper_1904_00861_amd import inputs as I

from gpu_helpers import banner

pytestmark = pytest.mark.gpu

KINDS = {
    "single": (lambda: I.tgv2d(16, seed=3), {}),
    "single_chunks": (lambda: I.tgv2d(16, seed=3), {D.OPT_CHUNK: 3}),
    "batch": (lambda: [I.tgv2d(14, seed=1), I.cavity(8), I.tgv2d(18, seed=2)], {}),
    "batch_no_tail": (lambda: [I.tgv2d(14, seed=1), I.cavity(8), I.tgv2d(18, seed=2)], {D.OPT_TAIL_LOOP: 0}),
}


@pytest.mark.parametrize("kind", list(KINDS))
def test_every_loop_runs_to_its_stop(kind):
    make, opts = KINDS[kind]
    banner(f"loop reports {kind}")
    seen = []
    for _ in range(20):
        sim = D.Sim(make(), precision=D.FP32)
        for k, v in opts.items():
            sim.set_option(k, v)
        _, reps = sim.step(40)
        sim.close()
        assert all(r["reason"] in (1, 2, 3) for step in reps for r in step)
        seen.append([[(r["iters"], r["reason"], r["rp_mean"], r["rv_mean"], r["pairs"]) for r in step]
                     for step in reps])
    assert all(s == seen[0] for s in seen)
