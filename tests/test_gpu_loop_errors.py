"""Errors found inside a pseudo-time loop while further launches of it are still in
flight: the context takes a new state afterwards, and steps from it as a fresh
context does. Single sims keep a second group of iterations in flight; chunked
loops and batches leave nothing behind."""
import numpy as np
import pytest

from paper_1904_00861_amd import dtsph as D
from paper_1904_00861_amd import inputs as I

from gpu_helpers import banner

pytestmark = pytest.mark.gpu


def _moving(n, seed):
    prob = I.tgv2d(n, seed=seed, jitter=0.05)
    prob.params = dict(prob.params, move=2)
    return prob


def _same(a, b):
    assert all(np.array_equal(a[k], b[k]) for k in a)


@pytest.mark.parametrize("prec", [D.FP64, D.FP32])
@pytest.mark.parametrize("kind", ["single", "single_chunks", "batch"])
def test_state_set_after_a_skin_error_is_accepted(kind, prec):
    banner(f"state set after a skin error, {kind} precision {prec}")
    probs = [_moving(30, 5)] + ([_moving(20, 6)] if kind == "batch" else [])
    fresh = D.Sim(probs, precision=prec)
    fresh.step(2)
    want = fresh.get_state()
    fresh.close()
    sim = D.Sim(probs, precision=prec)
    if kind == "single_chunks":
        sim.set_option(D.OPT_CHUNK, 3)
    for _ in range(3):
        sim.set_option(D.OPT_SKIN, 0)  # every iteration leaves the skin
        with pytest.raises(D.DtsphError) as e:
            sim.step(1)
        assert e.value.status == D.EOVERFLOW
        sim.set_option(D.OPT_SKIN, 1000)
        sim.set_state_from_problems()
        sim.step(2)
        _same(sim.get_state(), want)
        sim.set_state_from_problems()
        sim.set_option(D.OPT_SKIN, 0)
        sim.predict()
        with pytest.raises(D.DtsphError) as e:
            sim.pseudo_iterate(12)
        assert e.value.status == D.EOVERFLOW
        sim.set_option(D.OPT_SKIN, 1000)
        sim.set_state_from_problems()
        sim.step(2)
        _same(sim.get_state(), want)
        sim.set_state_from_problems()
    sim.close()
