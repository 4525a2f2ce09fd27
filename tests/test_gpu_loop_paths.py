"""The launches between two pair passes, at the sizes where their form changes.

Residual reduction: a sim's tiles fill one segment (256 tiles), two to four (one
workgroup takes them all) or more (an arrival count); the reports agree with those
of the same passes cut into fewer tiles, the state is the same bits. Wall pass:
four lanes per wall particle, lists shorter and longer than one round of gathers.
Loop of a single sim: groups of iterations in flight ahead of the reports against
chunks with a wait after each, same bits."""
import numpy as np
import pytest

from paper_1904_00861_amd import dtsph as D
from paper_1904_00861_amd import inputs as I

from gpu_helpers import banner, oracle_steps, rel_l2

pytestmark = pytest.mark.gpu


def _with(prob, **kw):
    prob = prob.copy()
    prob.params = dict(prob.params, **kw)
    return prob


def _loop(prob, prec, block, fixed):
    sim = D.Sim(prob, precision=prec)
    try:
        sim.set_option(D.OPT_LANES, 8)
        sim.set_option(D.OPT_BLOCK, block)
        sim.predict()
        _, reps = sim.pseudo_iterate(fixed)
        sim.correct()
        return reps[0], sim.get_state()
    finally:
        sim.close()


# tiles of 8 particles: 254 (one segment), 265, 512 (two), 1013 (four), 1036 (five)
@pytest.mark.parametrize("n", [45, 46, 64, 90, 91])
@pytest.mark.parametrize("kind,prec", [("tgv2d", D.FP64), ("tgv2d", D.FP32), ("cavity", D.FP64)])
def test_residual_segments(kind, prec, n):
    banner(f"residual segments {kind} {n}^2 precision {prec}")
    prob = I.tgv2d(n, seed=n) if kind == "tgv2d" else I.cavity(n)
    a, ga = _loop(prob, prec, 64, 4)
    b, gb = _loop(prob, prec, 256, 4)
    for f in ga:
        assert np.array_equal(ga[f], gb[f]), f
    # the same terms in another grouping: at most one rounding per term
    tol = n * n * 2.0 ** -53
    assert a["iters"] == b["iters"] == 4 and a["pairs"] == b["pairs"]
    assert a["rp_max"] == b["rp_max"] and a["rv_max"] == b["rv_max"]
    assert abs(a["rp_mean"] - b["rp_mean"]) <= tol * b["rp_mean"]
    assert abs(a["rv_mean"] - b["rv_mean"]) <= tol * b["rv_mean"]


TOL = {D.FP64: dict(v=1e-10, p=1e-11, x=1e-12), D.FP32: dict(v=1e-5, p=1e-4, x=1e-7)}


# fluid neighbours of a wall particle: up to about 14, 25 and 40
@pytest.mark.parametrize("hdx", [1.0, 1.4, 1.8])
@pytest.mark.parametrize("prec", [D.FP64, D.FP32])
def test_wall_pass_rounds(prec, hdx):
    prob = I.cavity(18)
    dx = 1.0 / 18
    prob = _with(prob, h=hdx * dx)
    banner(f"wall pass rounds h = {hdx} dx precision {prec}")
    sim = D.Sim(prob, precision=prec)
    try:
        sim.predict()
        sim.pseudo_iterate(4)
        sim.correct()
        g = sim.get_state()
    finally:
        sim.close()
    x, v, vp, p, _, _ = oracle_steps(prob, 1, 4)
    nf, t = prob.n_fluid, TOL[prec]
    assert rel_l2(g["v"][:nf], v[:nf]) <= t["v"]
    assert rel_l2(g["p"][:nf], p[:nf]) <= t["p"]
    assert rel_l2(g["x"], x) <= t["x"]


CASES = {
    "tgv2d_30": lambda: I.tgv2d(30, seed=5),
    "tgv3d_8": lambda: I.tgv3d(8, seed=3),
    "dam_0.05": lambda: I.dam_break(0.05),
    "cavity_steady_16": lambda: I.cavity(16, steady=True),
    "tgv2d_24_move": lambda: _with(I.tgv2d(24, seed=6), move=2),
    "tgv2d_24_shift": lambda: _with(I.tgv2d(24, seed=6, jitter=0.1), shift=1),
}


@pytest.mark.parametrize("prec", [D.FP64, D.FP32])
@pytest.mark.parametrize("case", list(CASES))
def test_groups_in_flight_match_chunks(case, prec):
    banner(f"groups in flight against chunks {case} precision {prec}")
    got = []
    for chunk in (0, 3):
        sim = D.Sim(CASES[case](), precision=prec)
        try:
            if chunk:
                sim.set_option(D.OPT_CHUNK, chunk)
            _, reps = sim.step(4)
            sim.predict()
            _, fixed = sim.pseudo_iterate(130)  # groups of 64 iterations
            sim.correct()
            got.append((reps, fixed, sim.get_state()))
        finally:
            sim.close()
    assert got[0][0] == got[1][0] and got[0][1] == got[1][1]
    assert got[0][1][0]["iters"] == 130
    for f in got[0][2]:
        assert np.array_equal(got[0][2][f], got[1][2][f]), f
