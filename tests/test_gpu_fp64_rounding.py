"""The FP64 pair pass to the last bits: the pressure rate of one pseudo-iteration
against the same sums in 80-bit arithmetic, on the same float64 inputs and constants.

Tolerance, from the operations of one pair: its separation is exact or rounded once,
1/r and 1/(r^2 + eta h^2) are good to 1 ulp, and about 16 further roundings enter a
term; a rounding is at most 0.5 ulp and 0.29 ulp rms. The kernel's polynomial
15 t1^4 - 6 t2^4 + t3^4 is a sum of larger terms, so errors are measured against the
sums with all signs made positive (scale below). For n = 28 (2D) or 113 (3D) terms that
makes a worst case of (20 + n) 2^-53 per unit of scale. Independent roundings give
0.29 sqrt(20) 2^-52 rms per term and, over n terms of alternating sign and like size, that
divided by sqrt(n); the bar on the rms is 1.5 times it. An error common to all terms, as
of a reciprocal square root that is off by 2^-48, exceeds it.
"""
import numpy as np
import pytest

from paper_1904_00861_amd import dtsph as D
from paper_1904_00861_amd import inputs as I

from gpu_helpers import banner

pytestmark = pytest.mark.gpu

L = np.longdouble
EPS = 2.0 ** -52


def _reference(prm, x, v, p):
    """Pressure rate and its scale per particle (80-bit sums over all pairs in reach)."""
    d, h = prm["dim"], prm["h"]
    c, m, rho = prm["beta"] * prm["vref"], prm["mass"], prm["rho0"]
    sigma = 7.0 / (478.0 * np.pi * h * h) if d == 2 else 1.0 / (120.0 * np.pi * h * h * h)
    kg = -5.0 * sigma / h
    k_div, k_lap = c * c * m * kg, 4.0 * m / (2.0 * rho) * (h * c / 16.0) * kg
    inv_h, den = L(1.0 / h), L(prm["eta"] * h * h)
    x, v, p = x[:, :d].astype(L), v[:, :d].astype(L), p.astype(L)
    out, scale = np.zeros(len(x), L), np.zeros(len(x), L)
    for i in range(len(x)):
        r = x[i] - x
        r2 = (r * r).sum(axis=1)
        j = (r2 < L(prm["kappa"] * h) ** 2) & (np.arange(len(x)) != i)
        r, r2 = r[j], r2[j]
        rr = np.sqrt(r2)
        t = [np.maximum(L(k) - rr * inv_h, L(0)) for k in (3, 2, 1)]
        poly = L(15) * t[2] ** 4 - L(6) * t[1] ** 4 + t[0] ** 4
        big = L(15) * t[2] ** 4 + L(6) * t[1] ** 4 + t[0] ** 4
        # and what one ulp of q = r / h does to the polynomial (t^4 each)
        big = big + L(4) * rr * inv_h * (L(15) * t[2] ** 3 + L(6) * t[1] ** 3 + t[0] ** 3)
        w = v[i] - v[j]
        div, dp = ((w * r).sum(axis=1)) / rr, (p[i] - p[j]) * rr / (r2 + den)
        out[i] = L(k_div) * (poly * div).sum() + L(k_lap) * (poly * dp).sum()
        scale[i] = abs(L(k_div)) * (big * (np.abs(w * r).sum(axis=1)) / rr).sum() \
            + abs(L(k_lap)) * (big * np.abs(dp)).sum()
    return out, scale


@pytest.mark.parametrize("lanes", [1, 2, 8])
@pytest.mark.parametrize("dim", [2, 3])
def test_pressure_rate_is_rounded_only(dim, lanes):
    prob = I.tgv2d(22, seed=11, jitter=0.3) if dim == 2 else I.tgv3d(9, seed=11, jitter=0.3)
    banner(f"FP64 rounding dim {dim} lanes {lanes}")
    # not periodic: the separations are differences of the coordinates
    prob.params.update(periodic=(0, 0, 0), lo=(-1.0,) * 3, hi=(2.0,) * 3)
    rng = np.random.default_rng(17)
    v = prob.v.copy()
    v[:, :dim] += 0.1 * rng.standard_normal((prob.n, dim))
    p = prob.p + 0.1 * rng.standard_normal(prob.n)
    zero = np.zeros(prob.n)
    sim = D.Sim(prob, precision=D.FP64)
    sim.set_option(D.OPT_LANES, lanes)
    sim.set_state(prob.x, prob.v, prob.v_prev, p, dict(x_iter=prob.x, v_iter=v, p_iter=p, dpdtau=zero))
    sim.pseudo_iterate(1)
    got = sim.get_state(loop=True)["dpdtau"]
    sim.close()
    # the pass reads V = V^n + (V_iter - V^n): the same sum in float64
    want, scale = _reference(prob.params, prob.x, prob.v + (v - prob.v), p)
    err = np.abs(got.astype(L) - want) / scale
    worst, rms = float(err.max()), float(np.sqrt((err * err).mean()))
    n = 28 if dim == 2 else 113
    print(f"[gpu-err] FP64 rounding dim {dim} lanes {lanes}: worst {worst / EPS:.2f} rms {rms / EPS:.2f} x 2^-52",
          flush=True)
    assert worst <= (20 + n) * EPS / 2
    assert rms <= 1.5 * 0.29 * np.sqrt(20.0 / n) * EPS
