"""GPU: the power law's deflection where it is hardest to interpolate, seen
through a source so steep that 1e-12 of the deflection shows: one masked pixel,
one sub-pixel, whose ray lands 1e-10 arcsec from the centre of an n = 4 source."""
import math

import numpy as np
import pytest

import oracle
from gpu_cases import say
from test_deflection_tables import LD, epl_series

pytestmark = pytest.mark.gpu
NPX, DPIX, TE, RS, N = 33, 0.125, 1.3, 0.3, 4.0
R_OFF = 1e-10          # arcsec
DEFL = 1e-13           # relative error of the deflection allowed: rsq_nr's 2e-14 in both
                       # direction components, amplified up to 3 times by the table's slope


def _ray(x, y, q, t):
    """alpha at (x, y) of a power law at the origin, phi = 0, in 80 bits."""
    X1, X2 = LD(q) * LD(x), LD(y)
    R = np.sqrt(X1 * X1 + X2 * X2)
    re, im = epl_series(np.array([X1 / R]), np.array([X2 / R]), q, t, 400)
    b = LD(TE) * np.sqrt(LD(q))
    mag = 2 * b ** LD(t) / (1 + LD(q)) * R ** (1 - LD(t))
    return mag * re[0], mag * im[0]


# the series (the most terms short of the cap, few, one group) and the table, slopes up to the steepest
@pytest.mark.parametrize("gamma", [2.0, 2.4, 2.95])
@pytest.mark.parametrize("q", [0.16, 0.29, 0.3, 0.35, 0.5, 1.0])
def test_power_law_next_to_a_steep_source(q, gamma):
    from paper_2503_08586_amd import binding
    say("case: power law, q %g, gamma %g, n = 4 source %g arcsec away" % (q, gamma, R_OFF))
    orc = oracle.default()
    bn = orc.bn(N)
    mid = (NPX - 1) // 2
    worst = 0.0
    with binding.LensContext(0) as c:
        for i, j in [(1, 8), (2, 10), (3, 9), (1, 14), (-2, 11), (4, 8), (0, 9), (-5, 13)]:
            x, y = i * DPIX, j * DPIX
            ax, ay = _ray(x, y, q, gamma - 1.0)
            p = np.zeros(20)
            p[[0, 1, 8, 9, 10]] = TE, q, 0.5, 1.0, 1.0
            p[[12, 13, 14, 15]] = 1.0, RS, N, 1.0
            p[17], p[18] = float(LD(x) - ax - LD(R_OFF) * LD(0.6)), float(LD(y) - ay - LD(R_OFF) * LD(0.8))
            p[19] = gamma
            r = float(np.hypot(LD(x) - ax - LD(p[17]), LD(y) - ay - LD(p[18])))
            want = orc.sersic(1.0, RS, N, bn, 1.0, 0.0, 0.0, 0.0, r, 0.0)
            mask = np.zeros((NPX, NPX), np.uint8)
            mask[mid + j, mid + i] = 1
            sigma = np.full((NPX, NPX), 0.25)
            lid = binding.lens_load_data(c.ctx, NPX, NPX, DPIX, 1, np.ones((1, 1)), np.zeros((NPX, NPX)), sigma, mask,
                                         mass_model=binding.LENS_MASS_EPL)
            got = math.sqrt(2.0 * (c.info(lid)["norm"] - c.loglike(lid, p[None])[0])) * 0.25
            c.unload(lid)
            # d ln I / d ln r = -(b / n) (r / R)^(1/n); 5e-7: the pixel and the exponent in FP32
            slope = bn / N * (r / RS) ** (1.0 / N)
            tol = slope * DEFL * float(np.hypot(ax, ay)) / r + 5e-7
            worst = max(worst, abs(got / want - 1.0) / tol)
            assert abs(got / want - 1.0) <= tol, (i, j, got / want - 1.0, tol)
    say("worst %.2f of the tolerance" % worst)
