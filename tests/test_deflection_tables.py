"""The per-proposal deflection tables as the device builds and reads them
(lens_device.h: table_node, table_poly, ray_trace_tab, pow_setup), in FP64 numpy
from the constants in the sources: polynomials in v = u NI - j from j = 0 up, an
entry past the last interval for u = 1, for the power law coefficients from
differences to a middle node, and its power of the radius from mantissa and
exponent tables.  The power law against its series in 80-bit numbers, the SIE
against the oracle's closed form."""
import os
import re

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2503_08586_amd", "csrc")
LD = np.longdouble
MAX_SLOPE = 1.95   # t = gamma - 1 of the steepest accepted slope


def _src(name):
    with open(os.path.join(CSRC, name)) as f:
        return f.read()


def _const(fname, name):
    m = re.search(r"\b%s\s*=\s*([-+0-9.eE]+)" % name, _src(fname))
    assert m, (fname, name)
    return float(m.group(1))


def _array(name):
    m = re.search(r"\b%s\[[^=]*=\s*\{(.*?)\};" % name, _src("lens_approx.h"), re.S)
    assert m, name
    return np.array([float(v) for v in re.findall(r"[-+0-9.eE]+(?=\s*[,}])", m.group(1) + ",")])


def epl_series(c, s, q, t, terms):
    """e^(i phi) sum_n a_n e^(2 i n phi) at e^(i phi) = c + i s (Tessore & Metcalf
    2015), in the precision of c and s."""
    one = c.dtype.type(1)
    f = (one - c.dtype.type(q)) / (one + c.dtype.type(q))
    a = [one]
    for n in range(1, terms):
        a.append(-f * (2 * n - 2 + c.dtype.type(t)) / (2 * n + 2 - c.dtype.type(t)) * a[-1])
    wr, wi = c * c - s * s, 2 * c * s
    sr, si = np.full_like(c, a[-1]), np.zeros_like(c)
    for n in range(terms - 2, -1, -1):
        sr, si = sr * wr - si * wi + a[n], sr * wi + si * wr
    return c * sr - s * si, c * si + s * sr


class Table:
    """The table of one proposal from the node values f(u, s) -> (T1, T2)."""

    def __init__(self, name, nodes_of):
        self.NI = int(_const("lens_internal.h", "k%sIntervals" % name))
        deg = int(_const("lens_approx.h", "k%sDeg" % name))
        node = _array("k%sNode" % name)
        M = _array("k%sInterp" % name).reshape(deg + 1, deg + 1)
        j = np.arange(self.NI)
        u = (j[:, None] + 0.5 + node) * (1.0 / self.NI)
        self.coef = []
        for f in nodes_of(u, np.sqrt((1 - u) * (1 + u))):
            mid = (deg + 1) // 2 if name == "Epl" else None
            ref = f[:, mid] if mid is not None else 0.0
            c = np.zeros((self.NI + 1, deg + 1))
            for k in range(deg + 1):
                if k != mid:
                    c[:-1] += M[:, k] * (f[:, k] - ref)[:, None]
            c[:-1, 0] += ref
            for i in range(deg):
                for k in range(deg - 1, i - 1, -1):
                    c[:-1, k] -= 0.5 * c[:-1, k + 1]
            c[-1, 0] = c[-2].sum()
            self.coef.append(c)

    def eval(self, c, s):
        un = np.abs(c) * self.NI
        j = un.astype(int)
        assert j.max() <= self.NI
        v = un - j
        out = []
        for C, x in zip(self.coef, (c, s)):
            h = C[j, -1]
            for i in range(C.shape[1] - 2, -1, -1):
                h = h * v + C[j, i]
            out.append(x * h)
        return out


def _directions():
    rng = np.random.default_rng(5)
    th = np.concatenate([rng.uniform(0, 2 * np.pi, 6000), np.pi / 2 + 0.02 * rng.normal(size=3000),
                         0.02 * rng.normal(size=1000), [0.0, np.pi / 2, np.pi, 1.5 * np.pi]])
    return np.cos(th), np.sin(th)


def _worst(got, ref):
    d = np.hypot(*[(g - r).astype(float) for g, r in zip(got, ref)])
    return (d / np.hypot(*[r.astype(float) for r in ref])).max()


# from the table's first axis ratio up; the bound is the interpolation error at the
# nearest singularity (1.0e-15 at q = 0.3, t = 1.95) and some ten roundings
@pytest.mark.parametrize("t", [0.05, 1.0, 1.4, MAX_SLOPE])
@pytest.mark.parametrize("q", [0.3, 0.35, 0.4, 0.5, 0.7, 0.95, 1.0])
def test_power_law_table_is_as_good_as_the_series(q, t):
    assert q * q >= _const("lens_device.h", "kSieTabQ2") - 1e-12
    terms = 2 if q == 1.0 else min(128, int(np.ceil(np.log(1e-16) / np.log((1 - q) / (1 + q)))) + 1)

    def nodes(u, s):
        re, im = epl_series(u, s, q, t, terms)
        return re / u, im / s

    c, s = _directions()
    ref = epl_series(c.astype(LD), s.astype(LD), q, t, 400 if q < 0.6 else 120)
    assert _worst(Table("Epl", nodes).eval(c, s), ref) < 4e-15


@pytest.mark.parametrize("q,tol", [(0.3, 6e-11), (0.4, 1e-11), (0.5, 2e-12), (0.7, 2e-13), (0.95, 1e-13)])
def test_sie_table_in_its_present_form(q, tol):
    """With the node values at 64 bits (atan, atanh) against 80 bits: the
    interpolation errors of test_sie_table_reproduces_the_deflection."""
    ce = np.sqrt(LD(1) - LD(q) * LD(q))

    def funcs(u, s):
        e = u.dtype.type(ce)
        x = e * u / u.dtype.type(q)
        z = e * s
        return np.arctan(x) / u, (np.log1p(z) - np.log1p(-z)) / 2 / s

    c, s = _directions()
    keep = (np.abs(c) > 1e-9) & (np.abs(s) > 1e-9)
    c, s = c[keep], s[keep]
    ref = funcs(np.abs(c).astype(LD), np.abs(s).astype(LD))
    got = Table("Sie", funcs).eval(c, s)
    assert _worst(got, [x.astype(LD) * r for x, r in zip((c, s), ref)]) < tol


@pytest.mark.parametrize("name", ["Epl", "Sie"])
def test_entry_past_the_last_interval(name):
    """u = 1 (and some roundings above) reads the entry behind the last one."""
    tab = Table(name, lambda u, s: (1.0 + u * u, 2.0 - u))
    for one in (1.0, 1.0 + 2.0 ** -51):
        got = tab.eval(np.array([one, -one]), np.array([0.0, 0.0]))
        assert np.allclose(got[0], [2.0, -2.0], rtol=1e-14) and np.all(np.abs(got[1]) == 0.0)


@pytest.mark.parametrize("t", [0.05, 0.5, 1.0, 1.4, MAX_SLOPE])
def test_power_of_the_radius(t):
    """R^(1 - t) = (m/m_j)^h m_j^h 2^(E h), R^2 = m 2^E, h = (1 - t)/2, with the
    binomial series to fifth order: its next term (8e-16 at most) and some ten
    roundings."""
    bits = int(_const("lens_internal.h", "kPowMantBits"))
    n, E0 = 1 << bits, int(re.search(r"kPowE0 = (-?\d+)", _src("lens_device.h")).group(1))
    h = 0.5 * (1.0 - t)
    rng = np.random.default_rng(2)
    R2 = 2.0 ** rng.uniform(E0, 28, 20000)
    m, E = np.frexp(R2)
    j = (np.floor(m * 2 * n) - n).astype(int)
    mj = 0.5 + (j + 0.5) / (2 * n)
    x = m * (1.0 / mj) - 1.0
    b = [1.0]
    for i in range(5):
        b.append(b[-1] * (h - i) / (i + 1))
    pw = ((((b[5] * x + b[4]) * x + b[3]) * x + b[2]) * x + b[1]) * x + 1.0
    got = pw * mj ** h * 2.0 ** (E * h)
    ref = R2.astype(LD) ** LD(h)
    assert np.abs((got / ref - 1).astype(float)).max() < 4e-15
