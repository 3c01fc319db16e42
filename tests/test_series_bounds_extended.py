"""The truncation bounds of the path lengths' extended series and of the H
pass, on the CPU against the constants in the sources (a range or order there
that the stated bounds no longer cover fails here).

The terms a series drops are summed at the end of its range, with every power
moment at its largest against T_2 = <g, x^2> (|T_k|, |P_k|, |N_k| <= X^(k-2)
T_2) and the path length near 2, to first order in what they change:

* alpha_Higher = c / b with c ~ T_2, b ~ T_2 / 2 - (2/15) aL Bp
  (lattice.hpp, ExtendedCfg): 2 dc / T_2 + 4 (2/15) aL dBp / T_2, and alpha_Lower
  2 dc1 / T_2;
* the mirror condition's root (MirrorSeriesCfg, MirrorExtendedCfg): dG / G',
  G' = T_2 / 2 up to a tenth of it at the extended range's end.
"""
import pathlib
import re
from fractions import Fraction

import pytest

CSRC = pathlib.Path(__file__).resolve().parents[1] / "paper_2203_12946_amd" / "csrc"
LATTICE = (CSRC / "lattice.hpp").read_text()
TERMS = 60


def _cfg(name, t):
    m = re.search(r"struct %s<%s> \{\s*static constexpr int K = (\d+);\s*static constexpr double X = ([0-9.]+);"
                  % (name, t), LATTICE)
    return int(m.group(1)), float(m.group(2))


def _taylor(num, den):
    """Taylor coefficients of num / den (ascending integer coefficients)."""
    c = []
    for n in range(TERMS):
        v = Fraction(num[n]) if n < len(num) else Fraction(0)
        v -= sum(Fraction(den[j]) * c[n - j] for j in range(1, min(n, len(den) - 1) + 1))
        c.append(v / den[0])
    return c


C1 = _taylor([2], [2, 1])
C = _taylor([60, 60, 11], [60, 90, 36, 3])
R = _taylor([80, 80, 19], [64, 96, 44, 6])


def _array(name):
    body = re.search(r"constexpr double %s\[\d+\] = \{(.*?)\};" % name, LATTICE, re.S).group(1)
    return [eval(v, {}, {}) for v in body.replace("\n", " ").split(",")]  # literals and quotients of literals


@pytest.mark.parametrize("name,exact", [("kC1", C1), ("kC", C), ("kR", R)])
def test_coefficients(name, exact):
    got = _array(name)
    assert len(got) >= 10
    for g, e in zip(got, exact):
        assert abs(g - float(e)) <= 2.0 ** -52 * abs(float(e)), (name, g, e)


@pytest.mark.parametrize("t,bound", [("float", 2.5e-8), ("double", 1.1e-15)])
def test_extended_closed_form(t, bound):
    K, X = _cfg("ExtendedCfg", t)
    aL = 2.0 + X / 3  # its first-order end: 2 + T_3 / (3 T_2)
    dc1 = sum(abs(float(C1[k - 2])) * X ** (k - 2) for k in range(K + 1, TERMS))
    dc = sum(abs(float(C[k - 2])) * X ** (k - 2) for k in range(K + 1, TERMS))
    dbp = sum(abs(float(R[m])) * aL ** m * X ** (m + 1) for m in range(K - 2, TERMS))
    assert 2 * dc1 < bound
    assert 2 * dc + 4 * (2.0 / 15.0) * aL * dbp < bound, 2 * dc + 4 * (2.0 / 15.0) * aL * dbp


@pytest.mark.parametrize("name,t,bound", [
    ("MirrorSeriesCfg", "float", 1.2e-8), ("MirrorSeriesCfg", "double", 6e-16),
    ("MirrorExtendedCfg", "float", 6e-8), ("MirrorExtendedCfg", "double", 6e-16)])
def test_mirror_series(name, t, bound):
    K, X = _cfg(name, t)
    dG = sum(X ** (k - 2) / (k - 1) * (2.0 ** (k - 1) / k - 1) for k in range(K + 1, TERMS))
    Gp = 0.5 if name == "MirrorSeriesCfg" else 0.45
    assert dG / Gp < bound, dG / Gp


def test_h_series():
    """log(v / w) = 2 atanh(z) to z^41 for |z| <= 0.375, relative to itself."""
    s = (CSRC / "eselbm_step.hip").read_text()
    last = int(re.search(r"double s = 1\.0 / (\d+)\.0;", s).group(1))
    lo, hi = re.search(r"v >= float\(([\d./ ]+)\) \* w && v <= ([\d.]+)f \* w", s).groups()
    lo = float(lo.split("/")[0]) / float(lo.split("/")[1])
    z = max((1 - lo) / (1 + lo), (float(hi) - 1) / (float(hi) + 1))
    assert abs(z - 0.375) < 1e-6
    assert z ** (last + 1) / (last + 2) / (1 - z * z) < 1e-18
