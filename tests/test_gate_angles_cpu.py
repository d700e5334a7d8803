"""Sine and cosine of the gate tables, over the reduction's ranges: quarter
turns, both sides of the octants, both sides of 2^20 radians (where the
library's reduction takes over) and non-finite angles.  The bound is half a
unit in the last place of 1 (5.6e-17) plus the roundings of the correction
term (|y^3 / 6| < 0.081 and |y^4 / 24 ..| < 0.02 at three to four of 2^-53 each,
3.4e-17)."""
import numpy as np
import pytest

from paper_2003_02989_amd import tq
from paper_2003_02989_amd.circuits import OPS

BOUND = 9.0e-17 + 1e-19
EIGHTHS = [k / 8 for k in range(-17, 18)]


@pytest.mark.parametrize("scale", [1.0, 64.0, 2.0**19, 2.0**20, 2.0**21 + 2.0**-20, 1e12])
def test_radians(scale):
    rng = np.random.default_rng(int(scale) % 1000)
    for v in [scale, -scale, np.nextafter(scale, 0)] + list(scale * rng.uniform(-2, 2, 400)):
        m, _ = tq.gate_matrix(OPS["RX"][0], [2.0 * v])
        x = np.longdouble(v)
        assert abs(np.longdouble(m[0, 0].real) - np.cos(x)) < BOUND, v
        assert abs(np.longdouble(-m[1, 0].imag) - np.sin(x)) < BOUND, v


@pytest.mark.parametrize("scale", [1.0, 64.0, 2.0**20, 2.0**40])
def test_half_turns(scale):
    rng = np.random.default_rng(int(scale) % 1000)
    pi = np.longdouble("3.14159265358979323846264338327950288")
    for v in EIGHTHS + [np.nextafter(e, 9) for e in EIGHTHS] + list(scale * rng.uniform(-2, 2, 400)):
        m, _ = tq.gate_matrix(OPS["ZPOW"][0], [v])
        x = np.longdouble(v - 2.0 * np.rint(v / 2.0)) * pi
        assert abs(np.longdouble(m[1, 1].real) - np.cos(x)) < BOUND, v
        assert abs(np.longdouble(m[1, 1].imag) - np.sin(x)) < BOUND, v
    for k in range(-8, 9):  # exact at the quarter turns
        m, _ = tq.gate_matrix(OPS["ZPOW"][0], [0.5 * k])
        assert m[1, 1] == [1, 1j, -1, -1j][k % 4]


@pytest.mark.parametrize("v", [np.inf, -np.inf, np.nan])
def test_non_finite(v):
    for op in ("RX", "ZPOW"):
        m, _ = tq.gate_matrix(OPS[op][0], [v])
        assert np.isnan(m[1, 1].real)
    assert tq.gate_matrix(OPS["ZPOW"][0], [v])[0][0, 0] == 1
