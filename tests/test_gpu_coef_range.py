"""The flux coefficients C4, C4 - e^{-s} and C2/dt at the ends of their argument's range:
against 60-digit values, for both signs, and their limits at infinity."""
import mpmath as mp
import numpy as np
import pytest

from paper_2312_16981_amd import ugkwp

pytestmark = pytest.mark.gpu


def _exact(s):
    s = mp.mpf(float(s))
    c4 = (1 - mp.exp(-s)) / s
    return c4, c4 - mp.exp(-s), (2 * c4 - 1 - mp.exp(-s)) / s


def test_coefficients_over_the_whole_range():
    """2e-15: at s = 1 and 2, where the closed forms take over, C4 - e^{-s} and 2 C4 - 1 - e^{-s}
    lose a factor 3.7 (0.264 of terms of 0.632 and 0.368; 0.27 of 0.865, 1 and 0.135), some
    9 and 12 times 2^-53 with an exponential of two roundings and a quotient of one, and a
    negative argument adds an exponential and two products."""
    a = np.concatenate([np.geomspace(1e-12, 600.0, 400), [1.0, 2.0, np.nextafter(1.0, 0), np.nextafter(2.0, 0)]])
    s = np.concatenate([a, -a, [1e16, 1e100, 1e300, 1.7e308]])
    got = ugkwp.eval_coef(s)
    with mp.workdps(60):
        for q, v in enumerate(s):
            for g, x in zip(got, _exact(v)):
                assert abs(mp.mpf(float(g[q])) - x) <= 2e-15 * abs(x) + mp.mpf(5e-324), (v, g[q])


def test_limits_at_infinity_and_nan():
    c4, w, c2 = ugkwp.eval_coef(np.array([np.inf, np.nan, 0.0]))
    assert (c4[0], w[0], c2[0]) == (0.0, 0.0, 0.0)
    assert np.isnan([c4[1], w[1], c2[1]]).all()
    assert (c4[2], w[2], c2[2]) == (1.0, 0.0, 0.0)
