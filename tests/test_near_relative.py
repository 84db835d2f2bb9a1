"""The near-pair rational (csrc/mds_coeffs.h) against mpmath in relative error,
and the sum of -ln Phi as the FP64 kernels carry it -- E = prod(1/Phi) - 1,
closed by ln(1 + E) -- restated in numpy."""
import mpmath as mp
import numpy as np
import pytest

from tests.test_coeffs import ARR, _horner, _max_rel

U = 2.0 ** -53


def _ratio(t):
    return (_horner(ARR["kNearP64"], t, np.float64).astype(np.longdouble) /
            _horner(ARR["kNearQ64"], t, np.float64).astype(np.longdouble))


def test_near_ratio_relative_error():
    # Horner's rule on positive coefficients at t >= 0: one rounding a step
    # (8 and 9 steps) and one of each coefficient, and the fit's own 2^-56
    assert all(c > 0 for c in ARR["kNearP64"] + ARR["kNearQ64"])
    t = np.linspace(0.0, 9.0, 901)
    assert _max_rel(_ratio(t), lambda v: mp.erfc(v / mp.sqrt(2)) * mp.exp(v * v / 2) / 2,
                    t) < 20 * U


def _log1p_product(E):
    g = 1.0 + E
    h, n = np.frexp(g)
    low = h < np.sqrt(0.5)
    f, n = np.where(low, 2 * h, h), n - low
    s = np.where(n == 0, E, f - 1.0) / (f + 1.0)
    return 2 * s * _horner(ARR["kAtanhA64"], s * s, np.float64) + n * np.log(2.0)


@pytest.mark.parametrize("lo,hi", [(0.0, 0.01), (0.0, 9.0), (4.0, 5.0), (7.0, 9.0)])
def test_sum_of_small_terms(lo, hi):
    # 256 pairs: x = e P/Q within 22 u (the rational, e) and t^2/2 u of e's
    # argument taken as exact here; each step of E adds at most 4 roundings
    # relative to 1 + E, a sum of one logarithm each in the mean
    rng = np.random.default_rng(3)
    t = rng.uniform(lo, hi, (256, 8))
    q = (np.exp(-0.5 * t.astype(np.longdouble) ** 2) * _ratio(t.ravel()).reshape(t.shape)).astype(float)
    E = np.zeros(8)
    for k in range(0, 256, 2):
        ua, ub = q[k] / (1 - q[k]), q[k + 1] / (1 - q[k + 1])
        u = ua + ub + ua * ub
        E = E + u + E * u
    got = _log1p_product(E)
    for c in range(8):
        ref = -mp.fsum(mp.log1p(-mp.erfc(mp.mpf(v) / mp.sqrt(2)) / 2) for v in t[:, c])
        assert abs(got[c] - ref) <= (30 + 4 * 128) * U * ref
