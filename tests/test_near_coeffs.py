"""The FP64 sweep's near-pair tables (csrc/mds_coeffs.h) against mpmath: the
weighted rational erfcx(t/sqrt 2)/2 ~ P/Q on [0, 9] and 2^f on |f| <= 1/2,
evaluated as the kernel evaluates them."""
import mpmath as mp
import numpy as np

from tests.test_coeffs import ARR, _horner, _max_rel


def test_near_ratio_absolute_error_under_its_weight():
    # fit 2.2e-17, plus the roundings of P and Q (2 ulp each, 4.5e-16 of a
    # value of at most 1/2)
    t = np.linspace(0.0, 9.0, 901)
    got = (_horner(ARR["kNearP64"], t, np.float64).astype(np.longdouble) /
           _horner(ARR["kNearQ64"], t, np.float64).astype(np.longdouble))
    assert ARR["kNearQ64"][0] == 1.0
    q = [mp.erfc(mp.mpf(float(v)) / mp.sqrt(2)) / 2 for v in t]
    e = [mp.exp(-mp.mpf(float(v)) ** 2 / 2) for v in t]
    err = max(abs(mp.mpf(str(g)) * w - v) for g, w, v in zip(got, e, q))
    assert err < 2.5e-16


def test_exp2_polynomial():
    f = np.linspace(-0.5, 0.5, 701)
    assert ARR["kExp2C64"][0] == 1.0
    assert _max_rel(_horner(ARR["kExp2C64"], f, np.float64), lambda v: mp.mpf(2) ** v, f) < 4.5e-16
