"""The constants of the FP64 walk's table-driven exp2 and log2 (csrc/wl_poly.h),
against mpmath at 40 digits: every table entry, and the steps of both functions,
the polynomials among them, carried out on the host with a fused multiply-add."""
from fractions import Fraction

import numpy as np
import pytest

from test_poly_header import coeffs, header

mp = pytest.importorskip("mpmath")

def test_tables():
    mp.mp.dps = 40
    e = coeffs(header(), "WL_EXP2_TAB")
    assert len(e) == 64
    assert e == [float(mp.power(2, mp.mpf(j) / 64)) for j in range(64)]
    t = coeffs(header(), "WL_LOG2_TAB")
    assert len(t) == 256
    for j in range(128):
        c, l = t[2 * j], t[2 * j + 1]
        assert c == float(1 / (1 + (mp.mpf(j) + mp.mpf(1) / 2) / 256))
        assert l == float(1 + mp.log(mp.mpf(c), 2))


def fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))


def hi_lo(x):
    b = int(np.float64(x).view(np.int64))
    return b >> 32, b & 0xFFFFFFFF


def from_hi_lo(hi, lo):
    return float(np.int64((hi << 32) | lo).view(np.float64))


def exp2_neg(t):
    """exp2_neg64 of the walk, step by step; returns (2^-t, the t it held)."""
    hi, lo = hi_lo(t)
    t = from_hi_lo(min(hi, 0x408FE000), lo)
    magic = 6755399441055744.0
    z = fma(-64.0, t, magic)
    n = np.int32(np.uint32(hi_lo(z)[1]))
    f = fma(z - magic, -0.015625, -t)
    assert abs(f) <= 1 / 128
    hi, lo = hi_lo(coeffs(header(), "WL_EXP2_TAB")[int(n) & 63])
    T = from_hi_lo(hi + ((int(n) >> 6) << 20), lo)
    c = coeffs(header(), "WL_EXP2M1_F64")
    p = c[-1]
    for k in c[-2::-1]:
        p = fma(p, f, k)
    return fma(T, f * p, T), t


def test_exp2_steps():
    """0.5 ulp of the last step and as much again for the table entry and the
    correction: 2^-52 in all, over the whole range, at the table's edges and on
    either side of them; beyond 1020 the value stays near 2^-1020."""
    mp.mp.dps = 40
    rng = np.random.default_rng(3)
    edges = (np.arange(0, 400) + 0.5) / 64
    ts = np.concatenate([[0.0, 1e-300, 2.0 ** -60], rng.uniform(0, 1020, 400),
                         rng.uniform(0, 3, 200), edges, np.nextafter(edges, 0),
                         np.nextafter(edges, 9), [1019.9999, np.nextafter(1020.0, 0), 1020.0]])
    for t in ts:
        got, held = exp2_neg(float(t))
        assert held == t
        want = mp.power(2, -mp.mpf(float(t)))
        assert abs(mp.mpf(got) - want) < mp.mpf(2) ** -52 * want, t
    for t in (1020.5, 1021.0, 1074.0, 1e6, 1e300, np.inf):
        got, held = exp2_neg(float(t))
        assert 1020.0 <= held < 1020.001
        assert 2.0 ** -1020.01 < got <= 2.0 ** -1020 * (1 + 1e-15) and held * got < 1e-303


def one_minus_log2(E):
    t, c = coeffs(header(), "WL_LOG2_TAB"), coeffs(header(), "WL_LOG2P1_F64")
    j = (hi_lo(1.0 + E)[0] >> 12) & 127
    r = fma(E, t[2 * j], t[2 * j] - 1.0)
    assert abs(r) <= 1 / 511, E
    p = c[-1]
    for k in c[-2::-1]:
        p = fma(p, r, k)
    return fma(-r, p, t[2 * j + 1])


def test_log2_steps():
    """1 - log2(1 + E) where 1 + E stays below 3/2 (the walk's E are below 0.37;
    values 0.415 to 1): the table entry's rounding, the correction's and the last
    step's, 2^-53 each."""
    mp.mp.dps = 40
    rng = np.random.default_rng(4)
    edges = np.arange(0, 128) / 256
    Es = np.concatenate([rng.uniform(0, 0.5, 400), 2.0 ** -rng.uniform(0, 1000, 200) / 2, edges,
                         np.nextafter(edges[1:], 0), np.nextafter(edges, 1),
                         [np.nextafter(0.5, 0)]])
    for E in Es[1.0 + Es < 1.5]:
        want = 1 - mp.log(1 + mp.mpf(float(E)), 2)
        assert abs(mp.mpf(one_minus_log2(float(E))) - want) < 3 * mp.mpf(2) ** -53, E
