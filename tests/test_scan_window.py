"""The rule that limits the tabulated scan of a one-cell node to a window of the
table (scan_window in csrc/dpo_search.h), on the CPU: the first minimum of
all tabulated evaluations, formed in float32 as the kernel forms them, lies in
the window wherever the rule gives one -- over smooth, steep, nearly flat,
cancelling and degenerate coefficients, and for tables from 8 to 1024 angles.
"""
import numpy as np
import pytest

f32 = np.float32
K_WINDOW = 24


def fma(a, b, c):
    # the product of two float32 is exact in float64; one rounding there, one here
    return (np.asarray(a, np.float64) * np.asarray(b, np.float64) + np.asarray(c, np.float64)).astype(f32)


def evaluations(x, y, z, w, g1, g2, d1, d2, K):
    """The float32 Q of every tabulated angle (K x n)."""
    u = -np.pi + 2.0 * np.pi * np.arange(K) / K
    q = np.empty((K, x.size), f32)
    for k in range(K):
        sn, cs = f32(np.sin(u[k])), f32(np.cos(u[k]))
        dv, dt = fma(g1, sn, d1) - d1, fma(g2, cs, d2) - d2
        q[k] = fma(fma(w, dt, y), dv, fma(z, dt, x))
    return q


def window(x, y, z, w, g1, g2, d1, d2, K):
    """First entry and number of entries of the rule's window (0: none)."""
    y0 = np.nextafter(f32(1.0 - np.cos(np.pi / K)), f32(4.0))
    step = f32(K / (2.0 * np.pi))
    b, c = y * g1, z * g2
    P, Q = np.abs(w) * g2 + np.abs(y), np.abs(w) * g1 + np.abs(z)
    with np.errstate(all="ignore"):
        top = (P * g1 + (Q * g2 + np.abs(x))).astype(f32)
        ulp = ((top.view(np.int32) & 0x7f800000).view(f32) * f32(1.1920929e-7)).astype(f32)
        E = f32(1.05) * (f32(0.5) * np.abs(w) * g1 * g2
                         + (f32(5.9604645e-8) * (P * (f32(6) * g1 + np.abs(d1)) + Q * (f32(6) * g2 + np.abs(d2))) + ulp))
        R = np.sqrt(b * b + c * c)
        h = f32(0.5) * y0 + E / R
        ok = (R > 1e-18) & (R < 1e18) & (h <= 1)
        s = np.sqrt(np.where(ok, h, 0))
        wid = f32(2) * step * (s * (f32(0.5708) * h + f32(1))) + f32(0.02)
        kc = np.arctan2(b, c).astype(f32) * step
        lo = np.ceil(kc - wid)
        n = np.floor(kc + wid) - lo + 1
        ok &= (n <= K_WINDOW) & (n <= K)
    flat = (y == 0) & (z == 0) & (w == 0)
    n = np.where(flat, 1, np.where(ok, np.nan_to_num(n), 0)).astype(int)
    return np.where(flat, 0, np.nan_to_num(lo)).astype(int), n


def coefficients(kind, n, rng):
    g1, g2 = (f32(rng.uniform(1e-4, 0.45, n)) for _ in range(2))
    d1, d2 = (f32(rng.uniform(-4, 4, n)) for _ in range(2))
    size = {"steep": 2.0, "mixed": None, "flat": -3.0, "one_axis": None, "cross": None, "large_value": 1.0}[kind]
    scale = 10.0 ** (rng.uniform(-4, 3, n) if size is None else rng.uniform(size - 1, size + 1, n))
    x = f32(rng.uniform(-1, 1, n) * 10.0 ** rng.uniform(-2, 3.2, n))
    y, z, w = (f32(rng.normal(size=n) * scale) for _ in range(3))
    if kind == "one_axis":
        (y if rng.random() < 0.5 else z)[:] = 0
        w[:] = 0
    if kind == "cross":
        y[:], z[:] = y * f32(1e-3), z * f32(1e-3)
    if kind == "large_value":
        x = f32(x * 1e3)
    return x, y, z, w, g1, g2, d1, d2


@pytest.mark.parametrize("kind", ["steep", "mixed", "flat", "one_axis", "cross", "large_value"])
@pytest.mark.parametrize("K", [8, 16, 64, 72, 257, 1024])
def test_window_holds_the_first_minimum(kind, K):
    rng = np.random.default_rng(K)
    n = 20000 if K < 200 else 4000
    c = coefficients(kind, n, rng)
    first = evaluations(*c, K).argmin(axis=0)
    lo, count = window(*c, K)
    inside = (first - lo) % K < count
    assert np.all(inside | (count == 0))
    if kind in ("steep", "one_axis") and K < 200:
        assert (count > 0).mean() > 0.5  # the rule is not vacuous


def test_degenerate_coefficients():
    one = np.ones(1, f32)
    z = 0 * one
    g = f32(0.02) * one
    # a plateau: one entry, the table's first
    assert window(7 * one, z, z, z, g, g, one, one, 64) == (0, 1)
    # no slope, a cross term only; non-finite or huge coefficients: no window
    for y, zz, w in ((z, z, one), (one * np.inf, one, z), (one * np.nan, one, z), (f32(3e30) * one, one, z)):
        assert window(one, y, zz, w, g, g, one, one, 64)[1] == 0
