"""The scan's window as the kernels form it (csrc/dpo_window.h, built for the host):
the first minimum over the window's entries, in the kernels' order across the
table's end, is the first minimum of all tabulated evaluations, value and entry -- with
exact root and reciprocal, and with both off by the error that the rule allows for,
up and down.  Coefficients as in the copy of the rule that test_scan_window.py
holds, with thrust displacements of either sign, minima at every entry of the
table and exact ties."""
import ctypes as C
import subprocess

import numpy as np
import pytest

from paper_2407_14675_amd import build
from tests.test_scan_window import coefficients

SOURCE = """
#include <cmath>
static float off = 0.0f;
static float root(float x) { return sqrtf(x) * (1.0f + off); }
static float recip(float x) { return (1.0f / x) * (1.0f + off); }
#define DPO_SQRT(x) root(x)
#define DPO_RCP(x) recip(x)
#include "dpo_window.h"

// f: g1, g2, d1, d2, x, y, z, w of the nodes, one after another.  Returns the number of
// nodes whose window's minimum is not the table's; windows: nodes that have one;
// widest, ends: the longest window, and windows across the table's end.
extern "C" int check(int n, const float* f, int K, float error, int* windows, int* widest, int* ends) {
  struct Angle { float x, y; };
  Angle tab[1024];
  for (int k = 0; k < K; k++) {
    const double u = -3.14159265358979323846 + 2.0 * 3.14159265358979323846 * (double)k / (double)K;
    tab[k] = {(float)std::sin(u), (float)std::cos(u)};
  }
  auto at = [&](int k) { return tab[k]; };
  off = error;
  int bad = 0;
  *windows = *widest = *ends = 0;
  for (int i = 0; i < n; i++) {
    const float* p = f + 8 * (size_t)i;
    const dpo::CellNode F{p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7]};
    int k0;
    const int m = dpo::scan_window(F, K, dpo::scan_y0_for(K), dpo::scan_k_for(K), k0);
    if (m == 0) continue;
    if (m < 0 || m > K || m > dpo::kWindow || k0 < 0 || k0 >= K) return -1;
    float q = INFINITY, v;
    int k = 0, e;
    for (int j = 0; j < K; j++) {
      const float t = dpo::cell_q(F, tab[j].x, tab[j].y);
      if (t < q) q = t, k = j;
    }
    dpo::scan_entries(F, K, at, k0, m, v, e);
    bad += !(v == q && e == k);
    (*windows)++;
    if (m > *widest) *widest = m;
    *ends += k0 + m > K;
  }
  return bad;
}
"""


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    d = tmp_path_factory.mktemp("window")
    (d / "window.cc").write_text(SOURCE)
    so = str(d / "window.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-fPIC", "-shared", "-I", build.CSRC,
                    str(d / "window.cc"), "-o", so], check=True)
    lib = C.CDLL(so)

    def call(f, K, error):
        f = np.ascontiguousarray(f, np.float32)
        out = [C.c_int() for _ in range(3)]
        bad = lib.check(len(f), f.ctypes.data_as(C.POINTER(C.c_float)), K, C.c_float(error), *map(C.byref, out))
        return bad, [o.value for o in out]

    return call


def nodes(kind, n, rng):
    x, y, z, w, g1, g2, d1, d2 = coefficients(kind, n, rng)
    sign = rng.choice([-1.0, 1.0], (2, n))
    return np.stack([g1 * sign[0], g2 * sign[1], d1, d2, x, y, z, w], axis=1)


@pytest.mark.parametrize("error", [0.0, 2e-7, -2e-7])
@pytest.mark.parametrize("K", [8, 9, 16, 64, 72, 257, 1024])
def test_window_finds_the_tables_first_minimum(check, K, error):
    rng = np.random.default_rng(K)
    n = 8000 if K < 200 else 1500
    for kind in ("steep", "mixed", "flat", "one_axis", "cross", "large_value"):
        f = nodes(kind, n, rng)
        bad, (windows, widest, ends) = check(f, K, error)
        assert bad == 0
        if kind in ("steep", "one_axis") and K < 200:
            assert windows > n // 2 and ends > 0


@pytest.mark.parametrize("K", [8, 64, 257, 1024])
def test_minimum_at_every_entry_and_between(check, K):
    """Pure first harmonics whose minimum is at an entry, half way to the next (a tie up
    to rounding) and next to the axes, where the arctangent changes its form."""
    u = -np.pi + 2 * np.pi * np.arange(8 * K) / (8 * K)
    u = np.concatenate([u, [s * np.pi / 4 * k + e for k in range(8) for s in (-1, 1) for e in (-1e-6, 0, 1e-6)]])
    for scale in (1e-2, 1.0, 50.0):
        f = np.zeros((u.size, 8))
        f[:, 0] = f[:, 1] = 0.02
        f[:, 2], f[:, 3] = 0.3, -1.7
        f[:, 4] = 3.0
        f[:, 5], f[:, 6] = -scale * np.sin(u), -scale * np.cos(u)
        for error in (0.0, 2e-7, -2e-7):
            bad, (windows, _, ends) = check(f, K, error)
            assert bad == 0 and (scale < 1 or (windows > u.size // 2 and ends > 0))


def test_plateaus_and_values_that_are_no_numbers(check):
    big = np.float32(3.4e38)
    rows = [[0.02, 0.02, 1, 1, 7, 0, 0, 0], [0.02, 0.02, 1, 1, 1, 0, 0, 1]]
    for v in (np.nan, np.inf, -np.inf, big):
        for k in (4, 5, 6, 7):
            r = [0.02, -0.02, 0.5, -0.5, 1, 1, 1, 1]
            r[k] = v
            rows.append(r)
    f = np.array(rows, np.float32)
    for K in (8, 64, 1024):
        for r in f:
            bad, _ = check(r[None], K, 0.0)
            assert bad == 0, r
    # a plateau has its first entry, no slope or a slope that is not finite has none
    assert check(f[:1], 64, 0.0)[1][0] == 1 and check(f[1:2], 64, 0.0)[1][0] == 0
