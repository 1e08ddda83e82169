"""Which form the direct sweeps take (csrc/dpo_forms.h, built for the host), at
sizes where both were measured: the cell cache where it is the faster by more
than two in a hundred, the keyed corners where they are."""
import ctypes as C
import subprocess

import pytest

from paper_2407_14675_amd import build

EX1, MID, HALF, TINY = 110 * 30**3, 60 * 25**3, 25 * 15**3, 12**4
TABLE, SCAN, SEEDED, WALK = range(4)


@pytest.fixture(scope="module")
def keep(tmp_path_factory):
    d = tmp_path_factory.mktemp("forms")
    (d / "forms.cc").write_text('#include "dpo_forms.h"\nextern "C" int keep(int m, int c, int h, int k, int n, float r)'
                                " { return dpo::keep_cells(m, c, h, k, n, r); }\n")
    so = str(d / "forms.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-I", build.CSRC, str(d / "forms.cc"), "-o", so], check=True)
    f = C.CDLL(so).keep
    return lambda mode, crown, heun, k, n, reach: bool(f(mode, crown, heun, k, n, C.c_float(reach)))


@pytest.mark.parametrize("mode,crown,heun,entries,nodes,reach,cells", [
    (TABLE, 1, 1, 72, EX1, 0.007, True),     # 395 us with cells, 542 without
    (TABLE, 1, 1, 36, EX1, 0.007, True),     # 235, 296
    (TABLE, 1, 1, 72, HALF, 0.004, False),   # 63, 51
    (TABLE, 1, 1, 48, EX1, 0.0725, False),   # 437, 406
    (SCAN, 1, 1, 64, MID, 0.006, False),     # 263, 215
    (SEEDED, 1, 1, 64, EX1, 0.007, False),   # 793, 654
    (WALK, 1, 1, 72, EX1, 0.007, False),     # 88, 80
    (TABLE, 1, 0, 72, TINY, 0.003, True),    # 28, 35
    (SCAN, 1, 0, 64, EX1, 0.007, True),      # 330, 422
    (SCAN, 1, 0, 64, EX1, 0.0725, False),    # 516, 458
    (WALK, 1, 0, 72, TINY, 0.003, True),     # 8.0, 9.3
    (TABLE, 0, 1, 72, EX1, 0.016, True),     # 473, 520
    (TABLE, 0, 1, 16, EX1, 0.016, False),    # 175, 160
    (TABLE, 0, 1, 72, EX1, 0.107, False),    # 612, 559
    (SCAN, 0, 1, 64, MID, 0.0148, False),    # 233, 210
    (TABLE, 0, 0, 72, EX1, 0.018, True),     # 350, 409
    (SCAN, 0, 0, 64, TINY, 0.007, False),    # 42, 39
    (WALK, 0, 0, 72, EX1, 0.018, False),     # 81, 72
    (TABLE, 0, 0, 72, 256 * 256 * 4, 1.0, False),  # eikonal, steps of a cell: 95, 56
    (SCAN, 0, 0, 64, 33 * 33 * 4, 1.0, False),     # 62, 41
    (TABLE, 0, 0, 72, EX1, float("nan"), False),
    (TABLE, 1, 1, 72, EX1, float("inf"), False),
])
def test_rule(keep, mode, crown, heun, entries, nodes, reach, cells):
    assert keep(mode, crown, heun, entries, nodes, reach) == cells
