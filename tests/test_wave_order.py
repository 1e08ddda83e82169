"""The places of a chunk's waves in the order of the factorised sweeps
(csrc/dpo_order.h, built for the host): every wave once, the one-cell waves marked,
a short last wave last, and the other waves spread over the workgroups that one
compute unit runs."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from paper_2407_14675_amd import build


@pytest.fixture(scope="module")
def place(tmp_path_factory):
    d = tmp_path_factory.mktemp("order")
    (d / "order.cc").write_text('#include "dpo_order.h"\nextern "C" unsigned long long place(int n, int ones, int c, int* s)'
                                " { return dpo::place_waves(n, ones, c, s); }\n")
    so = str(d / "order.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-I", build.CSRC, str(d / "order.cc"), "-o", so], check=True)
    f = C.CDLL(so).place
    f.restype = C.c_ulonglong

    def call(n, ones, chunk):
        slot = (C.c_int * 64)()
        bits = f(n, ones, chunk, slot)
        return np.array(slot[:(n + 63) // 64]), [(bits >> w) & 1 for w in range(64)]

    return call


@pytest.mark.parametrize("n", [1, 63, 64, 65, 128, 700, 4032, 4095, 4096])
def test_every_wave_once_and_marked(place, n):
    waves = (n + 63) // 64
    for ones in sorted({0, 1, min(63, n), min(64, n), n // 2, n * 9 // 10, max(0, n - 64), n - 1, n}):
        for chunk in range(9):
            slot, bits = place(n, ones, chunk)
            assert sorted(slot) == list(range(waves))
            if n % 64:
                assert slot[-1] == waves - 1
            # wave w holds the entries 64 w .. 64 w + 63 of one-cell nodes first, then the others
            for w in range(waves):
                assert bits[slot[w]] == (min(64 * w + 64, n) <= ones)
            assert sum(bits[waves:]) == 0


@pytest.mark.parametrize("share", [0.02, 0.08, 0.1, 0.25, 0.5])
@pytest.mark.parametrize("waves_per_group", [1, 2, 4, 8])
def test_no_unit_runs_them_all(place, share, waves_per_group):
    """One XCD: 32 units, whose k-th workgroups are neighbours in the list; one load of
    the unit (32 waves).  No unit has more than twice the mean of the other waves,
    and one workgroup of them (measured: 1.2 times and 3)."""
    units, load = 32, 32 // waves_per_group
    kinds = []
    for chunk in range(units * 32 // 64 + 1):
        _, bits = place(4096, int(4096 * (1 - share)), chunk)
        kinds += bits
    other = 1 - np.array(kinds[:units * 32]).reshape(load, units, waves_per_group)
    per_unit = other.sum(axis=(0, 2))
    assert per_unit.max() <= 2 * other.sum() / units + waves_per_group
