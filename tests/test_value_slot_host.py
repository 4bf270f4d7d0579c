"""The table of distinct thresholds (value_slot.hpp), compiled for the host: the values of grids, unshifted, shifted and
halved, spread over its slots.  With at most half of the slots taken a random placement probes 1.5 slots on average
when it finds a value (Knuth, linear probing); allowed are 4."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2212_10042_amd", "csrc")

PROG = r"""
#include <stdio.h>
#include "value_slot.hpp"
int main() {
    double v;
    int bits;
    while (scanf("%d %la", &bits, &v) == 2) printf("%llu\n", (unsigned long long)cse::value_slot(v, bits));
    return 0;
}
"""


@pytest.fixture(scope="module")
def slots(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ not found")
    d = tmp_path_factory.mktemp("slot")
    src, exe = os.path.join(d, "prog.cpp"), os.path.join(d, "prog")
    with open(src, "w") as f:
        f.write(PROG)
    subprocess.run([gxx, "-O2", "-std=c++17", "-I", CSRC, src, "-o", exe], check=True, capture_output=True)

    def call(values, bits):
        inp = "".join(f"{bits} {float(v).hex()}\n" for v in values)
        out = subprocess.run([exe], input=inp, capture_output=True, text=True, check=True).stdout
        return np.array(out.split(), dtype=np.int64)

    return call


def _centres(m, lo=-1.0, hi=1.0):
    w = (hi - lo) / m
    return lo + (np.arange(m) + 0.5) * w


GRIDS = {
    "16 and 1024 on [-1, 1]": np.concatenate([_centres(16), _centres(1024)]),
    "4096 on [-4, 4]": _centres(4096, -4.0, 4.0),
    "1024 shifted": _centres(1024) + 0.0123,
    "halved": np.concatenate([_centres(2 ** k, -3.0, 1.0) for k in range(3, 12)]),
    "32-bit fractions": np.random.default_rng(1).integers(1, 2 ** 32, 4096) / 2.0 ** 32,
}


@pytest.mark.parametrize("name", GRIDS)
@pytest.mark.parametrize("extra", [0, 4])   # tables as full as they get, and those of many tiles
def test_values_spread(slots, name, extra):
    values = np.unique(GRIDS[name])
    bits = 6
    while (1 << bits) < 2 * len(values):
        bits += 1
    bits += extra
    first = slots(values, bits)
    assert first.min() >= 0 and first.max() < 1 << bits
    taken, probes = set(), 0
    for i in first.tolist():
        probes += 1
        while i in taken:
            i = (i + 1) & ((1 << bits) - 1)
            probes += 1
        taken.add(i)
    assert probes <= 4 * len(values)
