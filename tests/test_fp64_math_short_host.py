"""The Phase II/III posterior's exp, log1p and erfc (fp64_math.hpp, Chebyshev expansions), compiled for
the host against mpmath at 30 digits: relative error of exp_short and log1p_short within 2 x 2^-52 (the
bound of the longer series they stand in for), of erfc_pos within 4 x 2^-52 on [0, 26] (three factors of
one rounding each and the polynomial's)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

mp = pytest.importorskip("mpmath")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2212_10042_amd", "csrc")

PROG = r"""
#include <math.h>
#include <stdio.h>
#include "fp64_math.hpp"
int main() {
    double x;
    while (scanf("%la", &x) == 1)
        printf("%a %a %a\n", fabs(x) <= 700.0 ? cse::exp_short(x) : NAN,
               (x >= 0.0 && x <= 1.0) ? cse::log1p_short(x / (2.0 + x)) : NAN,
               x >= 0.0 ? cse::erfc_pos(x, [](double d) { return 1.0 / d; }) : NAN);
    return 0;
}
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    d = tmp_path_factory.mktemp("fp64short")
    src, exe = os.path.join(d, "prog.cpp"), os.path.join(d, "prog")
    with open(src, "w") as f:
        f.write(PROG)
    subprocess.run([hipcc, "-O2", "-std=c++17", "-I", CSRC, src, "-o", exe], check=True, capture_output=True)

    def call(xs):
        inp = "".join(float(x).hex() + "\n" for x in xs)
        out = subprocess.run([exe], input=inp, capture_output=True, text=True, check=True).stdout.split("\n")
        return np.array([[float.fromhex(v) for v in line.split()] for line in out if line.strip()])

    return call


RANGES = {
    0: (mp.exp, np.concatenate([np.linspace(-700.0, 0.0, 1401), np.linspace(-1.0, 1.0, 401)]), 2.0),
    1: (mp.log1p, np.unique(np.concatenate([np.linspace(0.0, 1.0, 1001)[1:], np.geomspace(1e-300, 1.0, 600)])), 2.0),
    2: (mp.erfc, np.concatenate([np.linspace(0.0, 26.0, 1301), np.linspace(0.0, 3.0, 601), np.geomspace(1e-12, 1.0, 100)]),
        4.0),
}


@pytest.mark.parametrize("col", [0, 1, 2], ids=["exp_short", "log1p_short", "erfc_pos"])
def test_short_expansions(run, col):
    fn, xs, tol = RANGES[col]
    mp.mp.dps = 30
    w = max(float(abs((mp.mpf(g) - fn(mp.mpf(x))) / fn(mp.mpf(x)))) / 2.0**-52 for g, x in zip(run(xs)[:, col], xs))
    print(f"worst {w:.2f} x 2^-52")
    assert w <= tol


def test_erfc_beyond_its_range(run):
    r = run([27.0, 100.0, 1e300, float("inf")])[:, 2]
    assert np.all((r >= 0.0) & (r < 1e-300))
