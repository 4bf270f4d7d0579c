"""The Phase II/III posterior (hier_post.hpp), compiled for the host: its sums are the same bits whether one lane
takes all segments of the nodes or each lane one, and agree with scipy's quadrature of the same model's nodes."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2212_10042_amd", "csrc")

PROG = r"""
#include <math.h>
#include <stdio.h>
#include <vector>
#include "hier_post.hpp"
using namespace cse;
int main() {
    std::vector<HierNode> N(HP_NODES);
    const double lo = log(1e-6), h = (log(1e3) - lo) / (HP_NODES - 1);
    for (int j = 0; j < HP_NODES; ++j) {
        HierNode &d = N[j];
        d.ls2 = lo + h * j;
        d.s2 = exp(d.ls2);
        d.inv_s2 = 1.0 / d.s2;
        d.c = 100.0 / (d.s2 + 400.0);
        d.beta = d.c * d.inv_s2;
        d.lconst = -0.5 * (3.0 * d.ls2 + log(d.s2 + 400.0)) - 1.0005 * d.ls2 - 0.000005 * d.inv_s2 +
                   log(j == 0 || j == HP_NODES - 1 ? 0.5 * h : h) + d.ls2;
    }
    int y[4], m[4];
    while (scanf("%d %d %d %d %d %d %d %d", y, y + 1, y + 2, y + 3, m, m + 1, m + 2, m + 3) == 8) {
        const double n[4] = {(double)m[0], (double)m[1], (double)m[2], (double)m[3]};
        HierSums one, lanes, part;
        hier_segments(y, n, N.data(), 0, HP_SEGS, one, nullptr, 7);
        hier_zero(lanes);
        for (int s = 0; s < HP_SEGS; ++s) {   // a lane's segment, joined in ascending order
            hier_segments(y, n, N.data(), s, s + 1, part, nullptr, 7);
            hier_add(lanes, part, [](double v) { return v; });
        }
        for (int a = 0; a < 4; ++a) lanes.th0[a] = part.th0[a];
        for (const HierSums *H : {&one, &lanes}) {
            HierSummary o;
            hier_summary(*H, o);
            for (int i = 0; i < 3; ++i) printf("%a %a %a ", o.P[i], o.Sc[i], o.dvar[i]);
            for (int a = 0; a < 4; ++a) printf("%a %a ", o.mean[a], o.var[a]);
        }
        printf("\n");
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def states():
    r = np.random.default_rng(3)
    sizes = np.array([50, 75, 83, 100, 108, 116, 125, 133, 150])
    n = sizes[r.integers(0, 9, (400, 4))]
    n[:, :2] += 100 * r.integers(0, 3, (400, 1))
    y = r.binomial(n, r.uniform(0.1, 0.9, (400, 4)))
    y[0], y[1] = 0, n[1]   # no response, every response
    return y, n


@pytest.fixture(scope="module")
def summaries(states, tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    d = tmp_path_factory.mktemp("p23post")
    src, exe = os.path.join(d, "prog.cpp"), os.path.join(d, "prog")
    with open(src, "w") as f:
        f.write(PROG)
    subprocess.run([hipcc, "-x", "hip", "--offload-arch=gfx950", "-O2", "-std=c++17", "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"), src, "-o", exe], check=True, capture_output=True)
    inp = "".join(" ".join(str(v) for v in (*a, *b)) + "\n" for a, b in zip(*states))
    out = subprocess.run([exe], input=inp, capture_output=True, text=True, check=True).stdout.split("\n")
    return np.array([[float.fromhex(v) for v in line.split()] for line in out if line.strip()])


def test_same_bits_for_any_number_of_lanes(summaries):
    half = summaries.shape[1] // 2
    assert half == 17 and np.isfinite(summaries).all()
    assert np.array_equal(summaries[:, :half], summaries[:, half:])


def test_against_newton_in_numpy(states, summaries):
    """The same 90-node Laplace mixture with fully converged modes: relative 1e-9 (the modes' remaining error,
    1e-12, times the condition of the tails), dvar 1e-5 (its reference points are float32)."""
    from scipy.special import ndtr
    y, n = (v.astype(np.float64) for v in states)
    j = np.arange(90)
    ls2 = np.log(1e-6) + (np.log(1e3) - np.log(1e-6)) / 89 * j
    lw, z, mode, C, vd = [], [], [], [], []
    for k in range(90):
        s2 = np.exp(ls2[k])
        Q = (np.eye(4) - 100.0 / (s2 + 400.0)) / s2
        th = np.log((y + 0.5) / (n - y + 0.5))
        for _ in range(60):
            p = 1.0 / (1.0 + np.exp(-th))
            H = Q[None] + np.eye(4)[None] * (n * p * (1 - p))[:, None, :]
            th = th + np.linalg.solve(H, (y - n * p - (th + 1.34) @ Q)[..., None])[..., 0]
        p = 1.0 / (1.0 + np.exp(-th))
        H = Q[None] + np.eye(4)[None] * (n * p * (1 - p))[:, None, :]
        e = th + 1.34
        c = np.linalg.inv(H)
        lw.append((y * th - n * np.logaddexp(0.0, th)).sum(1) - 0.5 * np.einsum("na,ab,nb->n", e, Q, e)
                  - 0.5 * np.linalg.slogdet(H)[1] - 0.5 * (3 * ls2[k] + np.log(s2 + 400.0)) - 0.0005 * ls2[k] - 5e-6 / s2
                  + (np.log(0.5) if k in (0, 89) else 0.0))
        v = c[:, [1, 2, 3], [1, 2, 3]] + c[:, :1, 0] - 2 * c[:, 1:, 0]
        z.append((th[:, 1:] - th[:, :1]) / np.sqrt(v))
        mode.append(th)
        C.append(c[:, range(4), range(4)])
        vd.append(v)
    lw, z, mode, C, vd = (np.array(v) for v in (lw, z, mode, C, vd))
    w = np.exp(lw - lw.max(0))
    w = (w / w.sum(0))[..., None]
    mean = (w * mode).sum(0)
    var = (w * (C + (mode - mean) ** 2)).sum(0)
    dm = mode[..., 1:] - mode[..., :1]
    dvar = (w * (vd + (dm - (w * dm).sum(0)) ** 2)).sum(0)
    got = summaries[:, :17]
    np.testing.assert_allclose(got[:, 0:9:3], (w * ndtr(z)).sum(0), rtol=1e-9)
    np.testing.assert_allclose(got[:, 1:9:3], (w * ndtr(-z)).sum(0), rtol=1e-9)
    np.testing.assert_allclose(got[:, 2:9:3], dvar, rtol=1e-5)
    np.testing.assert_allclose(got[:, 9::2], mean, rtol=1e-9, atol=1e-10)
    np.testing.assert_allclose(got[:, 10::2], var, rtol=1e-9)
