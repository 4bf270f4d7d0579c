"""GPU: the 2-arm selection with few simulations per tile, at the edges of the ways it takes (a wave's registers up to 512
simulations, or 128 on grids of more than 256 batches; bracket histograms beyond), uneven counts in one platten.
Against the oracle: exact."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2212_10042_amd as cse
import workloads as W

pytestmark = pytest.mark.gpu


def _check(w, seed, alpha):
    print(f"[binom2 few sims] {len(w['sims'])} boxes x {w['sims'].min()}..{w['sims'].max()}", flush=True)
    P = cse.Platten.create("binom2", w["theta"], w["radii"], w["sims"])
    g = P.calibrate(seed, alpha=alpha, with_validation=False)
    torch.cuda.synchronize()
    oc = O.calibrate("binom2", w["theta"], w["radii"], w["sims"], seed, alpha)
    k = g["k"].cpu().numpy()
    same = k == oc["k"]
    assert same.mean() > 0.99 and ((k > 0).any() or w["sims"].max() < 10)   # one simulation: no rank
    assert np.array_equal(g["lambda_tile"].cpu().numpy()[same], oc["lam"][same])
    assert np.array_equal(g["reject_at_lambda"].cpu().numpy()[same], oc["reject_at_lam"][same])
    P.close()


@pytest.mark.parametrize("n", [1, 63, 64, 65, 128, 129, 511, 512, 513])
def test_few_batches(n):
    _check(W.binom2_grid(12, n, lo=-2.0, hi=0.5), n, 0.2)


@pytest.mark.parametrize("n", [127, 128, 129, 512])
def test_many_batches(n):
    _check(W.binom2_grid(184, n, lo=-2.0, hi=0.5), n, 0.05)


def test_uneven_counts():
    w = W.binom2_grid(16, 1, lo=-2.0, hi=0.5)
    w["sims"] = np.random.default_rng(3).choice([40, 100, 512, 600, 3000], len(w["sims"])).astype(np.int32)
    _check(w, 5, 0.1)
