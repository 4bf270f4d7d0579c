"""GPU: the 4-arm designs' count table, tile sets and calibration from candidate keys, at the edges of
their granules, chunks, slices and pilots.  The plain per-tile path (its own draws) gives the counts,
the oracle small grids whole, and the every-key path (the randomised calibration's first step) the
thresholds elsewhere.  Whole numbers and float32 keys: exact."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2212_10042_amd as cse
import workloads as W

pytestmark = pytest.mark.gpu


def _np(t):
    return t.cpu().numpy()


def _check(kind, theta, radii, sims, seed, alpha=0.025, cut=None):
    print(f"[h4 candidates] {kind} boxes={len(sims)} sims={sims.min()}..{sims.max()} alpha={alpha}", flush=True)
    P = cse.Platten.create(kind, theta, radii, sims, cut=cut)
    g = P.calibrate(seed, alpha=alpha)
    every = P.calibrate_tiebreak(seed, alpha=alpha)
    v = P.simulate(seed)
    R = torch.empty(P.n_tiles, dtype=torch.int32, device="cuda")
    cse.cse_simulate_per_tile(P.handle, seed, 0, P.n_tiles, R)
    torch.cuda.synchronize()
    assert torch.equal(g["reject"], R) and torch.equal(v["reject"], R)
    assert torch.equal(g["score_T"], v["score_T"])
    assert torch.equal(g["k"], every["k"])
    assert torch.equal(g["lambda_tile"], every["lambda_tile"])
    assert torch.equal(g["lambda_global"], every["lambda_global"])
    below, k, lam = _np(g["reject_at_lambda"]), _np(g["k"]), _np(g["lambda_tile"])
    sel = (k > 0) & np.isfinite(lam)
    assert np.all(below[sel] < k[sel])
    P.close()
    return g


@pytest.mark.parametrize("kind", ["hier4", "basket4"])
@pytest.mark.parametrize("n", [1, 15, 17, 63, 65, 130])
def test_small_counts_vs_oracle(kind, n):
    w = W.hier4_grid(2, n, lo=-0.3, hi=0.3, seed=n) if kind == "hier4" else W.basket_grid(2, n, lo=-2.2, hi=-1.2, seed=n)
    cut = 0.3
    g = _check(kind, w["theta"], w["radii"], w["sims"], n, alpha=0.05, cut=cut)
    v = O.validate(kind, w["theta"], w["radii"], w["sims"], n, 0.01, cut=cut)
    assert np.array_equal(_np(g["reject"]), v["R"])


@pytest.mark.parametrize("kind", ["hier4", "basket4"])
@pytest.mark.parametrize("n,alpha", [(1023, 0.025), (1024, 0.05), (1025, 0.025), (2047, 0.05), (4112, 0.01), (9000, 0.05),
                                     (20_000, 0.04), (20_000, 0.2)])
def test_pilot_and_slice_edges(kind, n, alpha):
    # (20,000, 0.04) keeps candidates, (20,000, 0.2) every key
    w = W.hier4_grid(2, n, lo=-0.08, hi=0.08, seed=3) if kind == "hier4" else W.basket_grid(2, n, lo=-1.9, hi=-1.6, seed=3)
    g = _check(kind, w["theta"], w["radii"], w["sims"], 5, alpha=alpha)
    assert int(_np(g["k"]).max()) > 0


def test_atoms():
    # arms at about one success in 35: a handful of outcomes, half of the keys equal
    w = W.basket_grid(2, 8000, lo=-3.6, hi=-3.4, seed=3)
    _check("basket4", w["theta"], w["radii"], w["sims"], 4, alpha=0.05)


@pytest.mark.parametrize("kind", ["hier4", "basket4"])
def test_scattered_boxes_uneven_counts(kind):
    # no two boxes share a threshold (the most rows a set can list), uneven simulation counts,
    # some boxes twice
    r = np.random.default_rng(7)
    th = r.uniform(-2.0, 0.3, (90, 4))
    th = np.concatenate([th, th[:9]])
    sims = r.choice([40, 1000, 1500, 3001], len(th)).astype(np.int32)
    _check(kind, th, np.full(th.shape, 0.02), sims, 9)
