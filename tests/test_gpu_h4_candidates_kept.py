"""GPU: 4-arm calibrations from candidates (CSE_OPT_H4_BRACKET = 1, whatever the size) at the edges of their granules,
chunks, slices and pilots, with atoms, uneven counts and alpha from 0.01 to its limit 0.05.  Rejection counts against
the per-tile path (its own draws), thresholds against those from every key: exact."""
import numpy as np
import pytest
import torch

import paper_2212_10042_amd as cse
import workloads as W

pytestmark = pytest.mark.gpu


def _check(kind, theta, radii, sims, seed, alpha):
    print(f"[h4 kept] {kind} boxes={len(sims)} sims={sims.min()}..{sims.max()} alpha={alpha}", flush=True)
    P = cse.Platten.create(kind, theta, radii, sims)
    every = P.calibrate_tiebreak(seed, alpha=alpha)   # always from every key
    plain = P.calibrate(seed, alpha=alpha)            # below 2^26 keys: from every key
    cse.cse_platten_set_option(P.handle, cse.CSE_OPT_H4_BRACKET, 1)
    g = P.calibrate(seed, alpha=alpha)
    R = torch.empty(P.n_tiles, dtype=torch.int32, device="cuda")
    cse.cse_simulate_per_tile(P.handle, seed, 0, P.n_tiles, R)
    torch.cuda.synchronize()
    assert torch.equal(g["reject"], R)
    for name in ("k", "lambda_tile", "lambda_global"):
        assert torch.equal(g[name], every[name]), name
    for name in ("score_T", "reject_at_lambda", "cp_upper", "tile_bound"):
        assert torch.equal(g[name], plain[name]), name
    P.close()
    return g


def _grid(kind, m, n, lo, hi):
    return W.hier4_grid(m, n, lo=lo, hi=hi, seed=3) if kind == "hier4" else W.basket_grid(m, n, lo=lo - 1.75, hi=hi - 1.75, seed=3)


@pytest.mark.parametrize("kind", ["hier4", "basket4"])
@pytest.mark.parametrize("n", [1, 15, 17, 63, 65, 130, 1023])
def test_every_key_is_a_candidate(kind, n):
    w = _grid(kind, 2, n, -0.3, 0.3)
    _check(kind, w["theta"], w["radii"], w["sims"], n, 0.05)


@pytest.mark.parametrize("kind", ["hier4", "basket4"])
@pytest.mark.parametrize("n,alpha", [(1024, 0.05), (1025, 0.025), (2047, 0.05), (4111, 0.05), (4112, 0.01), (9000, 0.05),
                                     (20_000, 0.04), (33_279, 0.025), (33_281, 0.025)])
def test_pilot_and_slice_edges(kind, n, alpha):
    w = _grid(kind, 2, n, -0.08, 0.08)
    g = _check(kind, w["theta"], w["radii"], w["sims"], 5, alpha)
    assert int(g["k"].max()) > 0


@pytest.mark.parametrize("n", [1500, 8000])
def test_atoms(n):
    # arms at about one success in 35: a handful of outcomes, half of the keys equal
    w = W.basket_grid(2, n, lo=-3.6, hi=-3.4, seed=3)
    _check("basket4", w["theta"], w["radii"], w["sims"], 4, 0.05)


@pytest.mark.parametrize("kind", ["hier4", "basket4"])
def test_scattered_boxes_uneven_counts(kind):
    r = np.random.default_rng(7)
    th = r.uniform(-2.0, 0.3, (290, 4))
    th = np.concatenate([th, th[:9]])   # some boxes twice
    sims = r.choice([40, 1000, 1500, 3001], len(th)).astype(np.int32)
    _check(kind, th, np.full(th.shape, 0.02), sims, 9, 0.025)
