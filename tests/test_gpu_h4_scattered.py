"""GPU: 4-arm plattens whose boxes share no thresholds: a set of tiles then lists as many count rows as it can,
and a workgroup's rows fill the LDS beside the pilot's histogram.  Rejection counts against the per-tile path
(its own draws), thresholds of the calibration from candidates against those from every key: exact."""
import numpy as np
import pytest
import torch

import paper_2212_10042_amd as cse

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["hier4", "basket4"])
@pytest.mark.parametrize("boxes,n", [(61, 1024), (62, 1100), (64, 4112), (200, 1500)])
def test_no_shared_thresholds(kind, boxes, n):
    print(f"[h4 scattered] {kind} {boxes} boxes x {n}", flush=True)
    r = np.random.default_rng(boxes)
    th = r.uniform(-2.0, 0.3, (boxes, 4))
    th[:, 0] += 3.0 if kind == "hier4" else -2.1   # every box in the null: one tile each
    P = cse.Platten.create(kind, th, np.full(th.shape, 1e-3), np.full(boxes, n, np.int32))
    assert P.n_tiles == boxes
    R = torch.empty(P.n_tiles, dtype=torch.int32, device="cuda")
    cse.cse_simulate_per_tile(P.handle, 5, 0, P.n_tiles, R)
    every = P.calibrate(5, alpha=0.05)
    cse.cse_platten_set_option(P.handle, cse.CSE_OPT_H4_BRACKET, 1)
    cand = P.calibrate(5, alpha=0.05)
    v = P.validate(5)
    torch.cuda.synchronize()
    for g in (every, cand, v):
        assert torch.equal(g["reject"], R)
        assert torch.equal(g["score_T"], every["score_T"])
        assert torch.equal(g["tile_bound"], every["tile_bound"])
    for name in ("k", "lambda_tile", "reject_at_lambda", "lambda_global"):
        assert torch.equal(cand[name], every[name]), name
    assert int(cand["k"].max()) > 0
    if kind == "hier4":   # the calibration did take candidates: without a margin it misses some
        cse.cse_platten_set_option(P.handle, cse.CSE_OPT_H4_MARGIN, 0.0)
        bare = P.calibrate(5, alpha=0.05)
        assert torch.equal(bare["lambda_tile"], every["lambda_tile"])
        assert cse.cse_work_counters(P.handle)["trials"] > 0
    P.close()
