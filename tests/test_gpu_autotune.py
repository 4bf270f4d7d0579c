"""GPU: what cse_autotune times and keeps."""
import pytest
import torch

import paper_2212_10042_amd as cse
import workloads as W

pytestmark = pytest.mark.gpu


def test_4arm_times_the_calibration_that_runs():
    """A platten that calibrates from candidates is tuned on them: the last selection before the call left tiles to
    regenerated keys (no margin); the pilots of the timed launches count anew, and with the margin back there are
    none.  The calibration is the same after the call."""
    w = W.hier4_grid(2, 3000, lo=-0.08, hi=0.08, seed=9)
    print("[autotune] hier4 from candidates", flush=True)
    P = cse.Platten.create("hier4", w["theta"], w["radii"], w["sims"])
    cse.cse_platten_set_option(P.handle, cse.CSE_OPT_H4_BRACKET, 1)
    before = P.calibrate(9)
    cse.cse_platten_set_option(P.handle, cse.CSE_OPT_H4_MARGIN, 0.0)
    P.calibrate(9)
    assert cse.cse_work_counters(P.handle)["trials"] > 0
    cse.cse_platten_set_option(P.handle, cse.CSE_OPT_H4_MARGIN, 6.0)
    value, _ = cse.cse_autotune(P.handle, seed=9)
    assert 1024 <= value <= 65536
    assert cse.cse_work_counters(P.handle)["trials"] == 0
    after = P.calibrate(9)
    torch.cuda.synchronize()
    for name in ("reject", "score_T", "k", "lambda_tile", "reject_at_lambda", "tile_bound"):
        assert torch.equal(before[name], after[name]), name
    P.close()


def test_phase23_small_platten():
    """Few items, many new states: every grid of the posterior kernel is timed and kept as it is, the default (trials per
    item 256, grid 512) among them, not cut down to a workgroup per four items."""
    w = W.phase23_grid((2, 2, 2, 2), 200, seed=3)
    print("[autotune] phase23, few items", flush=True)
    P = cse.Platten.create("phase23", w["theta"], w["radii"], w["sims"], cut=w["cut"])
    before = P.calibrate(9)
    chunk, grid = cse.cse_autotune(P.handle, seed=9)
    assert chunk in (64, 128, 256, 512) and grid in (512, 1024, 2048)
    after = P.calibrate(9)
    torch.cuda.synchronize()
    for name in ("reject", "score_T", "k", "lambda_tile", "reject_at_lambda", "tile_bound"):
        assert torch.equal(before[name], after[name]), name
    P.close()
