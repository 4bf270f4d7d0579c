"""GPU: 4-arm calibrations below the size from which candidate keys are kept by default, with every key (the
default there) and with candidates (CSE_OPT_H4_BRACKET = 1): pilots, slices and simulation counts at their
edges.  Float32 keys and whole numbers: exact."""
import pytest
import torch

import paper_2212_10042_amd as cse
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["hier4", "basket4"])
@pytest.mark.parametrize("m,n", [(2, 63), (3, 1023), (3, 1024), (2, 4112), (2, 33_000), (4, 9000)])
def test_candidates_give_what_every_key_gives(kind, m, n):
    print(f"[h4 rule] {kind} {m}^4 boxes x {n}", flush=True)
    w = W.hier4_grid(m, n, lo=-0.4, hi=0.4, seed=m) if kind == "hier4" else W.basket_grid(m, n, lo=-2.4, hi=-1.2, seed=m)
    P = cse.Platten.create(kind, w["theta"], w["radii"], w["sims"])
    got = []
    for option in (0, 1, 0):
        cse.cse_platten_set_option(P.handle, cse.CSE_OPT_H4_BRACKET, option)
        g = P.calibrate(11, alpha=0.025)
        torch.cuda.synchronize()
        got.append({k: g[k].clone() for k in ("reject", "score_T", "k", "lambda_tile", "lambda_global", "reject_at_lambda")})
    for g in got[1:]:
        for name, v in got[0].items():
            assert torch.equal(v, g[name]), name
    P.close()
