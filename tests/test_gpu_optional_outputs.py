"""GPU: outputs of the calibration that a caller may leave out (NULL): the others are the same without them."""
import pytest
import torch

import paper_2212_10042_amd as cse
import workloads as W

pytestmark = pytest.mark.gpu

GRIDS = {
    "ztest1": lambda: W.ztest_1d(20, 3000),
    "binom2": lambda: W.binom2_grid(12, 3000, lo=-2.0, hi=0.5),
    "hier4": lambda: W.hier4_grid(2, 3000, lo=-0.08, hi=0.08),
    "basket4": lambda: W.basket_grid(2, 3000, lo=-1.9, hi=-1.6),
    "phase23": lambda: W.phase23_grid((2, 2, 2, 2), 300),
}


def _calibrate(P, alpha, counts, noalloc=False):
    k = torch.empty(P.n_tiles, dtype=torch.int32, device="cuda")
    ap, lam = (torch.empty(P.n_tiles, dtype=torch.float64, device="cuda") for _ in range(2))
    below = torch.empty_like(k) if counts else None
    low = torch.empty(1, dtype=torch.float64, device="cuda")
    fn = cse.cse_calibrate_noalloc if noalloc else cse.cse_calibrate
    fn(P.handle, 3, alpha, ap, k, lam, low, below)
    torch.cuda.synchronize()
    return ap, k, lam, low


# alpha = 1e-6: no tile has k >= 1; margin 0: most 2-arm tiles are selected from the full histogram
@pytest.mark.parametrize("design,alpha,options", [(d, a, ()) for d in GRIDS for a in (0.05, 1e-6)] + [
    ("binom2", 0.05, ((cse.CSE_OPT_B2_MARGIN, 0.0),)),
    ("hier4", 0.05, ((cse.CSE_OPT_H4_BRACKET, 1),)),
    ("hier4", 0.05, ((cse.CSE_OPT_H4_BRACKET, 1), (cse.CSE_OPT_H4_MARGIN, 0.0))),
])
def test_without_counts_below_lambda(design, alpha, options):
    print(f"[optional outputs] {design} alpha={alpha} {options}", flush=True)
    w = GRIDS[design]()
    P = cse.Platten.create(design, w["theta"], w["radii"], w["sims"], cut=w.get("cut"))
    for option, value in options:
        cse.cse_platten_set_option(P.handle, option, value)
    whole = _calibrate(P, alpha, counts=True)
    for noalloc in (False, True):
        for a, b in zip(whole, _calibrate(P, alpha, counts=False, noalloc=noalloc)):
            assert torch.equal(a, b)
    P.close()
