"""GPU: 4-arm calibrations from candidates where a tile's keys crowd together (deep in the null, or few distinct
outcomes) at few simulations, and with a wide margin: the pilot's bound still admits only what the slices hold, so no
tile's keys are regenerated.  Against the every-key path: exact."""
import numpy as np
import pytest
import torch

import paper_2212_10042_amd as cse

pytestmark = pytest.mark.gpu


def _boxes(centre, m, w):
    ax = [c - w + (2 * np.arange(m) + 1) * w / m for c in centre]
    th = np.stack(np.meshgrid(*ax, indexing="ij"), -1).reshape(-1, 4)
    return th, np.full(th.shape, w / m)


DEEP = ("hier4", (1.0, -2.0, -2.0, -2.0))
RARE = ("hier4", (-3.5, -3.5, -3.5, -3.5))
BASKET = ("basket4", (-6.0, -6.0, -6.0, -6.0))


@pytest.mark.parametrize("design", [DEEP, RARE, BASKET], ids=["deep", "rare", "basket"])
@pytest.mark.parametrize("n,alpha,margin", [(1024, 0.05, None), (1500, 0.05, None), (2048, 0.05, None), (3001, 0.025, None),
                                            (9000, 0.05, None), (1024, 0.05, 100.0), (8192, 0.025, 30.0)])
def test_no_tile_regenerated(design, n, alpha, margin):
    kind, centre = design
    print(f"[h4 crowded] {kind} {centre} x {n}, alpha {alpha}, margin {margin}", flush=True)
    th, rd = _boxes(centre, 3, 0.05)
    P = cse.Platten.create(kind, th, rd, np.full(len(th), n, np.int32))
    every = P.calibrate_tiebreak(3, alpha=alpha)
    cse.cse_platten_set_option(P.handle, cse.CSE_OPT_H4_BRACKET, 1)
    if margin is not None:
        cse.cse_platten_set_option(P.handle, cse.CSE_OPT_H4_MARGIN, margin)
    g = P.calibrate(3, alpha=alpha)
    torch.cuda.synchronize()
    assert int(g["k"].max()) > 0
    assert torch.equal(g["k"], every["k"])
    assert torch.equal(g["lambda_tile"], every["lambda_tile"])
    if kind == "hier4":   # the basket design does not count them
        assert cse.cse_work_counters(P.handle)["trials"] == 0
    P.close()
