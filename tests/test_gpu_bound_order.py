"""GPU: the bound's search over grids that mix whole boxes and pieces, whose tiles go in an order of their
own and whose pieces share their vertices' terms, against the same tiles one box at a time (no mixing, the
tiles as they are): the same evaluations, hence the same bits.  Also Clopper-Pearson at the counts' ends."""
import numpy as np
import pytest
import torch

import paper_2212_10042_amd as cse
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["binom2", "hier4", "basket4"])
def test_mixed_tiles_give_what_single_boxes_give(kind):
    w = {"binom2": lambda: W.binom2_grid(6, 300, lower_triangle=True), "hier4": lambda: W.hier4_grid(3, 300, lo=-0.4, hi=0.4),
         "basket4": lambda: W.basket_grid(3, 300, lo=-2.4, hi=-1.2)}[kind]()
    P = cse.Platten.create(kind, w["theta"], w["radii"], w["sims"])
    print(f"[bound order] {kind}: {P.n_tiles} tiles", flush=True)
    g, v = P.calibrate(3, alpha=0.025), P.validate(3)
    torch.cuda.synchronize()
    box = np.asarray(P.tiles["box"])
    for b in range(0, len(w["theta"]), 5):
        ids = torch.as_tensor(np.flatnonzero(box == b))
        if len(ids) == 0:
            continue
        Q = cse.Platten.create(kind, w["theta"][b:b + 1], w["radii"][b:b + 1], w["sims"][b:b + 1])
        h, u = Q.calibrate(3, alpha=0.025), Q.validate(3)
        torch.cuda.synchronize()
        for name in ("alpha_prime", "k", "cp_upper", "tile_bound"):
            assert torch.equal(g[name].cpu()[ids], h[name].cpu()), name
        for name in ("cp_upper", "tile_bound", "q_star"):
            assert torch.equal(v[name].cpu()[ids], u[name].cpu()), name
        Q.close()
    P.close()
