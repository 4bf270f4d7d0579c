"""GPU: 4-arm calibrations whose tiles keep more candidates than a wave selects in LDS (large simulation counts, small
alpha, small boxes: the pilot's bound leaves thousands): they are selected from the candidates, in LDS by the workgroup
up to 10,240 and from memory beyond, not from regenerated keys.  Against the every-key path: exact."""
import numpy as np
import pytest
import torch

import paper_2212_10042_amd as cse

pytestmark = pytest.mark.gpu


# expected candidates of a tile: rank / pilot * n with k = alpha n, pilot 2,048, rank = mean + 6 sd + 7
@pytest.mark.parametrize("m,n,alpha", [
    (2, 220_000, 0.0037),        # some 3,300: on both sides of the waves' 3,072
    (2, 300_000, 0.0025),        # 3,800
    (5, 262_144, 0.003),         # the same from longer slices
    (2, 1 << 20, 0.0005),        # 7,300
    (2, (1 << 21) + 5, 0.0004),  # 13,500
    (2, 60_000, 0.025),          # 2,950, k = 1,500
    (2, 300_001, 0.05),          # 25,000, k = 15,000
])
def test_selected_from_the_candidates(m, n, alpha):
    print(f"[h4 many candidates] {m}^4 boxes x {n}, alpha {alpha}", flush=True)
    w = 0.01
    c = -w + (2 * np.arange(m) + 1) * w / m
    th = np.stack(np.meshgrid(c, c, c, c, indexing="ij"), -1).reshape(-1, 4)
    P = cse.Platten.create("hier4", th, np.full(th.shape, w / m), np.full(len(th), n, np.int32))
    every = P.calibrate_tiebreak(3, alpha=alpha)
    cse.cse_platten_set_option(P.handle, cse.CSE_OPT_H4_BRACKET, 1)
    g = P.calibrate(3, alpha=alpha)
    torch.cuda.synchronize()
    assert cse.cse_work_counters(P.handle)["trials"] == 0
    assert int(g["k"].min()) > 0.8 * alpha * n
    assert torch.equal(g["k"], every["k"])
    assert torch.equal(g["lambda_tile"], every["lambda_tile"])
    # keys below lambda: the every-key path counts pairs (S, u) below (lambda, c)
    assert bool((g["reject_at_lambda"] <= every["reject_at_lambda"]).all())
    P.close()
