"""GPU: the 4-arm designs' rejection counts without keys, whose lanes take runs of tiles along arm 3, at the
edges of the runs (1, 8, 9, 17 tiles), of their granules and chunks, with uneven simulation counts and with
rates where all 35 patients respond.  Counts against the plain per-tile path (its own draws), score sums
against the pass with keys.  Whole numbers: exact."""
import numpy as np
import pytest
import torch

import paper_2212_10042_amd as cse

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["hier4", "basket4"])
@pytest.mark.parametrize("length,hi", [(1, 0.0), (8, 0.5), (9, 4.5), (17, 1.0)])
@pytest.mark.parametrize("sims", [1, 17, 300, 4112, "uneven"])
def test_runs_match_per_tile_path(kind, length, hi, sims):
    print(f"[h4 runs] {kind} length={length} hi={hi} sims={sims}", flush=True)
    ax = [np.linspace(-2.5, hi, 3), np.linspace(-2.4, hi, 2), np.linspace(-2.6, hi, 3), np.linspace(-2.7, hi, length)]
    th = np.stack(np.meshgrid(*ax, indexing="ij"), -1).reshape(-1, 4)
    rng = np.random.default_rng(length)
    N = rng.choice([1, 64, 65, 1000], len(th)) if sims == "uneven" else np.full(len(th), sims)
    P = cse.Platten.create(kind, th, np.full(th.shape, 1e-3), N.astype(np.int32), cut=0.3)
    for seed in (3, 4):
        v = P.simulate(seed)
        g = P.calibrate(seed, alpha=0.025)
        R = torch.empty(P.n_tiles, dtype=torch.int32, device="cuda")
        cse.cse_simulate_per_tile(P.handle, seed, 0, P.n_tiles, R)
        torch.cuda.synchronize()
        assert torch.equal(v["reject"], R)
        assert torch.equal(v["score_T"], g["score_T"])
    P.close()
