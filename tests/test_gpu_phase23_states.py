"""Phase II/III design: trials whose looks share evaluated states (and read their counts from the
table per threshold) against the per-tile path, which draws every word and evaluates every look of
every trial by itself.  Counts are whole numbers and must be equal.
"""
import numpy as np
import pytest
import torch

import paper_2212_10042_amd as cse
import workloads as W

pytestmark = pytest.mark.gpu


def _grid(case):
    rng = np.random.default_rng(11)
    if case == "one_trial":          # a single state, the smallest table
        w = W.phase23_grid((1, 1, 1, 1), 1, seed=4)
    elif case == "many_items":       # more items than workgroups of the first look
        w = W.phase23_grid((7, 7, 7, 7), 65, seed=4)
    elif case == "uneven":           # rows as long as the longest tile of their threshold
        w = W.phase23_grid((2, 2, 2, 2), 1, seed=5)
        w["sims"] = rng.integers(1, 1500, len(w["theta"])).astype(np.int32)
    elif case == "table_full":       # total trials = slots of the state table
        w = W.phase23_grid((1, 1, 1, 1), 1, seed=6)
        w["theta"] = rng.uniform(-0.6, 0.6, (16, 4))
        w["radii"] = np.full((16, 4), 1e-3)
        w["sims"] = np.full(16, 4096, np.int32)
    else:                            # counts of more than 2^30 bytes: words drawn per trial
        w = W.phase23_grid((1, 1, 1, 1), 1, seed=6)
        w["theta"] = rng.uniform(-0.6, 0.6, (12, 4))
        w["radii"] = np.full((12, 4), 1e-3)
        w["sims"] = np.full(12, 420_000, np.int32)
    return w


@pytest.mark.parametrize("case", ["one_trial", "many_items", "uneven", "table_full", "no_count_table"])
def test_phase23_shared_states_match_per_tile_path(case):
    w = _grid(case)
    P = cse.Platten.create("phase23", w["theta"], w["radii"], w["sims"], cut=0.2)
    print(f"[phase23 states] {case}: {P.n_tiles} tiles", flush=True)
    for seed in (5, 6):              # the second call starts from the first one's tables
        a = P.simulate(seed=seed)
        R = torch.empty(P.n_tiles, dtype=torch.int32, device="cuda")
        cse.cse_simulate_per_tile(P.handle, seed, 0, P.n_tiles, R)
        torch.cuda.synchronize()
        assert torch.equal(R, a["reject"])
        c = cse.cse_work_counters(P.handle)
        N = int(np.asarray(w["sims"])[P.tiles["box"]].sum())
        assert c["trials"] == N and c["looks_phase2"] + c["looks_phase3"] <= 4 * N
        assert case == "one_trial" or int(R.sum()) > 0
    P.close()
