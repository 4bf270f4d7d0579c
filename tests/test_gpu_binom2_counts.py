"""GPU: the 2-arm count table (success counts per distinct threshold, shared by every tile) against
the oracle, at the edges of its granules, threshold groups and simulation windows.  Counts are
whole numbers: exact."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2212_10042_amd as cse
import workloads as W

pytestmark = pytest.mark.gpu


def _compare(theta, radii, sims, seed, calibrate=True):
    print(f"[b2 counts] boxes={len(sims)} sims={sims.min()}..{sims.max()} seed={seed}", flush=True)
    P = cse.Platten.create("binom2", theta, radii, sims, keep_all=True)
    v = O.validate("binom2", theta, radii, sims, seed, 0.01, keep_all=True)
    o = P.calibrate(seed) if calibrate else P.simulate(seed)
    torch.cuda.synchronize()
    assert np.array_equal(o["reject"].cpu().numpy(), v["R"])
    assert np.array_equal(o["score_T"].cpu().numpy(), v["score_box"][v["box"]])
    if calibrate:
        c = O.calibrate("binom2", theta, radii, sims, seed, 0.025, keep_all=True)
        same = o["k"].cpu().numpy() == c["k"]
        assert same.mean() > 0.99
        assert np.array_equal(o["lambda_tile"].cpu().numpy()[same], c["lam"][same])
        assert np.array_equal(o["reject_at_lambda"].cpu().numpy()[same], c["reject_at_lam"][same])
    P.close()


@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 33, 48, 63, 64, 65, 80, 127, 129])
def test_granule_and_chunk_edges(n):
    # 9 x 9 distinct thresholds: a full group and a group of one on each arm
    w = W.binom2_grid(9, n, lower_triangle=False, seed=n)
    _compare(w["theta"], w["radii"], w["sims"], n)


@pytest.mark.parametrize("shape", [(1, 1), (1, 70), (70, 1), (33, 65), (8, 64)])
def test_group_edges_order_and_duplicates(shape):
    # more thresholds than a workgroup's 32 x 64, boxes in random order, every third box twice,
    # some boxes missing, uneven simulation counts
    r = np.random.default_rng(shape[0] * 100 + shape[1])
    a = np.linspace(-2.5, 0.5, shape[0])
    b = np.linspace(-2.4, 0.7, shape[1])
    th = np.stack(np.meshgrid(a, b, indexing="ij"), -1).reshape(-1, 2)
    th = th[r.permutation(len(th))[: max(1, int(0.8 * len(th)))]]
    th = np.concatenate([th, th[::3]])
    sims = r.choice([100, 150, 333], len(th)).astype(np.int32)
    _compare(th, np.full(th.shape, 0.01), sims, 7)


def test_simulation_windows():
    # five simulation counts of 1,150,000 each have their own threshold groups: 138 MB of counts at
    # once, so the table takes the simulations in windows
    th = np.array([[-1.0, -1.1], [-1.5, -1.0], [0.2, 0.4], [-2.0, -1.2], [-0.7, -0.7]])
    sims = np.array([1_150_000, 1_150_001, 1_150_015, 1_150_016, 1_150_063], np.int32)
    _compare(th, np.full(th.shape, 0.01), sims, 11, calibrate=False)


@pytest.mark.parametrize("m,n", [(3, 65_535), (3, 65_536), (6, 70_001), (50, 300), (24, 1_000), (130, 200)])
def test_selection_bins_rounds_and_batches(m, n):
    # 16- and 32-bit histogram bins (65,535 simulations at most in 16 bits), brackets that take several
    # rounds of the LDS histogram, fewer and more batches than CUs
    w = W.binom2_grid(m, n, lo=-2.0 if m < 10 else -3.0, seed=n)
    _compare(w["theta"], w["radii"], w["sims"], n)
