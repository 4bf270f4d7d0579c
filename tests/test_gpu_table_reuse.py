"""GPU: plattens created one after the other, whose count tables may take over a destroyed one's memory
(larger, smaller, another design's, two alive at once), give what they give in any other order."""
import torch

import pytest

import paper_2212_10042_amd as cse
import workloads as W

pytestmark = pytest.mark.gpu


def _counts(kind, m, n):
    w = W.binom2_grid(m, n, lower_triangle=True) if kind == "binom2" else W.hier4_grid(m, n)
    P = cse.Platten.create(kind, w["theta"], w["radii"], w["sims"])
    g = P.simulate(7)
    torch.cuda.synchronize()
    return P, (g["reject"].clone(), g["score_T"].clone())


def test_tables_of_destroyed_plattens_are_reused_safely():
    cases = [("binom2", 40, 60_000), ("binom2", 12, 300), ("hier4", 3, 50_000), ("binom2", 60, 90_000)]
    ref = []
    for c in cases:
        P, r = _counts(*c)
        P.close()
        ref.append(r)
    order = [3, 0, 1, 2, 0, 3, 2, 1]
    for i in order:                       # one at a time
        P, r = _counts(*cases[i])
        assert all(torch.equal(a, b) for a, b in zip(r, ref[i]))
        P.close()
    alive = [_counts(*cases[i]) for i in (0, 3, 2)]   # several at once
    for (P, r), i in zip(alive, (0, 3, 2)):
        g = P.simulate(7)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(r, ref[i]))
        assert torch.equal(g["reject"], ref[i][0]) and torch.equal(g["score_T"], ref[i][1])
        P.close()
