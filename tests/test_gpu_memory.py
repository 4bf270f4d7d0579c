"""GPU: the device memory that the library keeps and asks for."""
import contextlib

import numpy as np
import pytest
import torch

import paper_2212_10042_amd as cse
import workloads as W

pytestmark = pytest.mark.gpu

MB = 1 << 20


def _free():
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


@contextlib.contextmanager
def _left(nbytes):
    """All but nbytes of the device's memory taken."""
    try:
        hog = torch.empty(_free() - nbytes, dtype=torch.uint8, device="cuda")
    except torch.OutOfMemoryError:
        pytest.skip("the device's free memory cannot be taken in one piece")
    try:
        yield
    finally:
        del hog
        torch.cuda.empty_cache()


def _keep_a_table():
    """A destroyed platten whose count table (about 109 MB) is kept."""
    cse.cse_release_cached_memory()
    w = W.binom2_grid(300, 120_000, lower_triangle=False)
    P = cse.Platten.create("binom2", w["theta"], w["radii"], w["sims"], keep_all=True)
    P.close()


def test_kept_table_is_released():
    print("[memory] release", flush=True)
    _keep_a_table()
    kept = _free()
    cse.cse_release_cached_memory()
    assert _free() - kept >= 100 * MB
    cse.cse_release_cached_memory()   # nothing left: no error


def test_kept_table_makes_room():
    """Short of memory, the library gives the kept table up before it reports an error."""
    print("[memory] kept table makes room for keys", flush=True)
    w = W.ztest_1d(64, 1 << 20)   # 256 MiB of keys
    P = cse.Platten.create("ztest1", w["theta"], w["radii"], w["sims"])
    ap, lam = (torch.empty(64, dtype=torch.float64, device="cuda") for _ in range(2))
    low, k = torch.empty(1, dtype=torch.float64, device="cuda"), torch.empty(64, dtype=torch.int32, device="cuda")
    _keep_a_table()
    with _left(206 * MB):
        plan = cse.cse_plan_calibrate(P.handle, 3, 0.025, ap, k, lam, low)   # allocates the keys; launches nothing
        cse.cse_plan_destroy(plan)
    g = P.calibrate(3)
    torch.cuda.synchronize()
    assert np.isfinite(g["lambda_tile"].cpu().numpy()).all()
    P.close()


def test_phase23_in_little_memory():
    """A Phase II/III platten of 34 million trials keeps 3.5 GB of states, records and counts; where 2 GiB are free it is
    created with less (shorter chunks, no counts) and gives the same results."""
    print("[memory] phase23 in 2 GiB", flush=True)
    w = W.phase23_grid((2, 2, 2, 2), 750_000)

    def run():
        before = _free()
        P = cse.Platten.create("phase23", w["theta"], w["radii"], w["sims"], cut=w["cut"])
        used = before - _free()
        v = P.validate(5)
        torch.cuda.synchronize()
        P.close()
        return used, {k: v[k].clone() for k in ("reject", "score_T", "tile_bound")}

    cse.cse_release_cached_memory()
    used, whole = run()
    assert used > 2048 * MB
    with _left(2048 * MB):
        used, little = run()
    assert used < 1024 * MB
    for name in whole:
        assert torch.equal(whole[name], little[name]), name


def _scattered(n, sims):
    """n basket boxes in the null that share no threshold, one tile each."""
    r = np.random.default_rng(n)
    th = r.uniform(-4.0, -1.8, (n, 4))
    return th, np.full(th.shape, 1e-4), np.full(n, sims, np.int32)


def test_scattered_boxes_in_little_memory():
    """12,000 boxes without a common threshold have a count table of 290 MB at the usual window; where 400 MiB are free a
    shorter one serves, and the validation is the same."""
    print("[memory] scattered boxes in 400 MiB", flush=True)
    grid = _scattered(12_000, 4_200)

    def run():
        P = cse.Platten.create("basket4", *grid)
        v = P.validate(5)
        torch.cuda.synchronize()
        P.close()
        return {k: v[k].clone() for k in ("reject", "score_T", "tile_bound")}

    cse.cse_release_cached_memory()
    whole = run()
    with _left(400 * MB):
        little = run()
    for name in whole:
        assert torch.equal(whole[name], little[name]), name


def test_many_scattered_boxes():
    """2.9 million boxes without a common threshold: more rows of the usual window than the table's 32-bit places reach,
    so shorter windows.  Sampled tiles against the per-tile path."""
    print("[memory] 2.9 million scattered boxes", flush=True)
    n = 2_900_000
    P = cse.Platten.create("basket4", *_scattered(n, 4_096))
    assert P.n_tiles == n
    v = P.simulate(5)
    R = torch.empty_like(v["reject"])
    for t in (0, 1, 64, 1_234_567, n - 1):
        cse.cse_simulate_per_tile(P.handle, 5, t, t + 1, R)
        torch.cuda.synchronize()
        assert int(R[t]) == int(v["reject"][t]), t
    P.close()
