"""Performance cases of the library: what a user runs, over the sizes they run it at.

A case names an operation on a platten (a grid of tiles) of one design:
  calibrate  thresholds, validation bound, counts and score gradient in one step
  band       validation (upper bound) and the lower side of a two-sided band
  validate   the validation procedure
  tiebreak   randomised calibration
  tie        the Type I Error of each box with its gradient, forward and backward
Grids are those of workloads.py with their origin moved by the seed, so every seed has
other thresholds and other random numbers.  The platten is made once in prepare(), as a
program that calibrates a design on a grid keeps it; the `tie` operation builds its own
on every call, as its entry point does.  Adaptive gridding is a sequence of plattens like
the small and the uneven ones here, with host decisions between them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2212_10042_amd as cse
import workloads as W

ALPHA, DELTA = 0.025, 0.01
N_ARM = 35

# ------------------------------------------------------------------------------ cases


def listed():
    return [
        # the paper's 1-D illustration: the smallest call, launches and latency count
        dict(name="ztest_64", op="calibrate", design="ztest1", m=64, sims=10_000),
        # a first look at a 2-arm design: a coarse ragged triangle, odd simulation count
        dict(name="binom2_20", op="calibrate", design="binom2", m=20, sims=1_001, tri=True),
        # gradient of the Type I Error inside an outer optimisation (autograd, platten per call)
        dict(name="tie_64", op="tie", design="binom2", m=64, sims=4_096, tri=True),
        # the ordinary 2-arm calibration of the benchmark
        dict(name="binom2_256", op="calibrate", design="binom2", m=256, sims=8_192, tri=True),
        # the benchmark's default: every box of the square, kept whether or not it meets the null
        dict(name="binom2_1024", op="calibrate", design="binom2", m=1_024, sims=16_384, tri=False),
        # two-sided band on a grid whose simulation counts were chosen box by box (2^11 .. 2^16)
        dict(name="binom2_181_band", op="band", design="binom2", m=181, sims=0, tri=True),
        # randomised calibration (ties broken by an adjoined uniform)
        dict(name="binom2_256_tiebreak", op="tiebreak", design="binom2", m=256, sims=8_192, tri=True),
        # a coarse 4-arm grid with an odd simulation count
        dict(name="hier4_5", op="calibrate", design="hier4", m=5, sims=3_001),
        # the 4-arm calibration of the benchmark
        dict(name="hier4_16", op="calibrate", design="hier4", m=16, sims=32_768),
        # validation of the basket trial at its fixed 85% rule
        dict(name="basket4_16", op="validate", design="basket4", m=16, sims=32_768),
        # a pilot of the Phase II/III design: few tiles of few trials
        dict(name="phase23_3", op="validate", design="phase23", m=3, sims=2_048),
        # the benchmark's Phase II/III sample: 1,024 boxes of 2^11 .. 2^16 trials
        dict(name="phase23_c5", op="calibrate", design="phase23", m=0, sims=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["ztest1", "binom2", "binom2", "binom2", "hier4", "hier4", "basket4", "phase23"])
    if kind == "ztest1":
        return dict(op=rng.choice(["calibrate", "band"]), design=kind, m=_log_int(rng, 16, 4_096),
                    sims=_log_int(rng, 1_000, 20_000))
    if kind == "binom2":
        op = rng.choice(["calibrate", "calibrate", "band", "tiebreak", "tie"])
        m = _log_int(rng, 12, 96 if op == "tie" else 700)
        uneven = op != "tie" and m <= 300 and rng.random() < 0.3
        return dict(op=op, design=kind, m=m, sims=0 if uneven else _log_int(rng, 700, 17_000),
                    tri=op == "tie" or rng.random() < 0.7)
    if kind in ("hier4", "basket4"):
        op = "calibrate" if kind == "hier4" else rng.choice(["validate", "validate", "calibrate"])
        return dict(op=op, design=kind, m=_log_int(rng, 3, 14), sims=_log_int(rng, 1_500, 33_000))
    return dict(op=rng.choice(["calibrate", "validate"]), design=kind, m=rng.randint(2, 4),
                sims=_log_int(rng, 700, 20_000))


# ------------------------------------------------------------------------------ inputs


def _grid(case, seed):
    """The workload dict of a case: its grid's origin and, where uneven, its counts follow the seed."""
    r = np.random.Generator(np.random.PCG64(int(seed)))
    shift = float(r.uniform(-0.05, 0.05))
    m, sims, design = case["m"], case["sims"], case["design"]
    if design == "ztest1":
        w = W.ztest_1d(m, sims, lo=-1.0, hi=0.0)
        w["theta"] = w["theta"] + min(shift, 0.0)   # every tile stays in the null
    elif design == "binom2":
        w = W.binom2_grid(m, max(sims, 1), lo=-3.0 + shift, hi=1.0 + shift, lower_triangle=case["tri"])
    elif design == "hier4":
        w = W.hier4_grid(m, sims, lo=-1.0 + shift, hi=1.0 + shift)
    elif design == "basket4":
        w = W.basket_grid(m, sims, lo=-3.5 + shift, hi=1.0 + shift)
    elif m == 0:
        w = W.phase23_grid((16, 16, 32, 32), None, lo=-0.9946 + shift, hi=1.1527 + shift, sims_seed=int(seed))
        w = W.subsample(w, np.arange(0, len(w["sims"]), 256))
    else:
        w = W.phase23_grid((m, m, m, m), sims, lo=-0.9946 + shift, hi=1.1527 + shift)
    if sims == 0 and design == "binom2":
        w["sims"] = W.uneven_sims(len(w["theta"]), seed=int(seed))
    w["seed"] = int(r.integers(0, 2 ** 62))
    return w


def prepare(case, seed):
    w = _grid(case, seed)
    if case["op"] == "tie":
        r = np.random.Generator(np.random.PCG64(int(seed) + 1))
        return dict(case=case, seed=w["seed"], radii=w["radii"], sims=w["sims"],
                    theta=torch.tensor(w["theta"], device="cuda"),
                    gout=torch.tensor(r.standard_normal(len(w["sims"])), device="cuda"))
    keep = case["design"] == "binom2" and not case["tri"]
    P = cse.Platten.create(w["design"], w["theta"], w["radii"], w["sims"], cut=w.get("cut"), keep_all=keep)
    return dict(case=case, seed=w["seed"], platten=P)


def run(state):
    op, seed = state["case"]["op"], state["seed"]
    if op == "tie":
        theta = state["theta"].detach().requires_grad_(True)
        f = cse.TIE.apply(theta, state["radii"], state["sims"], state["case"]["design"], seed)
        f.backward(state["gout"])
        return dict(tie=f.detach(), grad=theta.grad)
    P = state["platten"]
    if op == "calibrate":
        return P.calibrate(seed=seed, alpha=ALPHA, delta=DELTA)
    if op == "tiebreak":
        return P.calibrate_tiebreak(seed=seed, alpha=ALPHA)
    v = P.validate(seed=seed, delta=DELTA)
    if op == "validate":
        return v
    return dict(upper=v, lower=P.validate_lower(v["reject"], delta=DELTA))


# ------------------------------------------------------------------------------ work


def work(case):
    """Bytes: each tile's description read and its results written once.  Flops: per simulated
    tile the decision and the sums it enters (the statistic too where it is formed per tile),
    the random words once per simulation, the bound's search per tile; Phase II/III: one
    posterior of 90 nodes per trial."""
    design, op, m = case["design"], case["op"], case["m"]
    d = {"ztest1": 1, "binom2": 2, "hier4": 4, "basket4": 4, "phase23": 4}[design]
    if design == "ztest1":
        tiles = m
    elif design == "binom2":
        tiles = m * (m + 1) // 2 if case["tri"] else m * m
    elif design == "phase23" and m == 0:
        tiles = 1_177
    elif design == "basket4":
        tiles = int(1.12 * m ** 4)
    else:
        tiles = m ** 4
    sims = case["sims"] or 21_504   # mean of 2^11 .. 2^16
    longest = case["sims"] or 65_536
    per = {"ztest1": 3, "binom2": 4, "hier4": 9, "basket4": 9, "phase23": 90 * 400}[design]
    words = {"ztest1": 1, "binom2": 70, "hier4": 140, "basket4": 140, "phase23": 1_400}[design]
    searches = {"calibrate": 2, "tiebreak": 1, "validate": 1, "band": 2, "tie": 0}[op]
    out = {"calibrate": 48 + 16 * d, "tiebreak": 32, "validate": 28 + 16 * d, "band": 52 + 16 * d,
           "tie": 8 + 8 * d}[op]
    flops = tiles * sims * per + longest * words * 10 + tiles * searches * 40 * 20 * 2 * d
    return {"bytes": tiles * (16 * d + 4 + out), "flops": flops}


# ------------------------------------------------------------------------------ exact


def _philox(blk, sim, seed, n3=0):
    """Philox4x32-10 (Salmon et al., SC'11) at counters (blk, sim, n3, 0): four uint32 arrays."""
    m32 = np.uint64(0xFFFFFFFF)
    blk, sim = np.broadcast_arrays(np.asarray(blk, np.uint64), np.asarray(sim, np.uint64))
    c = [blk.copy(), sim.copy(), np.full(sim.shape, n3, np.uint64), np.zeros(sim.shape, np.uint64)]
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        p0, p1 = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), p1 & m32,
             (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), p0 & m32]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return [x.astype(np.uint32) for x in c]


def _log_beta_cf(a, b, x):
    """Log of the continued fraction of the incomplete beta function (modified Lentz), float64 arrays."""
    tiny = 1e-300
    c = np.ones_like(x)
    dd = 1.0 - (a + b) * x / (a + 1.0)
    dd = 1.0 / np.where(np.abs(dd) < tiny, tiny, dd)
    h = dd.copy()
    for i in range(1, 2_000):
        for num in (i * (b - i) * x / ((a + 2 * i - 1) * (a + 2 * i)),
                    -(a + i) * (a + b + i) * x / ((a + 2 * i) * (a + 2 * i + 1))):
            dd = 1.0 + num * dd
            dd = 1.0 / np.where(np.abs(dd) < tiny, tiny, dd)
            c = 1.0 + num / c
            c = np.where(np.abs(c) < tiny, tiny, c)
            step = dd * c
            h = h * step
        if np.all(np.abs(step - 1.0) < 2e-15):
            break
    return np.log(h)


def _cp_upper(R, N, delta):
    """Clopper-Pearson upper bound Beta^{-1}(1 - delta; R + 1, N - R) by bisection on the tail."""
    pairs, inv = np.unique(np.stack([R, N], 1), axis=0, return_inverse=True)
    r, n = pairs[:, 0].astype(np.float64), pairs[:, 1].astype(np.float64)
    full = r >= n
    a, b = r + 1.0, np.where(full, 1.0, n - r)
    lg = lambda v: torch.lgamma(torch.from_numpy(v)).numpy()  # noqa: E731
    lnb = lg(a + b) - lg(a) - lg(b)

    def log_upper_tail(x):   # log P(Beta(a, b) > x) by the fraction that converges there
        left = x < (a + 1.0) / (a + b + 2.0)
        lx, l1 = np.log(x), np.log1p(-x)
        p = np.exp(lnb + a * lx + b * l1 + _log_beta_cf(np.where(left, a, b), np.where(left, b, a),
                                                       np.where(left, x, 1.0 - x)) - np.log(np.where(left, a, b)))
        return np.where(left, np.log1p(-np.minimum(p, 1 - 1e-16)), np.log(np.maximum(p, 1e-300)))

    lo, hi = np.zeros_like(a), np.ones_like(a)
    for _ in range(60):
        x = 0.5 * (lo + hi)
        above = log_upper_tail(np.clip(x, 1e-300, 1 - 1e-16)) > math.log(delta)
        lo, hi = np.where(above, x, lo), np.where(above, hi, x)
    u = np.where(full, 1.0, 0.5 * (lo + hi))
    return u[np.asarray(inv).reshape(-1)]


def _search(fn, n):
    """Minimum over s in [-30, 30] of the quasi-convex fn(s), one per tile, by golden section."""
    g = (math.sqrt(5.0) - 1.0) / 2.0
    a, b = np.full(n, -30.0), np.full(n, 30.0)
    x1, x2 = b - g * (b - a), a + g * (b - a)
    f1, f2 = fn(x1), fn(x2)
    best = np.minimum(f1, f2)
    for _ in range(60):
        low = f1 <= f2
        a, b = np.where(low, a, x1), np.where(low, x2, b)
        y1, y2 = np.where(low, b - g * (b - a), x2), np.where(low, x1, a + g * (b - a))
        x = np.where(low, y1, y2)
        f = fn(x)
        f1, f2 = np.where(low, f, f2), np.where(low, f1, f)
        x1, x2 = y1, y2
        best = np.minimum(best, f)
    return best


def _tilt(design, theta, verts):
    """g(s)[tile] = max_v (A(theta + q v) - A(theta)) / q - (A(theta + v) - A(theta)), q = 1 + e^s."""
    if design == "ztest1":
        A = lambda t: 0.5 * t * t  # noqa: E731
    else:
        A = lambda t: N_ARM * np.logaddexp(0.0, t)  # noqa: E731
    A0 = A(theta)[:, None, :]
    tv = A(theta[:, None, :] + verts) - A0

    def g(s):
        q = (1.0 + np.exp(s))[:, None, None]
        return ((A(theta[:, None, :] + q * verts) - A0) / q - tv).sum(2).max(1)
    return g


def _upper(g, a):
    """inf_q max_v of the Tilt-Bound U at f(theta) = a."""
    with np.errstate(divide="ignore", over="ignore", invalid="ignore"):
        la = np.log(a)

        def f(s):
            t = np.exp(s)
            v = la * (t / (1.0 + t)) + g(s)   # 1 - 1/q = (q - 1) / q
            return np.where(np.isfinite(v), v, np.inf)
        out = np.exp(np.minimum(_search(f, len(a)), 0.0))
    return np.where(a <= 0.0, 0.0, out)


def _inverse(g, alpha, n):
    """sup_q min_v U^{-1}(alpha)."""
    with np.errstate(over="ignore", invalid="ignore"):
        def f(s):
            t = np.exp(s)
            v = (math.log(alpha) - g(s)) * ((1.0 + t) / t)
            return np.where(np.isfinite(v), -v, np.inf)
        return np.exp(-_search(f, n))


def _vertices(theta, radii, clip):
    """Displacements of each tile's vertices: the box, or its part with theta1 <= theta0 where the
    box is cut along its diagonal (equal sides, equal centres)."""
    n, d = theta.shape
    if d == 1:
        return np.stack([-radii, radii], 1)
    v = np.stack([np.stack([sx * radii[:, 0], sy * radii[:, 1]], 1) for sx, sy in ((-1, -1), (1, -1), (-1, 1), (1, 1))], 1)
    if clip:
        cut = np.abs(theta[:, 0] - theta[:, 1]) < 0.5 * radii[:, 0]
        v[cut, 2] = v[cut, 3]   # (-, +) lies outside theta1 <= theta0
    return v


def _pooled_z():
    y0, y1 = np.meshgrid(np.arange(N_ARM + 1.0), np.arange(N_ARM + 1.0), indexing="ij")
    pbar = (y0 + y1) / (2.0 * N_ARM)
    inside = (pbar > 0) & (pbar < 1)
    se = np.sqrt(np.where(inside, pbar * (1.0 - pbar) * 2.0 / N_ARM, 1.0))
    return np.where(inside, (y1 / N_ARM - y0 / N_ARM) / se, 0.0).reshape(-1)


def _binom2_hist(w):
    """Yields (tile, histogram over the 36 x 36 outcomes) of every box."""
    n1 = N_ARM + 1
    top = int(w["sims"].max())
    words = np.empty((72, top), np.uint32)
    sim = np.arange(top)
    for b in range(18):
        words[4 * b: 4 * b + 4] = _philox(b, sim, w["seed"])
    T = np.clip(np.floor(2.0 ** 32 / (1.0 + np.exp(-w["theta"])) + 0.5), 0, 2 ** 32 - 1).astype(np.uint32)
    y, at = [], []
    for arm in (0, 1):
        u, inv = np.unique(T[:, arm], return_inverse=True)
        x = words[arm * N_ARM: (arm + 1) * N_ARM]
        y.append([(x < t).sum(0).astype(np.int16) for t in u])
        at.append(np.asarray(inv).reshape(-1))
    y[0] = [v * np.int16(n1) for v in y[0]]
    for t in range(len(T)):
        n = int(w["sims"][t])
        yield t, np.bincount(y[0][at[0][t]][:n] + y[1][at[1][t]][:n], minlength=n1 * n1)


def exact(case, seed):
    """float64 results by numpy: the z-test, and the 2-arm design up to 4e8 simulated tiles.  None
    for the larger grids (minutes) and for the designs whose statistic is a 90-node posterior
    per outcome or per look (minutes too); None for whole numbers and for the location q_star of
    a flat optimum."""
    design, op = case["design"], case["op"]
    if design not in ("ztest1", "binom2"):
        return None
    w = _grid(case, seed)
    theta, radii, N = w["theta"], w["radii"], w["sims"].astype(np.int64)
    n = len(N)
    if int(N.sum()) > 400_000_000:
        return None
    in_null = np.ones(n, bool)
    if design == "binom2":
        in_null = theta[:, 1] - theta[:, 0] < radii[:, 0]
    tilt = _tilt(design, theta, _vertices(theta, radii, design == "binom2"))
    out = {}
    ap = k = None
    if op in ("calibrate", "tiebreak"):
        ap = _inverse(tilt, ALPHA, n)
        k = np.floor((N + 1) * ap).astype(np.int64)
    R, lam = np.zeros(n, np.int64), np.full(n, -np.inf)
    if design == "ztest1":
        x = _philox(0, np.arange(int(N.max())), w["seed"])
        u0, u1 = (((v >> np.uint32(9)).astype(np.float64) + 0.5) / 2.0 ** 23 for v in x[:2])
        Z = np.sqrt(-2.0 * np.log(u0)) * np.cos(2.0 * np.pi * u1)
        sz = np.zeros(n)
        for t in range(n):
            z = Z[: N[t]]
            rej = theta[t, 0] + z > 1.96
            R[t], sz[t] = rej.sum(), z[rej].sum()
            if k is not None and k[t] > 0:
                lam[t] = np.partition(-(theta[t, 0] + z), k[t] - 1)[k[t] - 1]
        grad = (sz / N)[:, None]
        score = dict(score_Z=sz)
    else:
        z = _pooled_z()
        order = np.argsort(-z, kind="stable")
        S = -z[order]
        y0, y1 = np.divmod(np.arange(z.size), N_ARM + 1)
        rej = z > 1.96
        sums = np.stack([rej, rej * y0, rej * y1], 1).astype(np.int64)
        T = np.zeros((n, 2), np.int64)
        for t, h in _binom2_hist(w):
            R[t], T[t, 0], T[t, 1] = h @ sums
            if k is not None and k[t] > 0:
                lam[t] = S[np.searchsorted(np.cumsum(h[order]), k[t])]
        mean = N_ARM / (1.0 + np.exp(-theta))
        grad = (T - R[:, None] * mean) / N[:, None]
        score = dict(score_T=None)
    if op == "tie":
        r = np.random.Generator(np.random.PCG64(int(seed) + 1))
        return dict(tie=R / N, grad=r.standard_normal(n)[:, None] * grad)
    lam_min = np.array([lam[in_null].min()])
    if op == "tiebreak":
        return dict(alpha_prime=ap, k=None, lambda_tile=lam, u_tile=None, lambda_global=lam_min, u_global=None,
                    reject_at_lambda=None)
    cp = _cp_upper(R, N, DELTA)
    out = dict(reject=None, grad=grad, cp_upper=cp, tile_bound=_upper(tilt, cp), score_T=None, score_Z=None)
    out.update(score)
    if op == "calibrate":
        out.update(alpha_prime=ap, k=None, lambda_tile=lam, lambda_global=lam_min, reject_at_lambda=None)
        return out
    out["q_star"] = None
    if op == "validate":
        return out
    cl = 1.0 - _cp_upper(N - R, N, DELTA)
    low = dict(cp_lower=cl, lower=1.0 - _upper(tilt, 1.0 - cl), q_star=None)
    return dict(upper=out, lower=low)
