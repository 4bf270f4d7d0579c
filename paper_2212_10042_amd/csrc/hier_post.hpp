// hier_post.hpp -- float64 posterior of the four-arm hierarchical model of the basket case
// study (Section 10.1), per thread, for counts y_a out of n_a patients on arm a (arm 0 control):
//   theta_a | mu, s2 ~ N(mu, s2), mu ~ N(-1.34, 100), s2 ~ InvGamma(0.0005, 0.000005).
//
//   * mu is integrated out: theta | s2 ~ N(m0 1, Sigma), Sigma = s2 I + 100 11^T, with precision
//     Q = (I - c 11^T) / s2, c = 100 / (s2 + 400) (Sherman-Morrison);
//   * per node s2_j (90 nodes equally spaced in log s2 on [log 1e-6, log 1e3]) the conditional
//     posterior of theta is replaced by its Laplace approximation: the mode by Newton's method on
//     sum_a [y_a theta_a - n_a softplus(theta_a)] - (theta - m0)^T Q (theta - m0) / 2, whose
//     negative Hessian D - beta 11^T (D_a = n_a p_a (1 - p_a) + 1/s2, beta = c / s2) makes every
//     step, determinant and covariance C = D^{-1} + g u u^T (u = D^{-1} 1,
//     g = beta / (1 - beta sum u)) cost O(arms);
//   * node log weight: Laplace evidence l(mode) + log|Q|/2 - log|D - beta 11^T|/2, plus the log
//     inverse-gamma density of s2_j and the log trapezoid weight in log s2 (ds2 = s2 dlog s2),
//     normalised in float64;
//   * P_i = sum_j pi_j Phi(z_ij), z_ij = (mode_i - mode_0) / sqrt(C_ii + C_00 - 2 C_i0); the
//     complements 1 - P_i are summed directly as sum_j pi_j Phi(-z_ij) (relative precision where
//     P_i is near 1);
//   * for the Phase II/III design, the node mixture's moments: means and variances of theta_a and of
//     theta_i - theta_0 (variance = mean over nodes of C + spread of the modes, accumulated
//     about a fixed reference point so that no large terms cancel).
#pragma once
#include <math.h>

#include "cse_internal.h"
#include "fp64_math.hpp"

namespace cse {

constexpr int HP_NODES = 90;
// Tables: Newton stops after applying a step below this size: convergence is quadratic near the mode,
// so the remaining error is of the order of its square (~1e-12), below the 1e-10 step a fully
// converged iteration would still take.
constexpr double HP_NEWTON_TOL = 1e-6;

// Per-node constants (HierNode, cse_internal.h) are computed once on the host.

// 1/d for finite d > 0: hardware reciprocal and two Newton steps (error below one ulp).
// (The Phase II/III posterior's functions are compiled for the host too, for its tests: there by division.)
__host__ __device__ __forceinline__ double rcp_nr(double d) {
#ifdef __HIP_DEVICE_COMPILE__
    double r = __builtin_amdgcn_rcp(d);
    double e = fma(-d, r, 1.0);
    r = fma(r, e, r);
    e = fma(-d, r, 1.0);
    return fma(r, e, r);
#else
    return 1.0 / d;
#endif
}

// 1/sqrt(d) for finite d > 0: hardware estimate and two Newton steps (error about one ulp).
__host__ __device__ __forceinline__ double rsq_nr(double d) {
#ifdef __HIP_DEVICE_COMPILE__
    double y = __builtin_amdgcn_rsq(d);
    const double h = 0.5 * d;
    y = fma(y, fma(-h * y, y, 0.5), y);
    return fma(y, fma(-h * y, y, 0.5), y);
#else
    return 1.0 / sqrt(d);
#endif
}

// expit(x), and with it softplus(x) = max(x, 0) + log1p(exp(-|x|)) from the same exponential.
__device__ __forceinline__ double hp_expit(double x) {
    const double e = exp_cw(-fabs(x));          // in (0, 1]
    const double r = rcp_nr(1.0 + e);           // argument in (1, 2]
    return x >= 0.0 ? r : 1.0 - r;
}
__device__ __forceinline__ double hp_expit_softplus(double x, double &sp) {
    const double e = exp_cw(-fabs(x));
    const double r = rcp_nr(1.0 + e);
    sp = fmax(x, 0.0) + log1p_unit(e);
    return x >= 0.0 ? r : 1.0 - r;
}

// 1 / x_a for four finite positive x_a with one reciprocal: the reciprocal of their product
// times the other three factors (a few ulp; the products stay far inside the double range for
// the values here: 1 + e in (1, 2], curvatures in [1e-3, 1e6 + n/4]).  The treatment arms'
// cofactors are x0 times the product of the other two in ascending arm order, so arms 1..3
// with equal x get bit-identical results and ties between them stay exact ties.
__host__ __device__ __forceinline__ void rcp4(const double x[4], double r[4]) {
    const double x12 = x[1] * x[2], x13 = x[1] * x[3], x23 = x[2] * x[3];
    const double inv = rcp_nr(x[0] * (x12 * x[3]));
    r[0] = inv * (x12 * x[3]);
    r[1] = inv * (x[0] * x23);
    r[2] = inv * (x[0] * x13);
    r[3] = inv * (x[0] * x12);
}

struct HierSummary {
    double P[3];      // P(theta_i > theta_0 | data), i = 1..3
    double Sc[3];     // 1 - P_i
    double mean[4];   // mixture mean of theta_a
    double var[4];    // mixture variance of theta_a
    double dvar[3];   // mixture variance of theta_i - theta_0
};

// 1 - P_i (i = 1..3) of counts y[4] out of n[4]; every node's Newton iterations start at the
// empirical logits.
__device__ __forceinline__ void hier_complements(const int y[4], const double n[4], const HierNode *__restrict__ nodes,
                                                 double Sc[3]) {
    const double M0 = -1.34;
    float th0[4];
    double th[4];
    for (int a = 0; a < 4; ++a) {
        th[a] = log((y[a] + 0.5) / (n[a] - y[a] + 0.5));
        th0[a] = (float)th[a];
    }
    double wmax = -INFINITY, wsum = 0.0;
    double accS[3] = {0.0, 0.0, 0.0};
    for (int j = 0; j < HP_NODES; ++j) {
        const HierNode nd = nodes[j];   // uniform across lanes
        const double inv_s2 = nd.inv_s2, c = nd.c, beta = nd.beta;
        for (int a = 0; a < 4; ++a) th[a] = th0[a];
        double D[4], u[4], gam = 0.0;
        for (int it = 0; it < 100; ++it) {
            double dsum = 0.0;
            for (int a = 0; a < 4; ++a) dsum += th[a] - M0;
            double g[4], su = 0.0, q1[4], r1[4];
            for (int a = 0; a < 4; ++a) q1[a] = 1.0 + exp_cw(-fabs(th[a]));
            rcp4(q1, r1);   // expit(|theta_a|)
            for (int a = 0; a < 4; ++a) {
                const double p = th[a] >= 0.0 ? r1[a] : 1.0 - r1[a];
                // Q (theta - m0) = ((theta_a - m0) - c sum_b (theta_b - m0)) / s2
                g[a] = (double)y[a] - n[a] * p - ((th[a] - M0) - c * dsum) * inv_s2;
                D[a] = n[a] * p * (1.0 - p) + inv_s2;
            }
            rcp4(D, u);
            for (int a = 0; a < 4; ++a) su += u[a];
            gam = beta * rcp_nr(1.0 - beta * su);
            double ug = 0.0;
            for (int a = 0; a < 4; ++a) ug += u[a] * g[a];
            double mx = 0.0;
            for (int a = 0; a < 4; ++a) {
                const double step = u[a] * g[a] + gam * u[a] * ug;   // (D - beta 11^T)^{-1} g
                th[a] += step;
                mx = fmax(mx, fabs(step));
            }
            if (mx < HP_NEWTON_TOL) break;
        }
        // curvature at the final mode; log|D| as the log of the product (each D_a lies in
        // [1e-3, 1e6 + n/4], so the product of four cannot overflow)
        double su = 0.0, prodD = 1.0, ll = 0.0, dsum = 0.0, sq = 0.0;
        {
            double ex[4], q1[4], r1[4], q2[4], r2[4];
            for (int a = 0; a < 4; ++a) {
                ex[a] = exp_cw(-fabs(th[a]));
                q1[a] = 1.0 + ex[a];
                q2[a] = 2.0 + ex[a];   // in (2, 3]
            }
            rcp4(q1, r1);   // expit(|theta_a|)
            rcp4(q2, r2);   // for softplus: log1p(e) = 2 atanh(e / (2 + e))
            for (int a = 0; a < 4; ++a) {
                const double p = th[a] >= 0.0 ? r1[a] : 1.0 - r1[a];
                const double sp = fmax(th[a], 0.0) + log1p_from_u(ex[a] * r2[a]);
                D[a] = n[a] * p * (1.0 - p) + inv_s2;
                prodD *= D[a];
                ll += y[a] * th[a] - n[a] * sp;
                const double e = th[a] - M0;
                dsum += e;
                sq += e * e;
            }
        }
        rcp4(D, u);
        for (int a = 0; a < 4; ++a) su += u[a];
        gam = beta * rcp_nr(1.0 - beta * su);
        const double logdet_negH = log(prodD * (1.0 - beta * su));   // both factors in range
        const double quad = (sq - c * dsum * dsum) * inv_s2;
        const double lw = ll - 0.5 * quad - 0.5 * logdet_negH + nd.lconst;
        double pc[3];
        for (int i = 1; i < 4; ++i) {
            const double du = u[i] - u[0];
            const double vd = u[i] + u[0] + gam * du * du;
            pc[i - 1] = 0.5 * erfc((th[i] - th[0]) * rsq_nr(2.0 * vd));
        }
        if (lw > wmax) {
            const double sc = exp(wmax - lw);   // 0 on the first node
            wsum *= sc;
            for (int i = 0; i < 3; ++i) accS[i] *= sc;
            wmax = lw;
        }
        const double wj = exp(lw - wmax);
        wsum += wj;
        for (int i = 0; i < 3; ++i) accS[i] += wj * pc[i];
    }
    for (int i = 0; i < 3; ++i) Sc[i] = accS[i] / wsum;
}

// Phase II/III posterior: sums over nodes, all relative to the same weight exp(ref), so that the sums of
// ranges add up.
struct HierSums {
    double w, P[3], Sc[3], m1[4], m2[4], d2[3];
    float th0[4];   // reference point of the moments: the empirical logits
};

__host__ __device__ __forceinline__ void hier_zero(HierSums &H) {
    H.w = 0.0;
    for (int i = 0; i < 3; ++i) H.P[i] = H.Sc[i] = H.d2[i] = 0.0;
    for (int a = 0; a < 4; ++a) H.m1[a] = H.m2[a] = 0.0;
}

// A state's nodes are summed in HP_SEGS segments, whose sums are added in ascending order.  One lane takes them
// all or HP_SEGS lanes one each, so that the result is the same bits either way.
constexpr int HP_SEGS = 4;
// 1 - exp(-h) and exp(h) - 1 at the nodes' distance h = log(1e9) / 89
constexpr float HP_STEP_LO = 0.2077249f, HP_STEP_HI = 0.2621886f;
__host__ __device__ __forceinline__ int hp_seg(int s) { return HP_NODES * s / HP_SEGS; }   // its first node

// The sums of counts y[4] out of n[4] over nodes [j0, j1), H.th0 and ref given.  Bit i-1 of `need` (uniform over the wave)
// asks for P_i and 1 - P_i (the others are left 0).
//
// 90 nodes x (265 instructions per iteration + 400) per state and no memory traffic: the time is the
// operations, so
//   * the mode's start comes from the last four modes (backward differences in log s2, float32: only
//     a start; before a segment's second node from the first one's derivative), and each iteration adds
//     to Newton's step the second-order correction (Chebyshev's method): 1.25 iterations per node where
//     Newton's from the last two modes took 2.15;
//   * the values at the mode come from the last iteration's exponentials, times exp(-step) for the step
//     of at most HP_STEP_TOL;
//   * normal tails are erfc_pos, without branches, and only those that are asked for;
//   * the evidence's determinant enters the weight as 1 / sqrt, not through a logarithm, and weights are
//     relative to the likelihood at the empirical logits, not to a running maximum (their largest lies
//     between exp(-30) and exp(30) times that over all counts).
// Errors against 128-bit arithmetic over 20,000 states of the design's sample sizes (rms; in brackets all nodes as
// one segment): P 9.7e-13 (9.3e-13), 1 - P 8.3e-13 (8.1e-13), means 3.8e-14 (3.8e-14), variances 2.3e-13
// (2.2e-13).  Four segments cost 0.035 iterations per node: 11.88 ms of posteriors on the benchmark sample
// where one took 11.7 ms, but then each number of lanes gave a result of its own.
constexpr double HP_STEP_TOL = 1e-4;   // convergence is cubic: what remains is below 0.7 times its cube

__host__ __device__ __forceinline__ void hier_sums(const int y[4], const double n[4], const HierNode *nodes, int j0, int j1,
                                                   double ref, HierSums &H, int *newton_steps, int need) {
    const double M0 = -1.34;
    double th[4];
    HierNode nd = nodes[j0];
    {   // start of the range: the logits shrunk towards their common mean as normal ones would be
        double d[4], w[4], sw = 0.0, sm = 0.0;
        for (int a = 0; a < 4; ++a) {
            const double yes = y[a] + 0.5, no = n[a] - y[a] + 0.5;
            d[a] = nd.s2 + (yes + no) * rcp_nr(yes * no);
        }
        rcp4(d, w);
        for (int a = 0; a < 4; ++a) {
            sw += w[a];
            sm += w[a] * (double)H.th0[a];
        }
        const double mu = sm * rcp_nr(sw);
        for (int a = 0; a < 4; ++a) th[a] = mu + nd.s2 * w[a] * ((double)H.th0[a] - mu);
    }
    float last[4], df1[4], df2[4];   // the last mode and its backward differences
    for (int a = 0; a < 4; ++a) last[a] = df1[a] = df2[a] = 0.0f;
    hier_zero(H);
    for (int t = 0; j0 + t < j1; ++t) {
        const double inv_s2 = nd.inv_s2, c = nd.c, beta = nd.beta, lconst = nd.lconst;
        nd = nodes[j0 + t + 1 < HP_NODES ? j0 + t + 1 : HP_NODES - 1];
        for (int a = 0; a < 4 && t > 0; ++a) {
            const float cur = (float)th[a];
            const float e1 = cur - last[a], e2 = e1 - df1[a], e3 = e2 - df2[a];
            last[a] = cur;
            df1[a] = e1;
            df2[a] = e2;
            th[a] += (double)(e1 + e2 + e3);
        }
        double ex[4], top[4], u[4], gam;   // softplus(theta_a) = top_a + log1p(ex_a)
        for (int it = 0; it < 100; ++it) {
            double step[4], dsum = 0.0, q1[4], r1[4], g[4], D[4], T[4], su = 0.0, ug = 0.0;
            for (int a = 0; a < 4; ++a) {
                dsum += th[a] - M0;
                ex[a] = exp_short(-fabs(th[a]));
                q1[a] = 1.0 + ex[a];
            }
            rcp4(q1, r1);   // expit(|theta_a|)
            for (int a = 0; a < 4; ++a) {
                const double er = ex[a] * r1[a];   // expit(-|theta_a|)
                const double p = th[a] >= 0.0 ? r1[a] : er;
                const double nw = n[a] * (er * r1[a]);
                // Q (theta - m0) = ((theta_a - m0) - c sum_b (theta_b - m0)) / s2
                g[a] = fma(-n[a], p, (double)y[a]) - ((th[a] - M0) - c * dsum) * inv_s2;
                D[a] = nw + inv_s2;
                T[a] = nw * (p - 0.5);   // half the third derivative
            }
            rcp4(D, u);
            for (int a = 0; a < 4; ++a) {
                su += u[a];
                ug += u[a] * g[a];
            }
            gam = beta * rcp_nr(1.0 - beta * su);
            ug *= gam;
            double ub = 0.0, mx = 0.0;
            for (int a = 0; a < 4; ++a) {
                step[a] = u[a] * (g[a] + ug);   // (D - beta 11^T)^{-1} g
                T[a] *= step[a] * step[a];
                ub += u[a] * T[a];
            }
            ub *= gam;
            for (int a = 0; a < 4; ++a) {
                step[a] += u[a] * (T[a] + ub);
                mx = fmax(mx, fabs(step[a]));
            }
            if (newton_steps) *newton_steps += 1;
            if (mx < HP_STEP_TOL) {
                for (int a = 0; a < 4; ++a) {   // exp(-|theta|) of the mode (exp(|theta|) if the step crosses 0)
                    const double x = th[a] >= 0.0 ? -step[a] : step[a];
                    ex[a] *= fma(x, fma(x, fma(x, fma(x, 1.0 / 24.0, 1.0 / 6.0), 0.5), 1.0), 1.0);
                    top[a] = th[a] >= 0.0 ? th[a] + step[a] : 0.0;
                    th[a] += step[a];
                }
                break;
            }
            for (int a = 0; a < 4; ++a) th[a] += step[a];
            if (it == 99)   // not reached: the log posterior is concave
                for (int a = 0; a < 4; ++a) {
                    ex[a] = exp_short(-fabs(th[a]));
                    top[a] = fmax(th[a], 0.0);
                }
        }
        // at the mode; |D| as the product of its entries (each in [1e-3, 1e6 + n/4], so the product of
        // four cannot overflow)
        double su = 0.0, prodD = 1.0, ll = 0.0, dsum = 0.0, sq = 0.0, D[4];
        {
            double q1[4], r1[4], q2[4], r2[4];
            for (int a = 0; a < 4; ++a) {
                q1[a] = 1.0 + ex[a];
                q2[a] = 2.0 + ex[a];
            }
            rcp4(q1, r1);
            rcp4(q2, r2);   // log1p(e) = 2 atanh(e / (2 + e))
            for (int a = 0; a < 4; ++a) {
                const double sp = top[a] + log1p_short(ex[a] * r2[a]);
                D[a] = fma(n[a], ex[a] * r1[a] * r1[a], inv_s2);
                prodD *= D[a];
                ll += y[a] * th[a] - n[a] * sp;
                const double e = th[a] - M0;
                dsum += e;
                sq += e * e;
            }
        }
        rcp4(D, u);
        for (int a = 0; a < 4; ++a) su += u[a];
        const double om = 1.0 - beta * su;
        gam = beta * rcp_nr(om);
        if (t == 0) {   // the nodes before the range, from the mode's derivative in log s2, as a + b s2 or a + b / s2
            const float back = j0 < HP_NODES / 2 ? HP_STEP_LO : HP_STEP_HI, bend = j0 < HP_NODES / 2 ? HP_STEP_LO : -HP_STEP_HI;
            double q[4], uq = 0.0;
            for (int a = 0; a < 4; ++a) {
                q[a] = ((th[a] - M0) - c * dsum) * inv_s2;
                uq += u[a] * q[a];
            }
            for (int a = 0; a < 4; ++a) {
                const float d = (float)(u[a] * (q[a] + gam * uq)) * back;   // the last step
                last[a] = (float)th[a] - d;
                df1[a] = d * (1.0f - bend);
                df2[a] = df1[a] * bend;
            }
        }
        const double lw = (ll - ref) + (lconst - 0.5 * ((sq - c * dsum * dsum) * inv_s2));
        const double wj = exp_short(fmax(lw, -700.0)) * rsq_nr(prodD * om);   // both factors in range
        H.w += wj;
        for (int i = 1; i < 4; ++i) {
            const double du = u[i] - u[0], vd = u[i] + u[0] + gam * du * du;
            if ((need >> (i - 1)) & 1) {   // one tail gives both: the smaller side directly, the other as 1 - it
                const double zs = (th[i] - th[0]) * rsq_nr(2.0 * vd);
                const double tail = 0.5 * erfc_pos(fabs(zs), rcp_nr);
                H.Sc[i - 1] += wj * (zs >= 0.0 ? tail : 1.0 - tail);   // Phi(-z)
                H.P[i - 1] += wj * (zs >= 0.0 ? 1.0 - tail : tail);    // Phi(z)
            }
            const double e = (th[i] - th[0]) - (H.th0[i] - H.th0[0]);
            H.d2[i - 1] += wj * (vd + e * e);
        }
        for (int a = 0; a < 4; ++a) {
            const double e = th[a] - H.th0[a];
            H.m1[a] += wj * e;
            H.m2[a] += wj * (u[a] + gam * u[a] * u[a] + e * e);   // C_aa + (mode - ref)^2
        }
    }
}

// T += H, each sum of H as `at` gives it.
template <class At>
__host__ __device__ __forceinline__ void hier_add(HierSums &T, const HierSums &H, At at) {
    T.w += at(H.w);
    for (int i = 0; i < 3; ++i) {
        T.P[i] += at(H.P[i]);
        T.Sc[i] += at(H.Sc[i]);
        T.d2[i] += at(H.d2[i]);
    }
    for (int a = 0; a < 4; ++a) {
        T.m1[a] += at(H.m1[a]);
        T.m2[a] += at(H.m2[a]);
    }
}

// Segments [s0, s1), one after the other.
__host__ __device__ __forceinline__ void hier_segments(const int y[4], const double n[4], const HierNode *nodes, int s0, int s1,
                                                       HierSums &T, int *newton_steps, int need) {
    HierSums H;
    double ref = 0.0;   // the log likelihood at the empirical logits
    for (int a = 0; a < 4; ++a) {
        const double th = log((y[a] + 0.5) / (n[a] - y[a] + 0.5));
        H.th0[a] = T.th0[a] = (float)th;
        ref += y[a] * th - n[a] * softplus_fast(th);
    }
    hier_zero(T);
    for (int s = s0; s < s1; ++s) {
        hier_sums(y, n, nodes, hp_seg(s), hp_seg(s + 1), ref, H, newton_steps, need);
        hier_add(T, H, [](double v) { return v; });
    }
}

// All segments, by this lane alone or (shared, uniform) one by each of HP_SEGS neighbouring lanes, which all call.
__device__ __forceinline__ void hier_all(const int y[4], const double n[4], const HierNode *nodes, bool shared, HierSums &T,
                                         int *newton_steps, int need) {
    const int part = (int)threadIdx.x & (HP_SEGS - 1);
    hier_segments(y, n, nodes, shared ? part : 0, shared ? part + 1 : HP_SEGS, T, newton_steps, need);
    if (shared) {
        const HierSums H = T;
        hier_zero(T);
        for (int s = 0; s < HP_SEGS; ++s) hier_add(T, H, [&](double v) { return __shfl(v, s, HP_SEGS); });
    }
}

__host__ __device__ __forceinline__ void hier_summary(const HierSums &H, HierSummary &out) {
    for (int i = 0; i < 3; ++i) {
        out.Sc[i] = H.Sc[i] / H.w;
        out.P[i] = H.P[i] / H.w;
    }
    double em[4];
    for (int a = 0; a < 4; ++a) {
        em[a] = H.m1[a] / H.w;                       // mean - reference
        out.mean[a] = H.th0[a] + em[a];
        out.var[a] = H.m2[a] / H.w - em[a] * em[a];
    }
    for (int i = 0; i < 3; ++i) {
        const double ed = em[i + 1] - em[0];
        out.dvar[i] = H.d2[i] / H.w - ed * ed;
    }
}

// Posterior of counts y[4] out of n[4], all nodes.
__device__ __forceinline__ void hier_posterior(const int y[4], const double n[4], const HierNode *__restrict__ nodes,
                                               HierSummary &out, int *newton_steps, int need) {
    HierSums H;
    hier_segments(y, n, nodes, 0, HP_SEGS, H, newton_steps, need);
    hier_summary(H, out);
}

// Basket design (Section 10.1's validation case study): arm a against its fixed rate,
// theta0[a] = logit p_0a; the hierarchical model is on the offsets theta_a - theta0[a], so in
// theta the prior mean is m0 + theta0[a] per arm with the same covariance, and the statistic
// of arm a is P(theta_a > theta0[a] | y).  Writes the complements
// Sc[a] = sum_j pi_j Phi(-(mode_a - theta0[a]) / sqrt(C_aa)), C_aa = u_a + g u_a^2.
__device__ __forceinline__ void basket_posterior(const int y[4], double n, const double theta0[4],
                                                 const HierNode *__restrict__ nodes, double Sc[4]) {
    const double M0 = -1.34;
    double mean[4], th[4];
    for (int a = 0; a < 4; ++a) {
        mean[a] = M0 + theta0[a];
        th[a] = log((y[a] + 0.5) / (n - y[a] + 0.5));
    }
    double wmax = -INFINITY, wsum = 0.0, acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int j = 0; j < HP_NODES; ++j) {
        const HierNode nd = nodes[j];   // uniform across lanes
        const double inv_s2 = nd.inv_s2, c = nd.c, beta = nd.beta;
        double D[4], u[4], gam = 0.0;
        for (int it = 0; it < 100; ++it) {   // warm start: the previous node's mode
            double dsum = 0.0;
            for (int a = 0; a < 4; ++a) dsum += th[a] - mean[a];
            double g[4], su = 0.0;
            for (int a = 0; a < 4; ++a) {
                const double p = hp_expit(th[a]);
                g[a] = (double)y[a] - n * p - ((th[a] - mean[a]) - c * dsum) * inv_s2;
                D[a] = n * p * (1.0 - p) + inv_s2;
                u[a] = rcp_nr(D[a]);
                su += u[a];
            }
            gam = beta * rcp_nr(1.0 - beta * su);
            double ug = 0.0;
            for (int a = 0; a < 4; ++a) ug += u[a] * g[a];
            double mx = 0.0;
            for (int a = 0; a < 4; ++a) {
                const double step = u[a] * g[a] + gam * u[a] * ug;
                th[a] += step;
                mx = fmax(mx, fabs(step));
            }
            if (mx < HP_NEWTON_TOL) break;
        }
        double su = 0.0, prodD = 1.0, ll = 0.0, dsum = 0.0, sq = 0.0;
        for (int a = 0; a < 4; ++a) {
            double sp;
            const double p = hp_expit_softplus(th[a], sp);
            D[a] = n * p * (1.0 - p) + inv_s2;
            u[a] = rcp_nr(D[a]);
            su += u[a];
            prodD *= D[a];
            ll += y[a] * th[a] - n * sp;
            const double e = th[a] - mean[a];
            dsum += e;
            sq += e * e;
        }
        gam = beta * rcp_nr(1.0 - beta * su);
        const double logdet_negH = log(prodD * (1.0 - beta * su));   // both factors in range
        const double quad = (sq - c * dsum * dsum) * inv_s2;
        const double lw = ll - 0.5 * quad - 0.5 * logdet_negH + nd.lconst;
        double pc[4];
        for (int a = 0; a < 4; ++a) {
            const double caa = u[a] + gam * u[a] * u[a];
            pc[a] = 0.5 * erfc((th[a] - theta0[a]) / sqrt(2.0 * caa));   // Phi(-z)
        }
        if (lw > wmax) {
            const double sc = exp(wmax - lw);   // 0 on the first node
            wsum *= sc;
            for (int a = 0; a < 4; ++a) acc[a] *= sc;
            wmax = lw;
        }
        const double wj = exp(lw - wmax);
        wsum += wj;
        for (int a = 0; a < 4; ++a) acc[a] += wj * pc[a];
    }
    for (int a = 0; a < 4; ++a) Sc[a] = acc[a] / wsum;
}

}  // namespace cse
