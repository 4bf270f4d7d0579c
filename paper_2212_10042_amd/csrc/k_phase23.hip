// k_phase23.hip -- the Phase II/III Bayesian selection design (Section 10.2 and the design
// appendix), one simulated trial per lane, decisions from the hierarchical posterior of
// hier_post.hpp (float64) at every look.
//
// Protocol (the reading of the appendix):
//   Phase II: 50 patients per arm; looks after 200, 300 and 400 randomised patients.  At each
//   look, for every active treatment arm i: p_best_i = P(theta_i is the largest of the four)
//   under independent normal marginals moment-matched to the posterior mixture (16-point
//   Gauss-Hermite), and p_succ_i = probability under a Gaussian predictive that adding 200
//   patients to arm i and to control gives P(theta_i > theta_0) > 0.95 at the end.  If some
//   active arm has p_succ > 0.70 (0.60 at the third look) the one with the largest p_best among
//   them is selected (ties: lowest index); otherwise, at looks 1-2, arms with p_best < 0.15 are
//   dropped (futility when none remains) and the next 100 patients are split evenly over the
//   remaining arms and control, the remainder discarded; at look 3 the trial stops.
//   Phase III: 100 + 100 on the selected arm s and control, interim: success if
//   P(theta_s > theta_0) > 0.95, futility if p_succ_s (100 added) < 0.20; else 100 + 100 more and
//   the final analysis.
//   Embedding (Section 9): patient j of arm a draws word a * 350 + j of the simulation's stream.
//   Statistic of a tile with null configuration b: -inf for an early success with s in b,
//   1 - P_final(theta_s > theta_0) for a final analysis with s in b, +inf otherwise; the
//   design's rule at lambda rejects (falsely) when S < lambda.
//
// The first look always has 50 patients per arm, so its decision is precomputed per outcome (51^4
// bytes, the same decision code run once per outcome when the platten is created).  Looks compute
// only the normal tails they use (none in Phase II, the selected arm's in Phase III).  Per trial: the
// key S is stored, and a rejection at the fixed lambda adds to the tile's R and to its sums of the
// observed counts and sample sizes (integer atomics: exact, order-independent).  All tiles together
// go look by look (k_p23_open, k_p23_post, k_p23_step); one tile by itself goes through k_phase23.
#include <math.h>

#include "cse_internal.h"
#include "hier_post.hpp"
#include "kernels.h"
#include "philox.hpp"

namespace cse {

namespace {

constexpr int P23_NMAX = 350;   // embedded patients per arm

// Add m patients to arm a (patients n .. n+m-1): count responses among their words.
__device__ __forceinline__ void p23_draw(int a, int m, uint32_t T, uint32_t k, uint32_t key0,
                                         uint32_t key1, int &n, int &y) {
    if (m <= 0) return;
    const uint32_t w0 = (uint32_t)(a * P23_NMAX + n), w1 = w0 + (uint32_t)m;   // [w0, w1)
    int cnt = 0;
    for (uint32_t b = w0 >> 2; b <= (w1 - 1) >> 2; ++b) {
        const u32x4 w = philox_block(b, k, key0, key1);
        const uint32_t base = b << 2;
        cnt += (base + 0 >= w0 && base + 0 < w1 && w.x < T) ? 1 : 0;
        cnt += (base + 1 >= w0 && base + 1 < w1 && w.y < T) ? 1 : 0;
        cnt += (base + 2 >= w0 && base + 2 < w1 && w.z < T) ? 1 : 0;
        cnt += (base + 3 >= w0 && base + 3 < w1 && w.w < T) ? 1 : 0;
    }
    n += m;
    y += cnt;
}

__device__ __forceinline__ double p23_Phi(double z) { return 0.5 * erfc(-z / sqrt(2.0)); }

// p_succ for d ~ N(md, vd), control / arm posterior means m0, mi, m_add patients per arm.
__device__ __forceinline__ double p23_psucc(double md, double vd, double m0, double mi, double m_add,
                                            double z95) {
    const double p0 = hp_expit(m0), pi = hp_expit(mi);
    const double V = 1.0 / (m_add * pi * (1.0 - pi)) + 1.0 / (m_add * p0 * (1.0 - p0));
    const double vf = vd * V / (vd + V);
    const double sd_mean = vd / sqrt(vd + V);
    return p23_Phi((md - z95 * sqrt(vf)) / sd_mean);
}

// Pairs of treatment arms with equal counts and sizes (bit 0: arms 1, 2; bit 1: 1, 3; bit 2: 2, 3).
__device__ __forceinline__ int p23_ties(int y1, int y2, int y3, int n1, int n2, int n3) {
    return ((y1 == y2 && n1 == n2) ? 1 : 0) | ((y1 == y3 && n1 == n3) ? 2 : 0) | ((y2 == y3 && n2 == n3) ? 4 : 0);
}

// Decision at Phase II look `look` (0..2) for the active treatment arms (bit i-1 = arm i):
// code = sel | (active after drops) << 2 | stop << 5, sel = 0 when no arm is selected.  Among
// the arms that qualify the largest p_best wins, the lowest index on ties; arms with equal
// counts and sizes have equal posteriors (exchangeable model), so they tie exactly whatever
// rounding their computed p_best carries: `ties` bit 0 (arms 1, 2), bit 1 (1, 3), bit 2 (2, 3).
__device__ __forceinline__ int p23_phase2(const HierSummary &s, int ties, int look, int active, const double *gh,
                                          double sqrt_pi, double z95) {
    const double thr = (look < 2) ? 0.70 : 0.60;
    int qual = 0;   // active arms with p_succ above the threshold
#pragma unroll
    for (int i = 1; i < 4; ++i)
        if (((active >> (i - 1)) & 1) &&
            p23_psucc(s.mean[i] - s.mean[0], s.dvar[i - 1], s.mean[0], s.mean[i], 200.0, z95) > thr)
            qual |= 1 << (i - 1);
    // p_best of the arms it is asked of: several that qualify, or those that may be dropped
    const int want = qual ? ((qual & (qual - 1)) ? qual : 0) : (look == 2 ? 0 : active);
    double pb[4] = {0.0, 0.0, 0.0, 0.0};
    if (want) {
        double isd[4];   // 1 / (sd * sqrt 2): Phi(z / sd) = erfc(-z isd) / 2
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) isd[kk] = rsq_nr(2.0 * s.var[kk]);
#pragma unroll
        for (int i = 1; i < 4; ++i) {
            if (!((want >> (i - 1)) & 1)) continue;
            const double si = sqrt(2.0 * s.var[i]);
            double acc = 0.0;
            for (int g = 0; g < 16; ++g) {
                const double t = s.mean[i] + si * gh[g];
                double prod = 1.0;
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) {
                    if (kk == i) continue;
                    const double x = (t - s.mean[kk]) * isd[kk], v = 0.5 * erfc_pos(fabs(x), rcp_nr);
                    prod *= x > 0.0 ? 1.0 - v : v;   // Phi(sqrt 2 x)
                }
                acc += gh[16 + g] * prod;
            }
            pb[i] = acc / sqrt_pi;
        }
    }
    int best = 0;
    double pb_best = 0.0;
#pragma unroll
    for (int i = 1; i < 4; ++i) {
        if (!((qual >> (i - 1)) & 1)) continue;
        const bool same = best != 0 && ((ties >> (best + i - 3)) & 1);   // best < i
        if (best == 0 || (pb[i] > pb_best && !same)) {
            best = i;
            pb_best = pb[i];
        }
    }
    if (best) return best | (active << 2);
    if (look == 2) return (active << 2) | (1 << 5);
#pragma unroll
    for (int i = 1; i < 4; ++i)
        if (((active >> (i - 1)) & 1) && pb[i] < 0.15) active &= ~(1 << (i - 1));
    return (active << 2) | ((active == 0 ? 1 : 0) << 5);
}

// Sample sizes between Phase II looks (50 + 25, 33 or 50 per step), by 4-bit code.
__device__ __forceinline__ int p23_ncode(int n) {
    return n == 50 ? 0 : (n == 75 ? 1 : (n == 83 ? 2 : (n == 100 ? 3 : (n == 108 ? 4 : (n == 116 ? 5 : (n == 125 ? 6 : (n == 133 ? 7 : 8)))))));
}
__device__ __forceinline__ int p23_ncode_size(int c) {
    return c == 0 ? 50 : (c == 1 ? 75 : (c == 2 ? 83 : (c == 3 ? 100 : (c == 4 ? 108 : (c == 5 ? 116 : (c == 6 ? 125 : (c == 7 ? 133 : 150)))))));
}

// The state of a trial about to be looked at, treatment arms in a canonical order (position p holds
// arm (perm >> 2 p) & 3): Phase II by (active, size, count), ties in arm order, so that "the lowest
// index among tied arms" is the same arm in both orders; Phase III the selected arm first, then the
// others.  Bits: y0..y3 9 each, size codes 4 each (without the patients of Phase III), look 3,
// active 3, top bit set.
__device__ __forceinline__ uint64_t p23_state(const int y[4], const int n[4], int look, int sel, int active, uint32_t &perm) {
    const int extra = look >= 3 ? 100 * (look - 2) : 0;   // Phase III patients of control and the selected arm
    uint32_t c[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const bool s = look >= 3 && sel == i + 1;
        const int code = p23_ncode(n[i + 1] - (s ? extra : 0));
        const uint32_t first = look >= 3 ? (s ? 0u : 1u) : (uint32_t)((active >> i) & 1);
        c[i] = (((first << 4 | (uint32_t)code) << 9 | (uint32_t)y[i + 1]) << 2) | (uint32_t)(i + 1);
    }
    auto order = [](uint32_t &a, uint32_t &b) {
        const uint32_t lo = min(a, b), hi = max(a, b);
        a = lo;
        b = hi;
    };
    order(c[0], c[1]);
    order(c[1], c[2]);
    order(c[0], c[1]);
    perm = (c[0] & 3u) | (c[1] & 3u) << 2 | (c[2] & 3u) << 4;
    uint64_t s = (uint64_t)y[0] | (uint64_t)p23_ncode(n[0] - extra) << 36;
    uint32_t act = 0u;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        s |= (uint64_t)((c[p] >> 2) & 511u) << (9 * (p + 1)) | (uint64_t)((c[p] >> 11) & 15u) << (36 + 4 * (p + 1));
        if (look < 3) act |= ((c[p] >> 15) & 1u) << p;
    }
    return s | (uint64_t)look << 52 | (uint64_t)act << 55 | 1ull << 63;
}

// A Phase II code's arms from positions back to arms.
__device__ __forceinline__ int p23_arms(int code, uint32_t perm) {
    const int sel = code & 3, act = (code >> 2) & 7;
    int a_sel = 0, a_act = 0;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        const int arm = (int)((perm >> (2 * p)) & 3u);
        if (sel == p + 1) a_sel = arm;
        if ((act >> p) & 1) a_act |= 1 << (arm - 1);
    }
    return a_sel | a_act << 2 | (code & 32);
}

}  // namespace

// Decision of the first look (50 patients per arm) for every outcome y in {0..50}^4, index
// ((y0 51 + y1) 51 + y2) 51 + y3; the trials take it from here instead of a posterior.
__global__ __launch_bounds__(128) void k_p23_look1(int64_t n_out, uint8_t *__restrict__ tbl,
                                                   const HierNode *__restrict__ nodes,
                                                   const double *__restrict__ gh, double sqrt_pi, double z95) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n_out) return;
    int y[4];
    int64_t v = idx;
    for (int a = 3; a >= 0; --a) {
        y[a] = (int)(v % 51);
        v /= 51;
    }
    const double n[4] = {50.0, 50.0, 50.0, 50.0};
    HierSummary s;
    hier_posterior(y, n, nodes, s, nullptr, 0);
    tbl[idx] = (uint8_t)p23_phase2(s, p23_ties(y[1], y[2], y[3], 50, 50, 50), 0, 7, gh, sqrt_pi, z95);
}

hipError_t launch_p23_look1(const Platten &P, hipStream_t st) {
    const int64_t n_out = 51LL * 51 * 51 * 51;
    hipLaunchKernelGGL(k_p23_look1, dim3((uint32_t)((n_out + 127) / 128)), dim3(128), 0, st, n_out, P.d_p23look1,
                       P.d_hnodes, P.d_gh, P.p23.sqrt_pi, P.p23.z95);
    return hipGetLastError();
}

// A state's outcome and the iterations of its posterior; shared (uniform): HP_SEGS neighbouring lanes have the same
// state and share its nodes.  Functions of their own, not inlined: the constants of their polynomials are then held
// in registers over one loop at a time, not over all loops of a kernel at once; and both paths below form
// the same bits.
#define P23_EVAL __device__ __attribute__((noinline))
__device__ __forceinline__ void p23_counts(uint64_t s, int extra, int y[4], int n[4]) {
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        y[a] = (int)((s >> (9 * a)) & 511u);
        n[a] = p23_ncode_size((int)((s >> (36 + 4 * a)) & 15u)) + (a < 2 ? extra : 0);
    }
}
// Phase II: the decision code, by position.
P23_EVAL uint2 p23_eval2(uint64_t s, bool shared, const HierNode *nodes, const double *gh, double sqrt_pi, double z95) {
    int y[4], n[4], steps = 0;
    p23_counts(s, 0, y, n);
    const double nd[4] = {(double)n[0], (double)n[1], (double)n[2], (double)n[3]};
    HierSums H;
    HierSummary h;
    hier_all(y, nd, nodes, shared, H, &steps, 0);
    hier_summary(H, h);
    return make_uint2((uint32_t)p23_phase2(h, p23_ties(y[1], y[2], y[3], n[1], n[2], n[3]), (int)((s >> 52) & 7u),
                                           (int)((s >> 55) & 7u), gh, sqrt_pi, z95),
                      (uint32_t)steps);
}
// Phase III (the selected arm is at position 1): interim 0 (go on), 1 (success) or 2 (futility), final analysis the
// bits of the float32 statistic.
__device__ __forceinline__ uint32_t p23_phase3(const HierSummary &h, int look, double z95) {
    if (look == 4) return __float_as_uint((float)h.Sc[0]);
    if (h.P[0] > 0.95) return 1u;
    return p23_psucc(h.mean[1] - h.mean[0], h.dvar[0], h.mean[0], h.mean[1], 100.0, z95) < 0.20 ? 2u : 0u;
}
P23_EVAL uint2 p23_eval3(uint64_t s, bool shared, const HierNode *nodes, double z95) {
    const int look = (int)((s >> 52) & 7u);
    int y[4], n[4], steps = 0;
    p23_counts(s, 100 * (look - 2), y, n);
    const double nd[4] = {(double)n[0], (double)n[1], (double)n[2], (double)n[3]};
    HierSums H;
    HierSummary h;
    hier_all(y, nd, nodes, shared, H, &steps, 1);
    hier_summary(H, h);
    return make_uint2(p23_phase3(h, look, z95), (uint32_t)steps);
}

// Either, for the lanes of a wave in any phase (tail, uniform: some are in Phase III).
P23_EVAL uint2 p23_eval(uint64_t s, bool tail, const HierNode *nodes, const double *gh, double sqrt_pi, double z95) {
    const int look = (int)((s >> 52) & 7u);
    int y[4], n[4], steps = 0;
    p23_counts(s, look >= 3 ? 100 * (look - 2) : 0, y, n);
    const double nd[4] = {(double)n[0], (double)n[1], (double)n[2], (double)n[3]};
    HierSums H;
    HierSummary h;
    hier_all(y, nd, nodes, false, H, &steps, tail ? 1 : 0);
    hier_summary(H, h);
    const int code = look < 3 ? p23_phase2(h, p23_ties(y[1], y[2], y[3], n[1], n[2], n[3]), look, (int)((s >> 55) & 7u), gh, sqrt_pi,
                                           z95)
                              : (int)p23_phase3(h, look, z95);
    return make_uint2((uint32_t)code, (uint32_t)steps);
}

// One tile by itself, trial by trial: a persistent grid; each wave pops items (simulation ranges) from
// a global queue, and every lane runs its own trial as a state machine, one posterior per step, and
// takes the next simulation as soon as its trial ends, so lanes whose trials stop early do not wait
// for long ones.
// Two waves per SIMD: the float64 posterior keeps about 250 registers live.
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_phase23(P23Args A) {
    const int lane = threadIdx.x & (WAVE - 1);
    const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (WAVE - lane));
    // wave-uniform current item
    int32_t it_tile = -1;
    uint32_t it_k = 0, it_end = 0;
    bool queue_open = true;

    // lane state: busy = a trial in progress; add[a] = patients to enrol on arm a before the
    // next look; look 0..2 Phase II, 3 Phase III interim, 4 final analysis
    bool busy = false;
    int32_t tile = 0;
    uint32_t k = 0, T[4] = {0u, 0u, 0u, 0u};
    int cfg = 0, look = 0, sel = 0, active = 0;
    int n[4] = {0, 0, 0, 0}, y[4] = {0, 0, 0, 0}, add[4] = {0, 0, 0, 0};
    int c_trials = 0, c_look2 = 0, c_look3 = 0, c_newton = 0;   // this lane's work (stats counters)

    bool fresh = false, done = false;
    float S = INFINITY;
    // Phase II decision code -> next enrolment (or the end of the trial)
    auto apply = [&](int code) {
        const int s_arm = code & 3;
        if (s_arm) {
            sel = s_arm;
#pragma unroll
            for (int a = 0; a < 4; ++a) add[a] = (a == 0 || a == s_arm) ? 100 : 0;
            look = 3;
        } else if ((code >> 5) & 1) {
            done = true;
        } else {
            active = (code >> 2) & 7;
            const int per = 100 / (__popc(active) + 1);
#pragma unroll
            for (int a = 0; a < 4; ++a) add[a] = (a == 0 || ((active >> (a - 1)) & 1)) ? per : 0;
            look += 1;
        }
    };
    // the trial's result: its key, and the rejection sums when S is below the cut
    auto finish = [&]() {
        if (A.keys) A.keys[A.key_off[tile] + k] = S;
        if (S < A.cut) {
            atomicAdd(&A.R[tile], 1u);
            if (A.sumT)
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    atomicAdd(&A.sumT[(int64_t)tile * 8 + a], (unsigned long long)y[a]);
                    atomicAdd(&A.sumT[(int64_t)tile * 8 + 4 + a], (unsigned long long)n[a]);
                }
        }
        busy = false;
        c_trials += 1;
    };

    for (;;) {
        // ---- give idle lanes the next simulations of the wave's item stream and run their first
        // look (a table lookup); a trial that ends there is finished at once and its lane takes
        // another, so that lanes do not sit out the posterior below ----
        for (;;) {
            unsigned long long need = __ballot(!busy);
            while (need) {
                if (it_k >= it_end) {
                    if (!queue_open) break;
                    uint32_t idx = 0;
                    if (lane == 0) idx = atomicAdd(A.counter, 1u);
                    idx = __builtin_amdgcn_readfirstlane(idx);
                    if ((int64_t)idx >= A.n_items) {
                        queue_open = false;
                        break;
                    }
                    const WorkItem W = A.items[idx];
                    it_tile = W.blk;
                    it_k = W.k_begin;
                    it_end = W.k_end;
                    continue;
                }
                const uint32_t avail = it_end - it_k;
                const uint32_t rank = (uint32_t)__popcll(need & below);
                if (((need >> lane) & 1ull) && rank < avail) {
                    busy = true;
                    fresh = true;
                    tile = it_tile;
                    k = it_k + rank;
                    for (int a = 0; a < 4; ++a) {
                        T[a] = A.tileT[(int64_t)tile * 4 + a];
                        n[a] = 0;
                        y[a] = 0;
                    }
                    cfg = A.cfg[tile];
                    look = 0;
                    sel = 0;
                    active = 7;
                }
                const uint32_t asked = (uint32_t)__popcll(need);
                it_k += asked < avail ? asked : avail;
                need = __ballot(!busy);
            }
            if (!__ballot(fresh)) break;   // nobody was given a trial: all lanes busy, or queue drained
            if (fresh) {
                // Phase II opens with 50 patients per arm; the first look's decision is tabulated
                fresh = false;
                done = false;
                S = INFINITY;
#pragma unroll
                for (int a = 0; a < 4; ++a) p23_draw(a, 50, T[a], k, A.key0, A.key1, n[a], y[a]);
                apply(A.look1[((y[0] * 51 + y[1]) * 51 + y[2]) * 51 + y[3]]);
                if (done) finish();
            }
        }
        if (!__ballot(busy)) break;   // queue drained and every trial finished
        if (busy) {
            // ---- enrol the patients of the next look, then one posterior look ----
#pragma unroll
            for (int a = 0; a < 4; ++a) p23_draw(a, add[a], T[a], k, A.key0, A.key1, n[a], y[a]);
            uint32_t perm;
            const uint64_t st = p23_state(y, n, look, sel, active, perm);
            const uint2 o = p23_eval(st, __ballot(look >= 3) != 0ull, A.nodes, A.gh, A.sqrt_pi, A.z95);
            c_newton += (int)o.y;
            if (look < 3) {
                c_look2 += 1;
                apply(p23_arms((int)o.x, perm));
            } else {
                const uint32_t out = o.x;
                c_look3 += 1;
                const bool in_b = (cfg >> (sel - 1)) & 1;
                done = true;
                if (look == 4) {
                    S = in_b ? __uint_as_float(out) : INFINITY;   // final analysis
                } else if (out == 1u) {
                    S = in_b ? -INFINITY : INFINITY;              // early success
                } else if (out == 0u) {
                    done = false;
#pragma unroll
                    for (int a = 0; a < 4; ++a) add[a] = (a == 0 || a == sel) ? 100 : 0;
                    look = 4;
                }
            }
            if (done) finish();
        }
    }
    if (A.stats) {
        // one atomic per counter and wave: reduce the lane counters across the wave first
        unsigned long long c[4] = {(unsigned long long)c_trials, (unsigned long long)c_look2,
                                   (unsigned long long)c_look3, (unsigned long long)c_newton};
#pragma unroll
        for (int i = 0; i < 4; ++i)
            for (int off = 32; off >= 1; off >>= 1) c[i] += __shfl_xor(c[i], off);
        if (lane == 0)
#pragma unroll
            for (int i = 0; i < 4; ++i) atomicAdd(&A.stats[i], c[i]);
    }
}

// ------------------------------------------------------------------------------------------
// All tiles together, look by look.  A look's outcome depends only on the trial's counts and sample
// sizes, and trials meet the same ones over and over (two null configurations of a box are the same
// trials; neighbouring tiles and simulations of a tile share counts; the treatment arms are
// exchangeable): of the benchmark sample's 37.5 million looks past the first, a seventh are distinct.
// So each look's posterior is evaluated once per distinct state of the call:
//   * k_p23_count: the successes of every simulation at every sample size, once per threshold (tiles
//     share thresholds), so that enrolling an arm is one load.  Above P23_TABLE_MAX bytes there is no
//     such table and trials draw their own words.  Benchmark sample: open 4.1 ms and the steps 2.6 ms
//     without it, 0.79 ms for the table, 0.75 and 1.4 ms with it;
//   * k_p23_open: every trial's first 50 patients per arm, the tabulated first look, and the
//     enrolment up to the next look; a trial that goes on leaves a record with its state's slot;
//   * k_p23_post: the posterior of every new state, one per lane, and the look's outcome into the
//     slot (states of Phase II and of Phase III in separate waves: they need different tails);
//   * k_p23_step: every open trial's outcome applied, its next patients enrolled, its next slot.
// post and step run once per look (at most four after the first).  The slots are an open-addressed
// table of 64-bit states (treatment arms sorted: p23_state) with at least as many places as trials (up
// to 2^27), cleared at the start of the call; a state that finds no place within P23_PROBES gets a
// slot of its own and is evaluated for its trial alone.  Trials go in chunks of p23_cap.
//
// open and step are bound by the latency of their loads and by counters that every workgroup adds to:
// one addition per wave and list made them 9.4, 9.1, 3.9 and 0.6 ms on the benchmark sample (23.3
// million trials), about 10 ns per addition to a line.  So a workgroup keeps its trials in a range of
// its own from the first look on, collects new slots in LDS for P23_STEPS passes, and adds once: 0.75,
// 0.8, 0.4 and 0.2 ms.  post (4.2, 5.3, 1.9 and 0.4 ms) is float64 arithmetic (hier_sums; 6.4, 8.3, 2.9
// and 0.6 ms with Newton's method and the library's functions).  All together: 144.8 ms trial by trial,
// 17 ms so.
// ------------------------------------------------------------------------------------------
namespace {

// Enrol arm a up to n patients in all (of them 100 phase in Phase III): its successes from the count
// table, or counted among the new patients' words.
__device__ __forceinline__ void p23_enrol(const P23Args &A, uint32_t tile, uint32_t k, int a, int add, int phase, int &n,
                                          int &y) {
    if (A.counts) {   // uniform
        n += add;
        const uint2 r = A.tile_row[4 * (int64_t)tile + a];
        const uint32_t c = (uint32_t)(p23_ncode(n - 100 * phase) + P23_NSIZE * phase);
        y = (int)A.counts[(size_t)(r.x + c * r.y) * 64u + k];
    } else {
        p23_draw(a, add, A.tileT[4 * (int64_t)tile + a], k, A.key0, A.key1, n, y);
    }
}

constexpr int P23_PROBES = 32;

// A wave's new slots since the last flush (Phase II from the front, Phase III from the back), and the
// workgroup's counts.
constexpr int P23_STEPS = 4;                    // passes of the workgroup between flushes
constexpr int P23_FRESH = P23_STEPS * WAVE;
struct P23Fresh {
    uint32_t *list;
    int n2 = 0, n3 = 0;   // uniform
};
struct P23Lds {
    uint32_t list[WG / WAVE][P23_FRESH];
    uint32_t n[WG / WAVE][2];
    uint32_t base[2];
    uint32_t begin, kept;
};

// The slot of state s: in the table, or one of its own.  Every lane of the wave calls; open: this lane
// has a state.  New states are appended to the round's list of their phase.
__device__ __forceinline__ uint32_t p23_slot(const P23Memo &M, int round, bool open, uint64_t s, P23Fresh &F) {
    const int lane = threadIdx.x & (WAVE - 1);
    uint32_t slot = 0u;
    bool fresh = false;
    if (open) {
        uint64_t h = s * 0x9E3779B97F4A7C15ull;
        h ^= h >> 32;
        h *= 0xD6E8FEB86659FD93ull;
        slot = (uint32_t)(h >> 32) & M.mask;
        int i = 0;
        for (; i < P23_PROBES; ++i) {
            unsigned long long *at = M.state + slot;
            unsigned long long cur = __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (cur == 0ull) {
                cur = atomicCAS(at, 0ull, (unsigned long long)s);
                if (cur == 0ull) {
                    fresh = true;
                    break;
                }
            }
            if (cur == s) break;
            slot = (slot + 1u) & M.mask;
        }
        if (i == P23_PROBES) {
            const uint32_t o = atomicAdd(M.count(round, 2), 1u);   // at most one per open trial
            M.own[o] = s;
            slot = M.mask + 1u + o;
            fresh = true;
        }
    }
    const bool p3 = ((s >> 52) & 7u) >= 3u;
    const unsigned long long below = (1ull << lane) - 1ull;
    const unsigned long long f2 = __ballot(fresh && !p3), f3 = __ballot(fresh && p3);
    if (fresh) {
        const int at = p3 ? P23_FRESH - 1 - (F.n3 + __popcll(f3 & below)) : F.n2 + __popcll(f2 & below);
        F.list[at] = slot;
    }
    F.n2 += __popcll(f2);
    F.n3 += __popcll(f3);
    return slot;
}

// The waves' new slots appended to the round's lists (the whole workgroup calls).
__device__ __forceinline__ void p23_flush(const P23Memo &M, int round, P23Fresh &F, P23Lds &L) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (lane < 2) L.n[wv][lane] = (uint32_t)(lane ? F.n3 : F.n2);
    __syncthreads();
    uint32_t off[2] = {0u, 0u}, all[2] = {0u, 0u};
#pragma unroll
    for (int w = 0; w < WG / WAVE; ++w)
#pragma unroll
        for (int ph = 0; ph < 2; ++ph) {
            if (w < wv) off[ph] += L.n[w][ph];
            all[ph] += L.n[w][ph];
        }
    if (threadIdx.x == 0 && all[0]) L.base[0] = atomicAdd(M.count(round, 0), all[0]);
    if (threadIdx.x == WAVE && all[1]) L.base[1] = atomicAdd(M.count(round, 1), all[1]);
    __syncthreads();
    for (int i = lane; i < F.n2; i += WAVE) M.list[0][L.base[0] + off[0] + (uint32_t)i] = F.list[i];
    for (int i = lane; i < F.n3; i += WAVE) M.list[1][L.base[1] + off[1] + (uint32_t)i] = F.list[P23_FRESH - 1 - i];
    F.n2 = F.n3 = 0;
}

// A trial between looks.
struct P23State {
    uint32_t tile, k;
    int y[4], n[4];
    int look, sel, active;
};

// Phase II outcome (code of p23_phase2) -> enrolment before the next look, or the end (returns true).
__device__ __forceinline__ bool p23_apply(int code, P23State &t, int add[4]) {
    const int s_arm = code & 3;
    if (s_arm) {
        t.sel = s_arm;
#pragma unroll
        for (int a = 0; a < 4; ++a) add[a] = (a == 0 || a == s_arm) ? 100 : 0;
        t.look = 3;
        return false;
    }
    if ((code >> 5) & 1) return true;
    t.active = (code >> 2) & 7;
    const int per = 100 / (__popc(t.active) + 1);
#pragma unroll
    for (int a = 0; a < 4; ++a) add[a] = (a == 0 || ((t.active >> (a - 1)) & 1)) ? per : 0;
    t.look += 1;
    return false;
}

__device__ __forceinline__ void p23_finish(const P23Args &A, const P23State &t, float S) {
    if (A.keys) A.keys[A.key_off[t.tile] + t.k] = S;
    if (S < A.cut) {
        atomicAdd(&A.R[t.tile], 1u);
        if (A.sumT)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                atomicAdd(&A.sumT[(int64_t)t.tile * 8 + a], (unsigned long long)t.y[a]);
                atomicAdd(&A.sumT[(int64_t)t.tile * 8 + 4 + a], (unsigned long long)t.n[a]);
            }
    }
}

// The records of the lanes whose trials go on, into the workgroup's range (every lane calls).
__device__ __forceinline__ void p23_keep(const P23Memo &M, int round, bool open, const P23State &t, uint32_t begin,
                                         P23Fresh &F, P23Lds &L) {
    const int lane = threadIdx.x & (WAVE - 1);
    uint32_t perm = 0u;
    const unsigned long long bal = __ballot(open);
    if (!bal) return;
    const uint64_t s = open ? p23_state(t.y, t.n, t.look, t.sel, t.active, perm) : 0ull;
    const uint32_t slot = p23_slot(M, round, open, s, F);
    uint32_t at = 0u;
    if (lane == 0) at = atomicAdd(&L.kept, (uint32_t)__popcll(bal));
    at = begin + (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
    if (open) {
        uint4 *__restrict__ r = M.trial[round & 1] + 2 * (size_t)(at + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull)));
        r[0] = make_uint4(t.tile, t.k, slot, (uint32_t)t.look | (uint32_t)t.sel << 3 | (uint32_t)t.active << 5 | perm << 8);
        r[1] = make_uint4((uint32_t)t.y[0] | (uint32_t)t.y[1] << 16, (uint32_t)t.y[2] | (uint32_t)t.y[3] << 16,
                          (uint32_t)t.n[0] | (uint32_t)t.n[1] << 16, (uint32_t)t.n[2] | (uint32_t)t.n[3] << 16);
    }
}

}  // namespace

// Count table: one workgroup per (chunk of 64 simulations, arm); the arm's 350 words go to LDS, each
// wave takes the arm's thresholds P23C_T at a time and stores the running counts at every sample size.
constexpr int P23C_T = 4;
__global__ __launch_bounds__(WG) void k_p23_count(const P23Row *__restrict__ rows, int4 first, int4 end, uint32_t key0,
                                                  uint32_t key1, uint16_t *__restrict__ out) {
    constexpr int NWV = WG / WAVE;
    constexpr int NB = (P23_NMAX + 3 + 3) / 4;   // blocks that hold an arm's words at any alignment
    __shared__ uint32_t words[4 * NB][WAVE];
    const int lane = threadIdx.x & (WAVE - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t chunk = blockIdx.x;
    const int arm = (int)blockIdx.y;
    const uint32_t k = chunk * WAVE + (uint32_t)lane;
    const uint32_t b0 = (uint32_t)(arm * P23_NMAX) >> 2, w0 = (uint32_t)(arm * P23_NMAX) & 3u;
    for (int b = wv; b < NB; b += NWV) {
        const u32x4 w = philox_block(b0 + (uint32_t)b, k, key0, key1);
        words[4 * b + 0][lane] = w.x;
        words[4 * b + 1][lane] = w.y;
        words[4 * b + 2][lane] = w.z;
        words[4 * b + 3][lane] = w.w;
    }
    __syncthreads();
    const int r0 = arm == 0 ? first.x : (arm == 1 ? first.y : (arm == 2 ? first.z : first.w));
    const int r1 = arm == 0 ? end.x : (arm == 1 ? end.y : (arm == 2 ? end.z : end.w));
    for (int r = r0 + wv * P23C_T; r < r1; r += NWV * P23C_T) {   // uniform over the wave
        uint32_t T[P23C_T], y[P23C_T];
#pragma unroll
        for (int i = 0; i < P23C_T; ++i) {
            T[i] = r + i < r1 ? rows[r + i].T : 0u;
            y[i] = 0u;
        }
        int done = 0;
        for (int n = 50; n <= P23_NMAX;) {   // the sample sizes in ascending order
            for (int j = done; j < n; ++j) {
                const uint32_t x = words[w0 + j][lane];
#pragma unroll
                for (int i = 0; i < P23C_T; ++i) y[i] += x < T[i] ? 1u : 0u;
            }
            done = n;
            int next = P23_NMAX + 1;
#pragma unroll
            for (int c = 0; c < P23_SIZES; ++c) {
                const int m = p23_ncode_size(c % P23_NSIZE) + 100 * (c / P23_NSIZE);
                if (m == n) {
#pragma unroll
                    for (int i = 0; i < P23C_T; ++i)
                        if (r + i < r1 && chunk < rows[r + i].stride)
                            out[((size_t)rows[r + i].at + (size_t)c * rows[r + i].stride + chunk) * WAVE + lane] = (uint16_t)y[i];
                } else if (m > n && m < next) {
                    next = m;
                }
            }
            n = next;
        }
    }
}

// Workgroup b takes the items [per b, per b + per) and a range of the records as long as their trials.
__global__ __launch_bounds__(WG) void k_p23_open(P23Args A, P23Memo M, int per) {
    __shared__ P23Lds L;
    const int i0 = (int)blockIdx.x * per, i1 = min((int)A.n_items, i0 + per);
    if (threadIdx.x == 0) {
        uint32_t n = 0;
        for (int i = i0; i < i1; ++i) n += A.items[i].k_end - A.items[i].k_begin;
        L.begin = atomicAdd(M.trials(), n);
        L.kept = 0u;
    }
    __syncthreads();
    const uint32_t begin = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.begin);
    P23Fresh F;
    F.list = L.list[threadIdx.x >> 6];
    int pass = 0;
    for (int i = i0; i < i1; ++i) {   // uniform
        const WorkItem W = A.items[i];
        for (uint32_t k0 = W.k_begin; k0 < W.k_end; k0 += WG) {   // uniform
            const uint32_t k = k0 + threadIdx.x;
            bool open = k < W.k_end;
            P23State t;
            t.tile = (uint32_t)W.blk;
            t.k = k;
            t.look = t.sel = 0;
            t.active = 7;
#pragma unroll
            for (int a = 0; a < 4; ++a) t.y[a] = t.n[a] = 0;
            if (open) {
                int add[4] = {50, 50, 50, 50};
#pragma unroll
                for (int a = 0; a < 4; ++a) p23_enrol(A, t.tile, k, a, add[a], 0, t.n[a], t.y[a]);
                if (p23_apply(A.look1[((t.y[0] * 51 + t.y[1]) * 51 + t.y[2]) * 51 + t.y[3]], t, add)) {
                    p23_finish(A, t, INFINITY);
                    open = false;
                } else {
#pragma unroll
                    for (int a = 0; a < 4; ++a)
                        if (add[a]) p23_enrol(A, t.tile, k, a, add[a], t.look == 3 ? 1 : 0, t.n[a], t.y[a]);
                }
            }
            p23_keep(M, 0, open, t, begin, F, L);
            if (++pass == P23_STEPS) {
                p23_flush(M, 0, F, L);
                pass = 0;
            }
        }
    }
    p23_flush(M, 0, F, L);   // ends the counting of L.kept
    if (threadIdx.x == 0) M.range[blockIdx.x] = make_uint2(begin, L.kept);
}

// Outcome of every new state of the round, one per lane or, where they are few, per `split` lanes: Phase
// II the decision code, Phase III interim 0 (go on), 1 (success) or 2 (futility), final analysis the bits
// of the float32 statistic.  Bound by its vector instructions, 740 per node and wave of 64 states, which
// take 93% of the cycles with two waves per SIMD (three measure the same).
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(P23_WAVES, P23_WAVES))) void k_p23_post(
    P23Args A, P23Memo M, int round) {
    const int lane = threadIdx.x & (WAVE - 1);
    const uint32_t wave = blockIdx.x * (WG / WAVE) + (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t waves = gridDim.x * (WG / WAVE);
    const uint32_t n2 = *M.count(round, 0), n3 = *M.count(round, 1);
    // Lanes per state: the batches that a wave takes one after the other, times the time of a lane's nodes
    // (a quarter more where lanes of a wave are at different nodes, since the wave iterates as long as its
    // slowest lane) and of a start and an end, about five nodes.  Rounds of the 3^4 x 1,024 grid with one
    // lane per state: 275, 280, 155 and 147 us; the last two, with HP_SEGS lanes, 61 and 51 us.  The outcome
    // is the same bits either way (hier_all).
    int split = 1;
    uint32_t best = ~0u;
    for (int q = 1; q <= HP_SEGS; q *= HP_SEGS) {
        const uint32_t nb = (n2 * q + WAVE - 1) / WAVE + (n3 * q + WAVE - 1) / WAVE;
        const uint32_t cost = ((nb + waves - 1) / waves) * (uint32_t)((q == 1 ? HP_NODES : HP_NODES * 5 / 4 / q) + 5);
        if (cost < best) {
            best = cost;
            split = q;
        }
    }
    const uint32_t b2 = (n2 * split + WAVE - 1) / WAVE, b3 = (n3 * split + WAVE - 1) / WAVE;
    int c_newton = 0;
    for (uint32_t b = wave; b < b2 + b3; b += waves) {   // uniform
        const bool p3 = b >= b2;
        const uint32_t i = ((p3 ? b - b2 : b) * WAVE + (uint32_t)lane) >> __builtin_ctz(split), last = (p3 ? n3 : n2) - 1u;
        const uint32_t slot = M.list[p3 ? 1 : 0][min(i, last)];
        const uint64_t s = slot <= M.mask ? M.state[slot] : M.own[slot - M.mask - 1u];
        const uint2 o = p3 ? p23_eval3(s, split > 1, A.nodes, A.z95)   // (uniform branch)
                           : p23_eval2(s, split > 1, A.nodes, A.gh, A.sqrt_pi, A.z95);
        if (i <= last) {
            c_newton += (int)o.y;
            if ((lane & (split - 1)) == 0) M.value[slot] = o.x;
        }
    }
    if (A.stats) {
        unsigned long long c = (unsigned long long)c_newton;
        for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off);
        if (lane == 0 && c) atomicAdd(&A.stats[3], c);
        if (wave == 0 && lane == 0) {
            if (round == 0) atomicAdd(&A.stats[0], (unsigned long long)*M.trials());
            atomicAdd(&A.stats[1], (unsigned long long)n2);
            atomicAdd(&A.stats[2], (unsigned long long)n3);
        }
    }
}

__global__ __launch_bounds__(WG) void k_p23_step(P23Args A, P23Memo M, int round) {
    __shared__ P23Lds L;
    const uint2 range = M.range[blockIdx.x];
    if (range.y == 0u) return;   // uniform
    if (threadIdx.x == 0) L.kept = 0u;
    __syncthreads();
    P23Fresh F;
    F.list = L.list[threadIdx.x >> 6];
    int pass = 0;
    for (uint32_t i0 = 0; i0 < range.y; i0 += WG) {   // uniform
        const uint32_t i = i0 + threadIdx.x;
        bool open = i < range.y;
        P23State t{};
        if (open) {
            const uint4 *__restrict__ r = M.trial[round & 1] + 2 * (size_t)(range.x + i);
            const uint4 u = r[0], v = r[1];
            t.tile = u.x;
            t.k = u.y;
            t.look = (int)(u.w & 7u);
            t.sel = (int)((u.w >> 3) & 3u);
            t.active = (int)((u.w >> 5) & 7u);
            const uint32_t perm = u.w >> 8;
            t.y[0] = (int)(v.x & 0xFFFFu);
            t.y[1] = (int)(v.x >> 16);
            t.y[2] = (int)(v.y & 0xFFFFu);
            t.y[3] = (int)(v.y >> 16);
            t.n[0] = (int)(v.z & 0xFFFFu);
            t.n[1] = (int)(v.z >> 16);
            t.n[2] = (int)(v.w & 0xFFFFu);
            t.n[3] = (int)(v.w >> 16);
            const uint32_t out = M.value[u.z];
            int add[4] = {0, 0, 0, 0};
            float S = INFINITY;
            bool done;
            if (t.look < 3) {
                done = p23_apply(p23_arms((int)out, perm), t, add);
            } else {
                const bool in_b = (A.cfg[t.tile] >> (t.sel - 1)) & 1;
                done = true;
                if (t.look == 4) {
                    S = in_b ? __uint_as_float(out) : INFINITY;   // final analysis
                } else if (out == 1u) {
                    S = in_b ? -INFINITY : INFINITY;              // early success
                } else if (out == 0u) {
                    done = false;
#pragma unroll
                    for (int a = 0; a < 4; ++a) add[a] = (a == 0 || a == t.sel) ? 100 : 0;
                    t.look = 4;
                }
            }
            if (done) {
                p23_finish(A, t, S);
                open = false;
            } else {
#pragma unroll
                for (int a = 0; a < 4; ++a)
                    if (add[a]) p23_enrol(A, t.tile, t.k, a, add[a], t.look >= 3 ? t.look - 2 : 0, t.n[a], t.y[a]);
            }
        }
        p23_keep(M, round + 1, open, t, range.x, F, L);
        if (++pass == P23_STEPS) {
            p23_flush(M, round + 1, F, L);
            pass = 0;
        }
    }
    p23_flush(M, round + 1, F, L);   // ends the counting of L.kept
    if (threadIdx.x == 0) M.range[blockIdx.x].y = L.kept;
}

namespace {
// Trials of items [i0, i1) (at most M.cap), all rounds.
hipError_t p23_run(const Platten &P, P23Args A, const WorkItem *items, int64_t n_items, int64_t grid, hipStream_t st) {
    P23Memo M = P.p23memo;
    A.items = items;
    A.n_items = n_items;
    hipError_t e = launch_zero(M.ctr, P23_COUNTERS * P23_CTR * sizeof(uint32_t), st);
    if (e != hipSuccess) return e;
    const int per = (int)((n_items + P23_BLOCKS - 1) / P23_BLOCKS);
    const uint32_t blocks = (uint32_t)((n_items + per - 1) / per);
    hipLaunchKernelGGL(k_p23_open, dim3(blocks), dim3(WG), 0, st, A, M, per);
    for (int r = 0; r + 1 < P23_ROUNDS; ++r) {
        hipLaunchKernelGGL(k_p23_post, dim3((uint32_t)grid), dim3(WG), 0, st, A, M, r);
        hipLaunchKernelGGL(k_p23_step, dim3(blocks), dim3(WG), 0, st, A, M, r);
    }
    return hipGetLastError();
}
}  // namespace

// Work items in chunks whose trials fit the records.
hipError_t launch_phase23_list(const Platten &P, uint64_t seed, const WorkItem *d_items, const WorkItem *h_items,
                               int64_t n_items, int64_t grid, uint32_t *R, unsigned long long *sumT, float *keys,
                               unsigned long long *stats, hipStream_t st) {
    P23Args A = P.p23;
    A.key0 = (uint32_t)seed;
    A.key1 = (uint32_t)(seed >> 32);
    A.R = R;
    A.sumT = sumT;
    A.keys = keys;
    A.stats = stats;
    hipError_t e = launch_zero(P.p23memo.state, ((size_t)P.p23memo.mask + 1) * sizeof(unsigned long long), st);
    if (e != hipSuccess) return e;
    if (P.d_p23counts)
        hipLaunchKernelGGL(k_p23_count, dim3((uint32_t)P.p23_chunks, 4), dim3(WG), 0, st, P.d_p23row,
                           make_int4(P.p23_arm_row[0], P.p23_arm_row[1], P.p23_arm_row[2], P.p23_arm_row[3]),
                           make_int4(P.p23_arm_row[1], P.p23_arm_row[2], P.p23_arm_row[3], P.p23_arm_row[4]), A.key0, A.key1,
                           P.d_p23counts);
    for (int64_t i = 0; i < n_items;) {
        int64_t j = i, trials = 0;
        while (j < n_items && (j == i || trials + (h_items[j].k_end - h_items[j].k_begin) <= P.p23_cap))
            trials += h_items[j].k_end - h_items[j].k_begin, ++j;
        if ((e = p23_run(P, A, d_items + i, j - i, grid, st)) != hipSuccess) return e;
        i = j;
    }
    return hipSuccess;
}

hipError_t launch_phase23(const Platten &P, uint64_t seed, uint32_t *R, unsigned long long *sumT, float *keys,
                          hipStream_t st) {
    const hipError_t e = launch_zero(P.d_p23stats, 4 * sizeof(unsigned long long), st);
    if (e != hipSuccess) return e;
    return launch_phase23_list(P, seed, P.d_p23items, P.p23_items.data(), (int64_t)P.p23_items.size(), P.p23_grid, R,
                               sumT, keys, P.d_p23stats, st);
}

// The plain path: one launch per tile over that tile's own queue items (no other tiles share
// the grid); counts only.
hipError_t launch_phase23_tile(const Platten &P, uint64_t seed, int64_t t, uint32_t *R_tile, hipStream_t st) {
    hipError_t e = launch_zero(P.d_queue, sizeof(uint32_t), st);
    if (e != hipSuccess) return e;
    P23Args A = P.p23;
    const int64_t i0 = P.p23_item_off[t], i1 = P.p23_item_off[t + 1];
    A.items = P.d_p23items + i0;
    A.n_items = i1 - i0;
    A.key0 = (uint32_t)seed;
    A.key1 = (uint32_t)(seed >> 32);
    A.R = R_tile - t;   // the kernel indexes R by tile id
    A.sumT = nullptr;
    A.keys = nullptr;
    A.stats = nullptr;
    hipLaunchKernelGGL(k_phase23, dim3((uint32_t)((A.n_items + 3) / 4)), dim3(WG), 0, st, A);
    return hipGetLastError();
}

}  // namespace cse
