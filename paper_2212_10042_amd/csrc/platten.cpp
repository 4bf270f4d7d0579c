// platten.cpp -- host side of the platten (Section 5, Definition 1): the null partition of
// each box, the vertices of every tile (float64), the Bernoulli thresholds, the design
// tables and the tile batches ("blocks") the kernels run.  Everything is uploaded once.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <functional>
#include <map>
#include <mutex>
#include <numeric>
#include <chrono>
#include <tuple>

#include "cse_internal.h"
#include "kernels.h"
#include "value_slot.hpp"

namespace cse {

static thread_local std::string g_err;
void set_error(const std::string &msg) { g_err = msg; }
const char *get_error() { return g_err.c_str(); }

namespace {

// Bernoulli(expit theta) from one uniform 32-bit word u: success iff u < T,
// T = round(2^32 / (1 + exp(-theta))), clamped to [0, 2^32 - 1].
uint32_t bern_threshold(double theta) {
    double p = 1.0 / (1.0 + exp(-theta));
    double t = floor(p * 4294967296.0 + 0.5);
    if (t < 0.0) t = 0.0;
    if (t > 4294967295.0) t = 4294967295.0;
    return (uint32_t)t;
}

// Pooled two-proportion z for y0 (control) and y1 (treatment) successes out of n each;
// 0 when the pooled rate is 0 or 1.
double pooled_z(int y0, int y1, int n) {
    double pbar = (double)(y0 + y1) / (2.0 * n);
    if (pbar <= 0.0 || pbar >= 1.0) return 0.0;
    double se = sqrt(pbar * (1.0 - pbar) * 2.0 / n);
    return ((double)y1 / n - (double)y0 / n) / se;
}

// Half-space g . x <= h.
struct HalfSpace {
    double g[MAX_D];
    double h;
};

// Solve the d x d system A x = b by Gaussian elimination with partial pivoting.
bool solve(int d, double A[MAX_D][MAX_D], double b[MAX_D], double x[MAX_D]) {
    for (int c = 0; c < d; ++c) {
        int piv = c;
        for (int r = c + 1; r < d; ++r)
            if (fabs(A[r][c]) > fabs(A[piv][c])) piv = r;
        if (fabs(A[piv][c]) < 1e-12) return false;
        if (piv != c) {
            for (int j = 0; j < d; ++j) std::swap(A[c][j], A[piv][j]);
            std::swap(b[c], b[piv]);
        }
        for (int r = c + 1; r < d; ++r) {
            double f = A[r][c] / A[c][c];
            for (int j = c; j < d; ++j) A[r][j] -= f * A[c][j];
            b[r] -= f * b[c];
        }
    }
    for (int r = d - 1; r >= 0; --r) {
        double s = b[r];
        for (int j = r + 1; j < d; ++j) s -= A[r][j] * x[j];
        x[r] = s / A[r][r];
    }
    return true;
}

// Vertices of the polytope {x : g_i . x <= h_i} (bounded by construction: it lies in a box).
// Every vertex is the solution of d active constraints; enumerate all d-subsets.
std::vector<std::vector<double>> enumerate_vertices(int d, const std::vector<HalfSpace> &H) {
    std::vector<std::vector<double>> V;
    const int m = (int)H.size();
    std::vector<int> idx(d);
    std::function<void(int, int)> rec = [&](int start, int depth) {
        if (depth == d) {
            double A[MAX_D][MAX_D], b[MAX_D], x[MAX_D];
            for (int r = 0; r < d; ++r) {
                for (int j = 0; j < d; ++j) A[r][j] = H[idx[r]].g[j];
                b[r] = H[idx[r]].h;
            }
            if (!solve(d, A, b, x)) return;
            for (int i = 0; i < m; ++i) {
                double s = 0.0;
                for (int j = 0; j < d; ++j) s += H[i].g[j] * x[j];
                if (s > H[i].h + 1e-12 * (1.0 + fabs(H[i].h))) return;
            }
            for (auto &v : V) {
                double dm = 0.0;
                for (int j = 0; j < d; ++j) dm = std::max(dm, fabs(v[j] - x[j]));
                if (dm <= 1e-12) return;
            }
            V.emplace_back(x, x + d);
            return;
        }
        for (int i = start; i < m; ++i) {
            idx[depth] = i;
            rec(i + 1, depth + 1);
        }
    };
    rec(0, 0);
    return V;
}

// 16-point Gauss-Hermite rule (weight e^{-x^2}): the nodes are the zeros of H_16, found by
// Newton's method on the orthonormal Hermite functions h_k (h_0 = pi^{-1/4},
// h_{k+1} = x sqrt(2/(k+1)) h_k - sqrt(k/(k+1)) h_{k-1}, h_16' = sqrt(32) h_15) from starting
// points bracketed by sign changes on a grid; weight 1 / (16 h_15(x)^2).
void gauss_hermite16(double *x, double *w) {
    const int n = 16;
    auto eval = [&](double t, double &hn, double &hn1) {
        double a = pow(M_PI, -0.25), b = sqrt(2.0) * t * a;
        for (int k = 1; k < n; ++k) {
            const double c = t * sqrt(2.0 / (k + 1)) * b - sqrt((double)k / (k + 1)) * a;
            a = b;
            b = c;
        }
        hn = b;
        hn1 = a;
    };
    int found = 0;
    double prev = -7.0, fp, dummy;
    eval(prev, fp, dummy);
    for (int g = 1; g <= 1400 && found < n; ++g) {
        const double t = -7.0 + 0.01 * g;
        double ft;
        eval(t, ft, dummy);
        if ((fp < 0.0) != (ft < 0.0)) {
            double r = 0.5 * (prev + t);
            for (int it = 0; it < 50; ++it) {
                double hn, hn1;
                eval(r, hn, hn1);
                const double step = hn / (sqrt(2.0 * n) * hn1);
                r -= step;
                if (fabs(step) < 1e-16 * (1.0 + fabs(r))) break;
            }
            double hn, hn1;
            eval(r, hn, hn1);
            x[found] = r;
            w[found] = 1.0 / (n * hn1 * hn1);
            ++found;
        }
        prev = t;
        fp = ft;
    }
}

// Node constants of the hierarchical posterior (Section 10.1 model: mu ~ N(-1.34, 100) integrated
// out, s2 ~ InvGamma(0.0005, 0.000005), trapezoid rule in log s2 with ds2 = s2 dlog s2).
std::vector<HierNode> hier_nodes() {
    const double TAU2 = 100.0, IG_A = 0.0005, IG_B = 0.000005;
    const double LS2_LO = log(1e-6), LS2_HI = log(1e3);
    const double h = (LS2_HI - LS2_LO) / (HIER_NODES - 1);
    std::vector<HierNode> v(HIER_NODES);
    for (int j = 0; j < HIER_NODES; ++j) {
        HierNode &nd = v[j];
        nd.ls2 = LS2_LO + h * j;
        nd.s2 = exp(nd.ls2);
        nd.inv_s2 = 1.0 / nd.s2;
        nd.c = TAU2 / (nd.s2 + 4.0 * TAU2);
        nd.beta = nd.c * nd.inv_s2;
        const double logdetQ = -(3.0 * nd.ls2 + log(nd.s2 + 4.0 * TAU2));   // determinant lemma
        const double logprior = IG_A * log(IG_B) - lgamma(IG_A) - (IG_A + 1.0) * nd.ls2 - IG_B * nd.inv_s2;
        const double logtrap = log((j == 0 || j == HIER_NODES - 1) ? 0.5 * h : h) + nd.ls2;
        nd.lconst = 0.5 * logdetQ + logprior + logtrap;
    }
    return v;
}

// Phi^{-1}(0.95) by Newton's method on Phi(z) = erfc(-z / sqrt 2) / 2.
double normal_q95() {
    double z = 1.6;
    for (int it = 0; it < 50; ++it) {
        const double f = 0.5 * erfc(-z / sqrt(2.0)) - 0.95;
        const double dens = exp(-0.5 * z * z) / sqrt(2.0 * M_PI);
        const double step = f / dens;
        z -= step;
        if (fabs(step) < 1e-16) break;
    }
    return z;
}

// Side streams of destroyed plattens, per device, for reuse (creating one costs ~35 us and
// destroying it ~30 us; a platten is destroyed only after the device has been synchronised,
// so a cached stream is idle).  Default priority, non-blocking.
std::mutex g_stream_mu;
std::map<int, std::vector<hipStream_t>> g_stream_cache;
constexpr size_t STREAM_CACHE_MAX = 16;

hipError_t take_side_stream(int device, hipStream_t *s) {
    {
        std::lock_guard<std::mutex> g(g_stream_mu);
        auto &v = g_stream_cache[device];
        if (!v.empty()) {
            *s = v.back();
            v.pop_back();
            return hipSuccess;
        }
    }
    return hipStreamCreateWithFlags(s, hipStreamNonBlocking);
}

void give_side_stream(int device, hipStream_t s) {
    {
        std::lock_guard<std::mutex> g(g_stream_mu);
        auto &v = g_stream_cache[device];
        if (v.size() < STREAM_CACHE_MAX) {
            v.push_back(s);
            return;
        }
    }
    (void)hipStreamDestroy(s);
}

// Count table of the last destroyed platten, per device (one buffer, at most B2_TABLE_MAX bytes and a
// little), for the next one: adaptive runs create a platten per round, and allocations of tens of MB cost
// ~190 us each.  A platten gives its table back after its own device has been synchronised.  The buffer is
// freed when a platten needs a larger one, when an allocation of the library fails (dev_malloc), and by
// cse_release_cached_memory.
struct TableBuf {
    void *p = nullptr;
    size_t bytes = 0;
};
std::mutex g_table_mu;
std::map<int, TableBuf> g_table_cache;
constexpr size_t TABLE_CACHE_MIN = (size_t)2 << 20;   // smaller allocations are cheap

// Frees the buffer of `device`, which is current; false when there is none.
bool drop_table(int device) {
    TableBuf t;
    {
        std::lock_guard<std::mutex> g(g_table_mu);
        std::swap(t, g_table_cache[device]);
    }
    if (t.p) (void)hipFree(t.p);
    return t.p != nullptr;
}

hipError_t take_table(int device, size_t bytes, TableBuf *t) {
    if (bytes >= TABLE_CACHE_MIN) {
        {
            std::lock_guard<std::mutex> g(g_table_mu);
            TableBuf &c = g_table_cache[device];
            if (c.bytes >= bytes) {
                *t = c;
                c = TableBuf();
                return hipSuccess;
            }
        }
        drop_table(device);
    }
    t->bytes = bytes;
    return dev_malloc(&t->p, bytes);
}

void give_table(int device, TableBuf t) {
    {
        std::lock_guard<std::mutex> g(g_table_mu);
        TableBuf &c = g_table_cache[device];
        if (t.bytes >= TABLE_CACHE_MIN && t.bytes <= (size_t)B2_TABLE_MAX + 4096 && t.bytes > c.bytes) std::swap(c, t);
    }
    if (t.p) (void)hipFree(t.p);
}

// The device of a platten made current, and the caller's again.
struct DeviceGuard {
    int cur = -1;
    bool other = false;
    explicit DeviceGuard(int device) {   // (-1: none yet)
        other = device >= 0 && hipGetDevice(&cur) == hipSuccess && cur != device && hipSetDevice(device) == hipSuccess;
    }
    ~DeviceGuard() {
        if (other) (void)hipSetDevice(cur);
    }
};

// Uploads gathered into one host buffer and copied with a single transfer into a device arena
// (one synchronous copy per arena instead of one per array: each costs ~15 us of fixed
// overhead).  The destinations are assigned when the arena is flushed and must not be read
// before; they are freed with the arena.
struct Stager {
    std::vector<unsigned char> host;
    std::vector<std::pair<void **, size_t>> dst;   // destination pointer, byte offset
    template <class T>
    void add(T **d, const T *src, size_t n) {
        *d = nullptr;
        if (n == 0) return;
        const size_t off = (host.size() + 255) & ~(size_t)255;
        host.resize(off + n * sizeof(T));
        memcpy(host.data() + off, src, n * sizeof(T));
        dst.emplace_back((void **)d, off);
    }
    int flush(Platten *P) {
        if (dst.empty()) return CSE_OK;
        void *a = nullptr;
        CSE_HIP_TRY(dev_malloc(&a, host.size()));
        P->arenas.emplace_back(a, host.size());
        CSE_HIP_TRY(hipMemcpy(a, host.data(), host.size(), hipMemcpyHostToDevice));
        for (auto &d : dst) *d.first = (unsigned char *)a + d.second;
        host.clear();
        dst.clear();
        return CSE_OK;
    }
};

template <class T>
int upload(T **dst, const T *src, size_t n) {
    if (n == 0) {
        *dst = nullptr;
        return CSE_OK;
    }
    CSE_HIP_TRY(dev_malloc((void **)dst, n * sizeof(T)));
    CSE_HIP_TRY(hipMemcpy(*dst, src, n * sizeof(T), hipMemcpyHostToDevice));
    return CSE_OK;
}

}  // namespace

hipError_t dev_malloc(void **p, size_t bytes) {
    hipError_t e = hipMalloc(p, bytes);
    int dev = 0;
    if (e == hipErrorOutOfMemory && hipGetDevice(&dev) == hipSuccess && drop_table(dev)) e = hipMalloc(p, bytes);
    if (e != hipSuccess) (void)hipGetLastError();   // reported here, not by the next launch
    return e;
}

int build_platten(const cse_design *design, int64_t n_boxes, const double *theta,
                  const double *radii, const int32_t *sims, int32_t flags, Platten *P) {
    Stager stage;   // read-only arrays: one transfer at the end of the tile setup
    if (!design || !theta || !radii || !sims || n_boxes < 1) {
        set_error("cse_platten_create: NULL argument or n_boxes < 1");
        return CSE_EINVAL;
    }
    if (design->reserved != 0) {
        set_error("cse_platten_create: design.reserved must be 0");
        return CSE_EINVAL;
    }
    const int kind = design->kind;
    int d = 0, p = 0;
    if (kind == CSE_ZTEST1) {
        d = 1;
        p = 1;
        P->family = FAM_NORMAL;
    } else if (kind == CSE_BINOM2_Z) {
        d = 2;
        p = 1;
        P->family = FAM_BINOM;
    } else if (kind == CSE_HIER4 || kind == CSE_PHASE23) {
        d = 4;
        p = 3;
        P->family = FAM_BINOM;
    } else if (kind == CSE_BASKET4) {
        d = 4;
        p = 4;
        P->family = FAM_BINOM;
        for (int a = 0; a < 4; ++a)
            if (!(fabs(design->theta0[a]) < 1e6)) {
                set_error("cse_platten_create: design.theta0 must be finite for the basket design");
                return CSE_EINVAL;
            }
    } else {
        set_error("cse_platten_create: unknown design kind");
        return CSE_EINVAL;
    }
    if (design->n_arms != d) {
        set_error("cse_platten_create: design.n_arms does not match the design kind");
        return CSE_EINVAL;
    }
    if (kind == CSE_PHASE23 && design->n_per_arm != P23_NMAX_ARM) {
        set_error("cse_platten_create: the Phase II/III design embeds n_per_arm = 350 patients per arm");
        return CSE_EUNSUPPORTED;
    }
    if (kind != CSE_PHASE23 && P->family == FAM_BINOM && design->n_per_arm != NP35) {
        set_error("cse_platten_create: binomial designs are built for n_per_arm = 35");
        return CSE_EUNSUPPORTED;
    }
    if (!(fabs(design->cut) < 1e300)) {
        set_error("cse_platten_create: design.cut must be finite");
        return CSE_EINVAL;
    }
    const bool keep_all = (flags & CSE_PLATTEN_KEEP_ALL) != 0;
    if (flags & ~CSE_PLATTEN_KEEP_ALL) {
        set_error("cse_platten_create: unknown flag");
        return CSE_EINVAL;
    }
    if (keep_all && p != 1) {
        set_error("cse_platten_create: KEEP_ALL is defined for single-hypothesis designs");
        return CSE_EINVAL;
    }
    for (int64_t i = 0; i < n_boxes; ++i) {
        if (sims[i] < 1 || sims[i] > (1 << 24)) {
            set_error("cse_platten_create: sims must lie in [1, 2^24]");
            return CSE_EINVAL;
        }
        for (int j = 0; j < d; ++j) {
            if (!(radii[i * d + j] > 0.0) || !(fabs(theta[i * d + j]) < 1e6)) {
                set_error("cse_platten_create: radii must be > 0 and theta finite");
                return CSE_EINVAL;
            }
        }
    }
    P->design = *design;
    P->d = d;
    P->p = p;
    P->n_per_arm = design->n_per_arm;
    P->n_boxes = n_boxes;
    CSE_HIP_TRY(hipGetDevice(&P->device));

    // Null hypotheses as half-spaces g . theta <= 0: z-test theta <= 0; multi-arm designs
    // (arm 0 control) theta_i - theta_0 <= 0.
    std::vector<HalfSpace> hyp(p);
    for (int j = 0; j < p; ++j) {
        HalfSpace hs{};
        if (kind == CSE_ZTEST1) {
            hs.g[0] = 1.0;
        } else {
            hs.g[j + 1] = 1.0;
            hs.g[0] = -1.0;
        }
        hs.h = 0.0;
        hyp[j] = hs;
    }

    // ---- the null partition of every box (Section 5) ----
    const int ncorner = 1 << d;
    std::vector<double> centre;   // simulation point of each tile
    if (kind == CSE_BASKET4) {
        // axis-aligned null boundaries theta_a = theta0[a]: each box is cut at the boundaries it
        // straddles and each piece with b != 0 (bit a: the piece lies in theta_a <= theta0[a])
        // is a box-shaped tile simulated at its own centre; a box's pieces by b ascending
        const double *t0 = design->theta0;
        for (int64_t i = 0; i < n_boxes; ++i) {
            const double *c = theta + i * d;
            const double *r = radii + i * d;
            double pc[4][2], pr[4][2];
            int pn[4], pin[4][2];
            for (int a = 0; a < 4; ++a) {
                const double lo = c[a] - r[a], hi = c[a] + r[a];
                if (lo < t0[a] && t0[a] < hi) {
                    pn[a] = 2;
                    pc[a][0] = 0.5 * (lo + t0[a]);
                    pr[a][0] = 0.5 * (t0[a] - lo);
                    pin[a][0] = 1;
                    pc[a][1] = 0.5 * (t0[a] + hi);
                    pr[a][1] = 0.5 * (hi - t0[a]);
                    pin[a][1] = 0;
                } else {
                    pn[a] = 1;
                    pc[a][0] = c[a];
                    pr[a][0] = r[a];
                    pin[a][0] = hi <= t0[a] ? 1 : 0;
                }
            }
            struct Piece {
                int b;
                double c[4], r[4];
            };
            std::vector<Piece> pieces;
            for (int i0 = 0; i0 < pn[0]; ++i0)
                for (int i1 = 0; i1 < pn[1]; ++i1)
                    for (int i2 = 0; i2 < pn[2]; ++i2)
                        for (int i3 = 0; i3 < pn[3]; ++i3) {
                            const int ix[4] = {i0, i1, i2, i3};
                            Piece q{};
                            for (int a = 0; a < 4; ++a) {
                                q.c[a] = pc[a][ix[a]];
                                q.r[a] = pr[a][ix[a]];
                                q.b |= pin[a][ix[a]] << a;
                            }
                            if (q.b) pieces.push_back(q);
                        }
            std::sort(pieces.begin(), pieces.end(), [](const Piece &x, const Piece &y) { return x.b < y.b; });
            for (auto &q : pieces) {
                P->tile_box.push_back(i);
                P->tile_cfg.push_back(q.b);
                P->tile_in_null.push_back(1);
                P->tile_is_box.push_back(1);
                for (int a = 0; a < d; ++a) {
                    P->tile_radii.push_back(q.r[a]);
                    centre.push_back(q.c[a]);
                }
                P->tile_nv.push_back(ncorner);
                P->vert_off.push_back((int32_t)(P->verts.size() / d));
                for (int m = 0; m < ncorner; ++m)
                    for (int a = 0; a < d; ++a) {
                        const double v = q.c[a] + (((m >> a) & 1) ? q.r[a] : -q.r[a]);
                        P->verts.push_back(v - q.c[a]);
                    }
            }
        }
    }
    // (kept over the boxes: most are whole, and allocating these for each took longer than clipping)
    std::vector<std::vector<double>> corners(ncorner, std::vector<double>(d)), V;
    std::vector<HalfSpace> cons, all;
    for (int64_t i = 0; i < (kind == CSE_BASKET4 ? 0 : n_boxes); ++i) {
        const double *c = theta + i * d;
        const double *r = radii + i * d;
        for (int m = 0; m < ncorner; ++m)
            for (int j = 0; j < d; ++j) corners[m][j] = c[j] + (((m >> j) & 1) ? r[j] : -r[j]);
        bool met = false;
        for (int b = 1; b < (1 << p); ++b) {
            cons.clear();
            for (int j = 0; j < p; ++j) {
                HalfSpace hs = hyp[j];
                if (!((b >> j) & 1)) {  // complement of H_j, closed: g . x >= h
                    for (int a = 0; a < d; ++a) hs.g[a] = -hs.g[a];
                    hs.h = -hs.h;
                }
                cons.push_back(hs);
            }
            bool empty = false, inside = true;
            for (auto &hs : cons) {
                double mn = 1e300, mx = -1e300;
                for (auto &x : corners) {
                    double s = -hs.h;
                    for (int a = 0; a < d; ++a) s += hs.g[a] * x[a];
                    mn = std::min(mn, s);
                    mx = std::max(mx, s);
                }
                if (mn >= 0.0) empty = true;   // the constraint holds at most on a face
                if (mx > 0.0) inside = false;
            }
            if (empty) continue;
            if (!inside) {
                all.clear();
                for (int a = 0; a < d; ++a) {
                    HalfSpace up{}, dn{};
                    up.g[a] = 1.0;
                    up.h = c[a] + r[a];
                    dn.g[a] = -1.0;
                    dn.h = -(c[a] - r[a]);
                    all.push_back(up);
                    all.push_back(dn);
                }
                for (auto &hs : cons) all.push_back(hs);
                V = enumerate_vertices(d, all);
                if ((int)V.size() < d + 1) continue;
                // full dimension <=> the vertex centroid satisfies every constraint strictly
                std::vector<double> cen(d, 0.0);
                for (auto &v : V)
                    for (int a = 0; a < d; ++a) cen[a] += v[a] / (double)V.size();
                bool interior = true;
                for (auto &hs : all) {
                    double s = 0.0;
                    for (int a = 0; a < d; ++a) s += hs.g[a] * cen[a];
                    if (!(s < hs.h - 1e-12)) interior = false;
                }
                if (!interior) continue;
            }
            met = true;
            const std::vector<std::vector<double>> &W = inside ? corners : V;
            P->tile_box.push_back(i);
            P->tile_cfg.push_back(b);
            P->tile_in_null.push_back(1);
            P->tile_is_box.push_back(inside ? 1 : 0);
            for (int a = 0; a < d; ++a) P->tile_radii.push_back(r[a]);
            P->tile_nv.push_back((int32_t)W.size());
            P->vert_off.push_back((int32_t)(P->verts.size() / d));
            for (auto &v : W)
                for (int a = 0; a < d; ++a) P->verts.push_back(v[a] - c[a]);
        }
        if (!met && keep_all) {
            P->tile_box.push_back(i);
            P->tile_cfg.push_back(1);
            P->tile_in_null.push_back(0);
            P->tile_is_box.push_back(1);
            for (int a = 0; a < d; ++a) P->tile_radii.push_back(r[a]);
            P->tile_nv.push_back(ncorner);
            P->vert_off.push_back((int32_t)(P->verts.size() / d));
            for (auto &v : corners)
                for (int a = 0; a < d; ++a) P->verts.push_back(v[a] - c[a]);
        }
    }
    P->n_tiles = (int64_t)P->tile_box.size();
    if (P->n_tiles == 0) {
        set_error("cse_platten_create: no box meets the null hypothesis space");
        return CSE_EINVAL;
    }
    P->vert_off.push_back((int32_t)(P->verts.size() / d));
    P->tile_theta.resize(P->n_tiles * d);
    P->tile_N.resize(P->n_tiles);
    std::vector<int64_t> key_off(P->n_tiles, -1), key_stride(P->n_tiles, 64);
    for (int64_t t = 0; t < P->n_tiles; ++t) {
        for (int a = 0; a < d; ++a)
            P->tile_theta[t * d + a] = kind == CSE_BASKET4 ? centre[t * d + a] : theta[P->tile_box[t] * d + a];
        P->tile_N[t] = sims[P->tile_box[t]];
        P->max_N = std::max(P->max_N, P->tile_N[t]);
        P->total_sims += P->tile_N[t];
        if (P->tile_nv[t] > 64) {
            set_error("cse_platten_create: a tile has more than 64 vertices");
            return CSE_EUNSUPPORTED;
        }
        P->max_nv = std::max(P->max_nv, P->tile_nv[t]);
    }
    if (P->family == FAM_BINOM) {
        P->tile_T.resize(P->n_tiles * d);
        for (int64_t t = 0; t < P->n_tiles * d; ++t) P->tile_T[t] = bern_threshold(P->tile_theta[t]);
    }

    // ---- tile batches ----
    std::vector<int64_t> &blk_sims = P->blk_sims;   // n_sims per block, for the work items
    if (kind == CSE_ZTEST1) {
        std::map<int32_t, std::vector<int64_t>> byN;
        for (int64_t t = 0; t < P->n_tiles; ++t) byN[P->tile_N[t]].push_back(t);
        std::vector<Blk1> blks;
        for (auto &kv : byN) {
            auto &ts = kv.second;
            for (size_t s = 0; s < ts.size(); s += B1T) {
                Blk1 B{};
                for (int j = 0; j < B1T; ++j) {
                    B.tile[j] = -1;
                    B.theta[j] = 0.0f;
                }
                for (size_t j = 0; j < B1T && s + j < ts.size(); ++j) {
                    B.tile[j] = (int32_t)ts[s + j];
                    B.theta[j] = (float)P->tile_theta[ts[s + j]];
                }
                B.n_sims = kv.first;
                blks.push_back(B);
            }
        }
        P->n_blocks = (int64_t)blks.size();
        for (auto &B : blks) {
            blk_sims.push_back(B.n_sims);
            B.key_base = P->n_keys;
            for (int j = 0; j < B1T; ++j)
                if (B.tile[j] >= 0) key_off[B.tile[j]] = B.key_base + (int64_t)j * B.n_sims;
            P->n_keys += (int64_t)B1T * B.n_sims;
        }
        if (int e = upload((Blk1 **)&P->d_blocks, blks.data(), blks.size())) return e;
    } else if (kind == CSE_HIER4 || kind == CSE_BASKET4) {
        // distinct values per arm -> coordinates; tiles ordered by simulation count, thresholds of arms
        // 0 and 1, 8 x 8 blocks of arms 2 and 3, 64 consecutive ones of a count to a set
        struct At {
            int32_t n, c[4], tile, cfg, at;
        };
        std::vector<At> order(P->n_tiles);
        for (int64_t t = 0; t < P->n_tiles; ++t) {
            order[t].n = P->tile_N[t];
            order[t].tile = (int32_t)t;
            order[t].cfg = P->tile_cfg[t];
        }
        std::vector<double> uv[4];   // distinct values, ascending; found in an open-addressed table first
        {
            int bits = 6;
            while (((size_t)1 << bits) < 2 * (size_t)P->n_tiles) ++bits;
            const size_t slots = (size_t)1 << bits;
            std::vector<int32_t> slot(slots), rank, by;
            for (int a = 0; a < 4; ++a) {
                std::fill(slot.begin(), slot.end(), -1);
                for (int64_t t = 0; t < P->n_tiles; ++t) {
                    const double v = P->tile_theta[t * 4 + a] + 0.0;   // one zero
                    size_t i = (size_t)value_slot(v, bits);
                    while (slot[i] >= 0 && uv[a][slot[i]] != v) i = (i + 1) & (slots - 1);
                    if (slot[i] < 0) {
                        slot[i] = (int32_t)uv[a].size();
                        uv[a].push_back(v);
                    }
                    order[t].c[a] = slot[i];
                }
                by.resize(uv[a].size());
                rank.resize(uv[a].size());
                std::iota(by.begin(), by.end(), 0);
                std::sort(by.begin(), by.end(), [&](int32_t x, int32_t y) { return uv[a][x] < uv[a][y]; });
                for (size_t i = 0; i < by.size(); ++i) rank[by[i]] = (int32_t)i;
                for (auto &o : order) o.c[a] = rank[o.c[a]];
                std::sort(uv[a].begin(), uv[a].end());
            }
        }
        std::sort(order.begin(), order.end(), [](const At &x, const At &y) {
            if (x.n != y.n) return x.n < y.n;
            if (x.c[0] != y.c[0]) return x.c[0] < y.c[0];
            if (x.c[1] != y.c[1]) return x.c[1] < y.c[1];
            if ((x.c[2] ^ y.c[2]) >> 3) return x.c[2] < y.c[2];
            if ((x.c[3] ^ y.c[3]) >> 3) return x.c[3] < y.c[3];
            if (x.c[2] != y.c[2]) return x.c[2] < y.c[2];
            return x.c[3] != y.c[3] ? x.c[3] < y.c[3] : x.tile < y.tile;
        });
        // threshold groups: per simulation count and arm, the coordinates present, 8 to a group
        std::vector<Grp4> grps;
        std::vector<std::pair<int32_t, int32_t>> at_arm[4];   // per tile in order and arm: (group, threshold)
        for (int a = 0; a < 4; ++a) at_arm[a].resize(order.size());
        for (size_t i = 0; i < order.size();) {
            size_t j = i;
            while (j < order.size() && order[j].n == order[i].n) ++j;
            for (int a = 0; a < 4; ++a) {
                std::vector<std::pair<int32_t, int32_t>> of(uv[a].size(), {-1, -1});
                for (size_t q = i; q < j; ++q) of[order[q].c[a]].first = 0;   // present
                int n = 0;
                for (size_t c = 0; c < of.size(); ++c) {
                    if (of[c].first < 0) continue;
                    if (n++ % 8 == 0) {
                        Grp4 g{};
                        g.arm = a;
                        g.n_sims = order[i].n;
                        grps.push_back(g);
                    }
                    Grp4 &g = grps.back();
                    of[c] = std::make_pair((int32_t)grps.size() - 1, g.n_thr);
                    g.T[g.n_thr++] = bern_threshold(uv[a][c]);
                }
                for (size_t q = i; q < j; ++q) at_arm[a][q] = of[order[q].c[a]];
            }
            i = j;
        }
        // count table: all simulations at once where that fits B2_TABLE_MAX, else windows (at least the
        // pilot's simulations, a multiple of every slice)
        auto granules = [](int32_t n) { return ((int64_t)n + GRAN2 - 1) / GRAN2; };
        auto units = [&](int64_t win) {
            int64_t n = 0;
            for (auto &g : grps) n += std::min(win, granules(g.n_sims)) * (g.arm < 2 ? g.n_thr : 8 + g.n_thr);
            return n;
        };
        P->b4_win = H4_SLICE_MAX;
        while (P->b4_win < granules(P->max_N)) P->b4_win *= 2;
        while (P->b4_win > H4_SLICE_MAX && units(P->b4_win) * 16 > B2_TABLE_MAX) P->b4_win /= 2;
        // boxes without common thresholds take 24 KB each at that window: beyond H4_TABLE_MAX, or an eighth of the
        // free memory, shorter ones (then without candidates, whose pilot and slices lie in one window)
        if (units(P->b4_win) * 16 > B2_TABLE_MAX) {
            size_t free_bytes = 0, all_bytes = 0;
            CSE_HIP_TRY(hipMemGetInfo(&free_bytes, &all_bytes));
            const int64_t most = std::max<int64_t>(B2_TABLE_MAX, std::min<int64_t>(H4_TABLE_MAX, (int64_t)(free_bytes / 8)));
            while (P->b4_win > 4 && units(P->b4_win) * 16 > most) P->b4_win /= 2;
        }
        for (auto &g : grps) {
            g.stride = std::min(P->b4_win, granules(g.n_sims));
            g.row = P->b4_units;
            P->b4_units += g.stride * (g.arm < 2 ? g.n_thr : 8 + g.n_thr);
        }
        if (P->b4_units >= ((int64_t)1 << 32)) {
            set_error("cse_platten_create: too many distinct thresholds for the count table");
            return CSE_ENOMEM;
        }
        P->n_grp4 = (int32_t)grps.size();
        std::vector<int32_t> at(P->n_tiles);
        std::vector<uint32_t> rows;
        // place of row i of group g (its codes: 8 + i) in the list that begins at row_at, appended if new
        std::vector<int64_t> row_place(16 * grps.size(), -1);
        auto row_of = [&](int64_t row_at, int32_t g, int32_t i) {
            int64_t &q = row_place[16 * (size_t)g + i];
            if (q < row_at) {
                q = (int64_t)rows.size();
                rows.push_back((uint32_t)(grps[g].row + i * grps[g].stride));
            }
            return (uint16_t)(q - row_at);
        };
        for (size_t i = 0; i < order.size();) {
            H4Set S{};
            S.row_at = (int64_t)rows.size();
            S.n_sims = order[i].n;
            S.key_base = P->n_keys;
            while (S.n_lanes < WAVE && i < order.size() && order[i].n == S.n_sims &&
                   (int64_t)rows.size() - S.row_at + H4_ROWS <= H4_SET_ROWS) {
                const At &o = order[i];
                const int l = S.n_lanes++;
                S.tile[l] = o.tile;
                S.cfg[l] = (uint32_t)P->tile_cfg[o.tile];
                for (int a = 0; a < 4; ++a) {
                    const auto pl = at_arm[a][i];
                    S.row[a][l] = row_of(S.row_at, pl.first, pl.second);
                    if (a >= 2) S.row[a + 2][l] = row_of(S.row_at, pl.first, 8 + pl.second);
                }
                at[o.tile] = (int32_t)(P->h4set.size() * WAVE) + l;
                ++i;
            }
            for (int l = S.n_lanes; l < WAVE; ++l) {
                S.tile[l] = -1;
                S.cfg[l] = S.cfg[0];
                for (int a = 0; a < H4_ROWS; ++a) S.row[a][l] = S.row[a][0];
            }
            S.n_rows = (int32_t)((int64_t)rows.size() - S.row_at);
            P->h4_max_rows = std::max(P->h4_max_rows, S.n_rows);
            for (int l = 0; l < S.n_lanes; ++l) {
                key_off[S.tile[l]] = S.key_base + (int64_t)l * WAVE;
                key_stride[S.tile[l]] = (int64_t)S.n_lanes * WAVE;
            }
            P->n_keys += ((int64_t)S.n_sims + 63) / 64 * 64 * S.n_lanes;
            blk_sims.push_back(S.n_sims);
            P->h4set.push_back(S);
        }
        P->n_blocks = P->n_h4set = (int64_t)P->h4set.size();
        // runs along arm 3: the tiles of one count, thresholds of arms 0, 1 and 2 and configuration, in
        // pieces of up to H4_RUN
        {
            std::vector<At> by = order;   // at: place in `order`
            for (size_t i = 0; i < by.size(); ++i) by[i].at = (int32_t)i;
            for (size_t i = 0, j; i < by.size(); i = j) {   // a count and pair of thresholds of arms 0 and 1 at a time
                for (j = i + 1; j < by.size() && std::tie(by[i].n, by[i].c[0], by[i].c[1]) == std::tie(by[j].n, by[j].c[0], by[j].c[1]);)
                    ++j;
                std::sort(by.begin() + i, by.begin() + j, [](const At &x, const At &y) {
                    if (x.cfg != y.cfg) return x.cfg < y.cfg;
                    if (x.c[2] != y.c[2]) return x.c[2] < y.c[2];
                    return x.c[3] != y.c[3] ? x.c[3] < y.c[3] : x.tile < y.tile;
                });
            }
            auto end_of = [&](size_t i) {
                const At &x = by[i];
                size_t j = i + 1;
                while (j < by.size() && std::tie(x.n, x.c[0], x.c[1], x.cfg, x.c[2]) ==
                                            std::tie(by[j].n, by[j].c[0], by[j].c[1], by[j].cfg, by[j].c[2]))
                    ++j;
                return j;
            };
            auto close = [&](int lanes) {
                H4Run &S = P->h4run.back();
                for (int l = lanes; l < WAVE; ++l) {
                    for (int r = 0; r < H4_RUN; ++r) S.tile[r][l] = -1;
                    for (int a = 0; a < 3 + H4_RUN; ++a) S.row[a][l] = S.row[a][0];
                    S.cfg[l] = S.cfg[0];
                }
                S.n_rows = (int32_t)((int64_t)rows.size() - S.row_at);
                P->h4_run_rows = std::max(P->h4_run_rows, S.n_rows);
            };
            int lanes = 0;
            // pieces of one length together: a set takes as long as its longest
            struct Piece {
                int32_t n, len;
                size_t b;
            };
            std::vector<Piece> pieces;
            for (size_t i = 0, j; i < by.size(); i = j) {
                j = end_of(i);
                const int64_t len = (int64_t)(j - i), parts = (len + H4_RUN - 1) / H4_RUN;
                for (int64_t q = 0; q < parts; ++q) {
                    const size_t b = i + (size_t)(len * q / parts), e = i + (size_t)(len * (q + 1) / parts);
                    pieces.push_back({by[b].n, (int32_t)(e - b), b});
                }
            }
            std::stable_sort(pieces.begin(), pieces.end(), [](const Piece &x, const Piece &y) {
                return std::make_tuple(x.n, -x.len) < std::make_tuple(y.n, -y.len);
            });
            for (const Piece &pc : pieces) {
                if (P->h4run.empty() || lanes == WAVE || P->h4run.back().n_sims != pc.n ||
                    (int64_t)rows.size() - P->h4run.back().row_at > H4_ROWS * WAVE - (3 + H4_RUN)) {
                    if (!P->h4run.empty()) close(lanes);
                    P->h4run.emplace_back();
                    P->h4run.back().n_sims = pc.n;
                    P->h4run.back().row_at = (int64_t)rows.size();
                    lanes = 0;
                }
                H4Run &S = P->h4run.back();
                S.cfg[lanes] = (uint32_t)by[pc.b].cfg;
                for (int a = 0; a < 3; ++a) S.row[a][lanes] = row_of(S.row_at, at_arm[a][by[pc.b].at].first, at_arm[a][by[pc.b].at].second);
                for (int r = 0; r < H4_RUN; ++r) {
                    const At &o = by[r < pc.len ? pc.b + r : pc.b];
                    S.tile[r][lanes] = r < pc.len ? o.tile : -1;
                    S.row[3 + r][lanes] = row_of(S.row_at, at_arm[3][o.at].first, at_arm[3][o.at].second);
                }
                S.n_run = std::max(S.n_run, pc.len);
                ++lanes;
            }
            if (lanes) close(lanes);
            stage.add(&P->d_h4run, P->h4run.data(), P->h4run.size());
        }
        stage.add(&P->d_grp4, grps.data(), grps.size());
        stage.add(&P->d_h4at, at.data(), at.size());
        stage.add(&P->d_h4rows, rows.data(), rows.size());
        // chunks of four granules are read whole: up to three units past a row's end
        {
            TableBuf t;
            CSE_HIP_TRY(take_table(P->device, (size_t)(P->b4_units + 4) * 16, &t));
            P->d_b4tab = (uint4 *)t.p;
            P->table_bytes = t.bytes;
        }
        CSE_HIP_TRY(dev_malloc((void **)&P->d_h4u, (size_t)P->n_tiles * sizeof(float)));
        CSE_HIP_TRY(dev_malloc((void **)&P->d_h4eq, (size_t)P->n_tiles * sizeof(uint32_t)));

        // posterior table of the design (once per platten)
        const std::vector<HierNode> nodes = hier_nodes();
        if (int e = upload(&P->d_hnodes, nodes.data(), nodes.size())) return e;
        const int64_t m = P->n_per_arm + 1;
        P->h4_outcomes = m * m * m * m;
        CSE_HIP_TRY(dev_malloc((void **)&P->d_h4tbl, (size_t)P->h4_outcomes * sizeof(float4)));
        const auto t0 = std::chrono::steady_clock::now();
        if (kind == CSE_BASKET4)
            CSE_HIP_TRY(launch_basket_table(P->n_per_arm, design->theta0, P->d_h4tbl, P->d_hnodes, nullptr));
        else
            CSE_HIP_TRY(launch_hier4_table(P->n_per_arm, P->d_h4tbl, P->d_hnodes, nullptr));
        const int n_cfg = kind == CSE_BASKET4 ? 15 : 7;
        CSE_HIP_TRY(dev_malloc((void **)&P->d_h4bits, (size_t)n_cfg * H4_BITS * sizeof(uint64_t)));
        CSE_HIP_TRY(launch_h4_bits(P->d_h4tbl, (float)design->cut, n_cfg, P->d_h4bits, nullptr));
        CSE_HIP_TRY(dev_malloc((void **)&P->d_h4plane, (size_t)n_cfg * H4_PLANE * sizeof(float)));
        CSE_HIP_TRY(launch_h4_planes(P->d_h4tbl, n_cfg, P->d_h4plane, nullptr));
        CSE_HIP_TRY(hipDeviceSynchronize());
        P->table_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
        if (int e = upload(&P->d_tileT, P->tile_T.data(), P->tile_T.size())) return e;   // regenerated keys
        CSE_HIP_TRY(dev_malloc((void **)&P->d_h4fb, sizeof(uint32_t)));
        CSE_HIP_TRY(hipMemset(P->d_h4fb, 0, sizeof(uint32_t)));
    } else if (kind == CSE_PHASE23) {
        // one trial per lane: keys contiguous per tile, work items of p23_chunk simulations
        for (int64_t t = 0; t < P->n_tiles; ++t) {
            key_off[t] = P->n_keys;
            key_stride[t] = 64;   // contiguous: chunk c of 64 keys starts at 64 c
            P->n_keys += P->tile_N[t];
        }
        if (int e = plan_queue_items(P, P->p23_chunk, -1)) return e;
        {
            // the records of a chunk's trials, and a table of at least as many slots as trials (2^27 at most),
            // in one allocation: at most an eighth of the free memory (fewer trials a chunk, fewer slots), or
            // half as much again and again where that cannot be had
            size_t free_bytes = 0, all_bytes = 0;
            CSE_HIP_TRY(hipMemGetInfo(&free_bytes, &all_bytes));
            P->p23_cap = std::max<int64_t>(P23_CAP_MIN, std::min<int64_t>(P->total_sims, P23_CAP_MAX));
            uint64_t slots = P23_SLOTS_MIN;
            while (slots < (1u << 27) && slots < (uint64_t)P->total_sims) slots *= 2;
            P23Memo &M = P->p23memo;
            size_t off, o_state, o_value, o_own, o_l0, o_l1, o_t0, o_t1, o_range, o_ctr;
            for (;;) {
                const size_t cap = (size_t)P->p23_cap;
                off = 0;
                auto take = [&](size_t bytes) {
                    const size_t at = off;
                    off += (bytes + 255) & ~(size_t)255;
                    return at;
                };
                o_state = take(slots * 8), o_value = take((slots + cap) * 4), o_own = take(cap * 8), o_l0 = take(cap * 4),
                o_l1 = take(cap * 4), o_t0 = take(cap * 32), o_t1 = take(cap * 32), o_range = take(P23_BLOCKS * sizeof(uint2)),
                o_ctr = take(P23_COUNTERS * P23_CTR * sizeof(uint32_t));
                const bool least = P->p23_cap == P23_CAP_MIN && slots == P23_SLOTS_MIN;
                if (off <= free_bytes / 8 || least) {
                    const hipError_t e = dev_malloc(&P->d_p23mem, off);
                    if (e == hipSuccess) break;
                    if (least) CSE_HIP_TRY(e);
                }
                P->p23_cap = std::max<int64_t>(P23_CAP_MIN, P->p23_cap / 2);
                slots = std::max<uint64_t>(P23_SLOTS_MIN, slots / 2);
            }
            M.mask = (uint32_t)(slots - 1);
            unsigned char *m = (unsigned char *)P->d_p23mem;
            M.state = (unsigned long long *)(m + o_state);
            M.value = (uint32_t *)(m + o_value);
            M.own = (uint64_t *)(m + o_own);
            M.list[0] = (uint32_t *)(m + o_l0);
            M.list[1] = (uint32_t *)(m + o_l1);
            M.trial[0] = (uint4 *)(m + o_t0);
            M.trial[1] = (uint4 *)(m + o_t1);
            M.range = (uint2 *)(m + o_range);
            M.ctr = (uint32_t *)(m + o_ctr);
        }
        if (int e = upload(&P->d_tileT, P->tile_T.data(), P->tile_T.size())) return e;
        if (int e = upload(&P->d_cfg, P->tile_cfg.data(), P->tile_cfg.size())) return e;
        CSE_HIP_TRY(dev_malloc((void **)&P->d_queue, sizeof(uint32_t)));
        CSE_HIP_TRY(dev_malloc((void **)&P->d_p23stats, 4 * sizeof(unsigned long long)));
        // count table rows: each arm's distinct thresholds, for the simulations of its longest tile
        {
            std::vector<P23Row> rows;
            std::vector<uint2> tile_row(4 * (size_t)P->n_tiles);
            uint64_t at = 0;
            for (int a = 0; a < 4; ++a) {
                std::vector<std::pair<uint32_t, int32_t>> v(P->n_tiles);   // (threshold, simulations)
                for (int64_t t = 0; t < P->n_tiles; ++t) v[t] = {P->tile_T[4 * t + a], P->tile_N[t]};
                std::sort(v.begin(), v.end());
                const size_t first = rows.size();
                for (size_t i = 0; i < v.size(); ++i) {
                    if (i + 1 < v.size() && v[i + 1].first == v[i].first) continue;   // the largest count is last
                    P23Row r{};
                    r.T = v[i].first;
                    r.arm = a;
                    r.at = (uint32_t)std::min<uint64_t>(at, 0xFFFFFFFFull);
                    r.stride = (uint32_t)((v[i].second + 63) / 64);
                    P->p23_chunks = std::max<int64_t>(P->p23_chunks, r.stride);
                    at += (uint64_t)r.stride * P23_SIZES;
                    rows.push_back(r);
                }
                P->p23_arm_row[a + 1] = (int32_t)rows.size();
                for (int64_t t = 0; t < P->n_tiles; ++t) {
                    const auto it = std::lower_bound(rows.begin() + first, rows.end(), P->tile_T[4 * t + a],
                                                     [](const P23Row &r, uint32_t T) { return r.T < T; });
                    tile_row[4 * t + a] = make_uint2(it->at, it->stride);
                }
            }
            size_t free_bytes = 0, all_bytes = 0;
            CSE_HIP_TRY(hipMemGetInfo(&free_bytes, &all_bytes));
            const size_t bytes = at * 64 * sizeof(uint16_t);
            // (an eighth of the free memory at most; without it trials draw their own words)
            if (at * 64 * sizeof(uint16_t) <= (uint64_t)P23_TABLE_MAX && bytes <= free_bytes / 8 &&
                dev_malloc((void **)&P->d_p23counts, bytes) == hipSuccess) {
                P->n_p23row = (int32_t)rows.size();
                if (int e = upload(&P->d_p23row, rows.data(), rows.size())) return e;
                if (int e = upload(&P->d_p23tilerow, tile_row.data(), tile_row.size())) return e;
            }
        }
        P23Args &A = P->p23;
        A.counts = P->d_p23counts;
        A.tile_row = P->d_p23tilerow;
        A.counter = P->d_queue;
        A.tileT = P->d_tileT;
        A.cfg = P->d_cfg;
        A.cut = (float)design->cut;
        double gh[32];
        gauss_hermite16(gh, gh + 16);
        if (int e = upload(&P->d_gh, gh, 32)) return e;
        A.gh = P->d_gh;
        const std::vector<HierNode> nodes = hier_nodes();
        if (int e = upload(&P->d_hnodes, nodes.data(), nodes.size())) return e;
        A.nodes = P->d_hnodes;
        A.sqrt_pi = sqrt(M_PI);
        A.z95 = normal_q95();
        // decisions of the first look (50 patients per arm) for every outcome, once per platten
        CSE_HIP_TRY(dev_malloc((void **)&P->d_p23look1, (size_t)51 * 51 * 51 * 51));
        A.look1 = P->d_p23look1;
        {
            const auto t0 = std::chrono::steady_clock::now();
            CSE_HIP_TRY(launch_p23_look1(*P, nullptr));
            CSE_HIP_TRY(hipDeviceSynchronize());
            P->table_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
        }
    } else {
        // distinct arm values -> integer coordinates; 8 x 8 coordinate blocks per N class
        std::vector<double> u0, u1;
        for (int64_t t = 0; t < P->n_tiles; ++t) {
            u0.push_back(P->tile_theta[t * 2 + 0]);
            u1.push_back(P->tile_theta[t * 2 + 1]);
        }
        std::sort(u0.begin(), u0.end());
        u0.erase(std::unique(u0.begin(), u0.end()), u0.end());
        std::sort(u1.begin(), u1.end());
        u1.erase(std::unique(u1.begin(), u1.end()), u1.end());
        std::map<std::tuple<int32_t, int64_t, int64_t>, std::vector<Blk2>> blkmap;
        for (int64_t t = 0; t < P->n_tiles; ++t) {
            int64_t c0 = std::lower_bound(u0.begin(), u0.end(), P->tile_theta[t * 2]) - u0.begin();
            int64_t c1 = std::lower_bound(u1.begin(), u1.end(), P->tile_theta[t * 2 + 1]) - u1.begin();
            auto key = std::make_tuple(P->tile_N[t], c0 / B2U, c1 / B2V);
            auto &vec = blkmap[key];
            int slot = (int)(c0 % B2U) * B2V + (int)(c1 % B2V);
            Blk2 *B = nullptr;
            for (auto &b : vec)
                if (b.tile[slot] < 0) {
                    B = &b;
                    break;
                }
            if (!B) {
                Blk2 nb{};
                for (int j = 0; j < B2U * B2V; ++j) nb.tile[j] = -1;
                int64_t b0 = (c0 / B2U) * B2U, b1 = (c1 / B2V) * B2V;
                // past the last distinct value: repeat it (no tile there; the thresholds stay ascending)
                for (int u = 0; u < B2U; ++u)
                    nb.T0[u] = bern_threshold(u0[std::min<size_t>(b0 + u, u0.size() - 1)]);
                for (int v = 0; v < B2V; ++v)
                    nb.T1[v] = bern_threshold(u1[std::min<size_t>(b1 + v, u1.size() - 1)]);
                nb.n_sims = P->tile_N[t];
                vec.push_back(nb);
                B = &vec.back();
            }
            B->tile[slot] = (int32_t)t;
        }
        std::vector<Blk2> blks;
        for (auto &kv : blkmap)
            for (auto &b : kv.second) {
                blks.push_back(b);
                P->blk_row.push_back(std::get<1>(kv.first));
                P->blk_col.push_back(std::get<2>(kv.first));
            }
        P->n_blocks = (int64_t)blks.size();
        // threshold groups: one per (simulation count, row) and (simulation count, column) of blocks
        std::vector<Grp2> grps;
        {
            std::map<std::pair<int32_t, int64_t>, int32_t> rows, cols;
            for (size_t b = 0; b < blks.size(); ++b)
                for (int arm = 0; arm < 2; ++arm) {
                    auto &m = arm ? cols : rows;
                    const int64_t at = arm ? P->blk_col[b] : P->blk_row[b];
                    auto ins = m.emplace(std::make_pair(blks[b].n_sims, at), (int32_t)grps.size());
                    if (ins.second) {
                        Grp2 g{};
                        memcpy(g.T, arm ? blks[b].T1 : blks[b].T0, sizeof g.T);
                        g.arm = arm;
                        g.n_sims = blks[b].n_sims;
                        grps.push_back(g);
                    }
                    (arm ? P->blk_cg : P->blk_rg).push_back(ins.first->second);
                }
        }
        // count table: all simulations of every group at once where that fits B2_TABLE_MAX, else
        // equal windows of simulations (at least one chunk of 64)
        auto granules = [](const Grp2 &g) { return ((int64_t)g.n_sims + GRAN2 - 1) / GRAN2; };
        auto units = [&](int64_t win) {
            int64_t n = 0;
            for (auto &g : grps) n += std::min(win, granules(g)) * (g.arm ? 1 : 2);
            return n;
        };
        P->b2_win = (((int64_t)P->max_N + GRAN2 - 1) / GRAN2 + 3) / 4 * 4;
        while (P->b2_win > 4 && units(P->b2_win) * UNIT2 > B2_TABLE_MAX) P->b2_win = (P->b2_win / 2 + 3) / 4 * 4;
        P->b2_units = units(P->b2_win);
        {
            int64_t u = 0, r = 0;
            for (auto &g : grps) {
                g.unit = u;
                g.rec = r;
                u += std::min(P->b2_win, granules(g)) * (g.arm ? 1 : 2);
                r += ((int64_t)g.n_sims + 63) / 64 * 64;
            }
            P->b2_recs = r;
        }
        P->n_grp2 = (int32_t)grps.size();
        for (size_t b = 0; b < blks.size(); ++b) {
            Blk2 &B = blks[b];
            blk_sims.push_back(B.n_sims);
            B.rec0 = grps[P->blk_rg[b]].rec;
            B.rec1 = grps[P->blk_cg[b]].rec;
            for (int j = 0; j < B2U * B2V; ++j)
                if (B.tile[j] >= 0) key_off[B.tile[j]] = (int64_t)b;   // placed
            // key slots: 16 bytes per (simulation, block); the groups' entries (8 bytes per
            // simulation and group, at most two groups per block) never take more
            P->n_keys += ((int64_t)B.n_sims + 63) / 64 * 64;
        }
        stage.add(&P->d_grp2, grps.data(), grps.size());
        stage.add((Blk2 **)&P->d_blocks, blks.data(), blks.size());

        // design tables of the pooled z test
        const int n = P->n_per_arm, n1 = n + 1;
        P->n_outcomes = n1 * n1;
        std::vector<int32_t> cut(n1);
        std::vector<double> S(n1 * n1);
        for (int y0 = 0; y0 <= n; ++y0) {
            cut[y0] = n1;   // no y1 rejects
            for (int y1 = 0; y1 <= n; ++y1) {
                double z = pooled_z(y0, y1, n);
                S[y0 * n1 + y1] = -z;
                if (z > design->cut && cut[y0] == n1) cut[y0] = y1;
            }
            // the kernels use {y1 >= c(y0)}: this needs z increasing in y1 for fixed y0
            for (int y1 = 0; y1 <= n; ++y1)
                if ((pooled_z(y0, y1, n) > design->cut) != (y1 >= cut[y0])) {
                    set_error("internal: pooled z rejection region is not monotone in y1");
                    return CSE_EUNSUPPORTED;
                }
        }
        // the calibration selection classifies outcomes by cut points on y1 per y0: S must not
        // increase with y1 for fixed y0 (so {y1 : S < s} is a suffix for every s)
        for (int y0 = 0; y0 <= n; ++y0)
            for (int y1 = 0; y1 < n; ++y1)
                if (S[y0 * n1 + y1 + 1] > S[y0 * n1 + y1]) {
                    set_error("internal: the 2-arm statistic is not monotone in y1");
                    return CSE_EUNSUPPORTED;
                }
        // and, so that cut points ascend with y0, it must not decrease with y0 for fixed y1
        for (int y0 = 0; y0 < n; ++y0)
            for (int y1 = 0; y1 <= n; ++y1)
                if (S[(y0 + 1) * n1 + y1] < S[y0 * n1 + y1]) {
                    set_error("internal: the 2-arm statistic is not monotone in y0");
                    return CSE_EUNSUPPORTED;
                }
        std::vector<int32_t> order(n1 * n1), group(n1 * n1);
        std::iota(order.begin(), order.end(), 0);
        std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return S[a] < S[b]; });
        std::vector<int32_t> pos(n1 * n1);
        for (int j = 0; j < n1 * n1; ++j) {
            group[j] = (j > 0 && S[order[j]] == S[order[j - 1]]) ? group[j - 1] : j;
            pos[order[j]] = j;
        }
        stage.add(&P->d_cut_tbl, cut.data(), cut.size());
        stage.add(&P->d_S_tbl, S.data(), S.size());
        stage.add(&P->d_S_order, order.data(), order.size());
        stage.add(&P->d_S_group, group.data(), group.size());
        stage.add(&P->d_S_pos, pos.data(), pos.size());
        // tie groups of S in ascending order: first position of each (and n1 * n1 after the
        // last), and per group g the cut vector cut_g(y0) = #{y1 : S(y0, y1) >= S_g}, so that
        // S < S_g iff y1 >= cut_g(y0); group n_groups has cut 0 (every outcome below it)
        {
            std::vector<int32_t> gstart;
            for (int j = 0; j < n1 * n1; ++j)
                if (group[j] == j) gstart.push_back(j);
            const int ng = (int)gstart.size();
            std::vector<uint8_t> gcut((size_t)(ng + 1) * n1, 0);
            // S does not increase with y1, so a row's cut falls as S_g rises: one walk per row (counting each
            // from 0 took 0.14 of the 0.85 ms that creating a platten of 2,080 tiles took)
            std::vector<double> Sg(ng);
            for (int g = 0; g < ng; ++g) Sg[g] = S[order[gstart[g]]];
            for (int y0 = 0; y0 <= n; ++y0) {
                int c = n1;
                for (int g = 0; g < ng; ++g) {
                    while (c > 0 && !(S[y0 * n1 + c - 1] >= Sg[g])) --c;
                    gcut[(size_t)g * n1 + y0] = (uint8_t)c;
                }
            }
            gstart.push_back(n1 * n1);
            P->n_groups = ng;
            stage.add(&P->d_gstart, gstart.data(), gstart.size());
            stage.add(&P->d_gcut, gcut.data(), gcut.size());
        }
    }

    for (int64_t t = 0; t < P->n_tiles; ++t)
        if (key_off[t] < 0) {
            set_error("internal: a tile was not placed in any batch");
            return CSE_EINVAL;
        }

    // ---- work items (launch shapes; cse_autotune may rebuild them) ----
    for (int64_t b = 0; b < P->n_blocks; ++b) P->block_sims += blk_sims[b];
    if (kind == CSE_ZTEST1)
        if (int e = plan_work_items(P, P->tune_waves)) return e;
    // default workgroup counts, measured (the 2-arm design's: plan_group_items, from its rectangles)
    if (kind == CSE_BINOM2_Z) P->tune_wgs = 0;
    if (kind == CSE_BINOM2_Z)
        if (int e = plan_group_items(P, P->tune_wgs)) return e;
    if (kind == CSE_HIER4 || kind == CSE_BASKET4)
        if (int e = plan_h4_items(P, 0)) return e;
    if (kind != CSE_ZTEST1) P->n_items = P->n_gitems;

    stage.add(&P->d_theta, P->tile_theta.data(), P->tile_theta.size());
    stage.add(&P->d_N, P->tile_N.data(), P->tile_N.size());
    stage.add(&P->d_vert_off, P->vert_off.data(), P->vert_off.size());
    stage.add(&P->d_verts, P->verts.data(), P->verts.size());
    stage.add(&P->d_radii, P->tile_radii.data(), P->tile_radii.size());
    stage.add(&P->d_is_box, P->tile_is_box.data(), P->tile_is_box.size());
    // order of the tiles in the bound's search: whole boxes, then pieces by their vertices (a wave takes as
    // long as its longest tile, and both forms where it holds both); as they are where all are of one kind
    if (std::find(P->tile_is_box.begin(), P->tile_is_box.end(), 1) != P->tile_is_box.end() &&
        std::find(P->tile_is_box.begin(), P->tile_is_box.end(), 0) != P->tile_is_box.end()) {
        auto cls = [&](int64_t t) { return P->tile_is_box[t] ? 0 : 1 + std::min<int32_t>(P->vert_off[t + 1] - P->vert_off[t], 255); };
        std::vector<int64_t> at(258, 0);
        for (int64_t t = 0; t < P->n_tiles; ++t) ++at[cls(t) + 1];
        for (size_t i = 1; i < at.size(); ++i) at[i] += at[i - 1];
        P->border.resize(P->n_tiles);
        for (int64_t t = 0; t < P->n_tiles; ++t) P->border[at[cls(t)]++] = (int32_t)t;
        stage.add(&P->d_border, P->border.data(), P->border.size());
    }
    stage.add(&P->d_in_null, P->tile_in_null.data(), P->tile_in_null.size());
    if (kind != CSE_BINOM2_Z) {
        stage.add(&P->d_key_off, key_off.data(), key_off.size());
        stage.add(&P->d_key_stride, key_stride.data(), key_stride.size());
    }
    // N classes for the Clopper-Pearson table
    {
        std::vector<int32_t> cls(P->tile_N.begin(), P->tile_N.end());
        std::sort(cls.begin(), cls.end());
        cls.erase(std::unique(cls.begin(), cls.end()), cls.end());
        std::vector<int64_t> off(cls.size()), base(P->n_tiles);
        int64_t e = 0;
        for (size_t c = 0; c < cls.size(); ++c) {
            off[c] = e;
            e += (int64_t)cls[c] + 1;
            P->max_cls_N = std::max(P->max_cls_N, cls[c]);
        }
        for (int64_t t = 0; t < P->n_tiles; ++t)
            base[t] = off[std::lower_bound(cls.begin(), cls.end(), P->tile_N[t]) - cls.begin()];
        P->n_cls = (int32_t)cls.size();
        P->n_cp = e;
        stage.add(&P->d_cls_N, cls.data(), cls.size());
        stage.add(&P->d_cls_off, off.data(), off.size());
        stage.add(&P->d_cp_base, base.data(), base.size());
        if (int r = stage.flush(P)) return r;
        if (kind == CSE_PHASE23) P->p23.key_off = P->d_key_off;
        CSE_HIP_TRY(dev_malloc((void **)&P->d_cp_mark, (size_t)e * sizeof(uint32_t)));
        CSE_HIP_TRY(dev_malloc((void **)&P->d_cp_tbl, (size_t)e * sizeof(double)));
    }
    const size_t nt = (size_t)P->n_tiles;
    CSE_HIP_TRY(dev_malloc((void **)&P->d_Rw, nt * sizeof(uint32_t)));
    // score sums: sum of T per arm; the Phase II/III design also sums the observed n per arm
    const size_t tw = (kind == CSE_PHASE23) ? 2 * (size_t)d : (size_t)d;
    CSE_HIP_TRY(dev_malloc((void **)&P->d_Tw, nt * tw * sizeof(unsigned long long)));
    CSE_HIP_TRY(dev_malloc((void **)&P->d_Zw, nt * sizeof(unsigned long long)));
    CSE_HIP_TRY(dev_malloc((void **)&P->d_apw, nt * sizeof(double)));
    CSE_HIP_TRY(dev_malloc((void **)&P->d_kw, nt * sizeof(int32_t)));
    CSE_HIP_TRY(dev_malloc((void **)&P->d_lamw, nt * sizeof(double)));
    CSE_HIP_TRY(dev_malloc((void **)&P->d_lamg, sizeof(double)));
    CSE_HIP_TRY(dev_malloc((void **)&P->d_minpart, 2 * MIN_PARTS * sizeof(double)));
    if (kind == CSE_BINOM2_Z) {
        TableBuf t;
        CSE_HIP_TRY(take_table(P->device, (size_t)P->b2_units * UNIT2, &t));
        P->d_b2tab = (uint4 *)t.p;
        P->table_bytes = t.bytes;
        CSE_HIP_TRY(dev_malloc((void **)&P->d_b2cut, (size_t)P->n_blocks * B2U * (NP35 + 1) * sizeof(uint4)));
        CSE_HIP_TRY(dev_malloc((void **)&P->d_b2br, nt * sizeof(int2)));
        CSE_HIP_TRY(dev_malloc((void **)&P->d_b2fb, sizeof(uint32_t)));
    }
    CSE_HIP_TRY(take_side_stream(P->device, &P->side));
    for (hipEvent_t *e : {&P->ev_sim, &P->ev_val, &P->ev_fork, &P->ev_inv})
        CSE_HIP_TRY(hipEventCreateWithFlags(e, hipEventDisableTiming));
    return CSE_OK;
}

// Work items of the one-wave-per-block kernels: each block's simulations split into slices of
// whole 64-simulation chunks so that the grid has about target_waves waves.
int plan_work_items(Platten *P, int64_t target_waves) {
    std::vector<WorkItem> items;
    const int64_t slices = std::max<int64_t>(1, (target_waves + P->n_blocks - 1) / P->n_blocks);
    for (int64_t b = 0; b < P->n_blocks; ++b) {
        const int64_t N = P->blk_sims[b];
        const int64_t chunks = (N + WAVE - 1) / WAVE;
        const int64_t per = std::max<int64_t>(1, (chunks + slices - 1) / slices) * WAVE;
        for (int64_t k0 = 0; k0 < N; k0 += per) {
            WorkItem w{};
            w.blk = (int32_t)b;
            w.k_begin = (uint32_t)k0;
            w.k_end = (uint32_t)std::min<int64_t>(N, k0 + per);
            items.push_back(w);
        }
    }
    P->shape_gen->fetch_add(1);   // plans captured on the old arrays become stale
    if (P->d_items) CSE_HIP_TRY(hipFree(P->d_items));
    P->d_items = nullptr;
    P->n_items = (int64_t)items.size();
    P->tune_waves = target_waves;
    return upload(&P->d_items, items.data(), items.size());
}

// Wave items of the 4-arm designs: each set's granules in slices of a power of two, so that the grid
// has about target_wgs workgroups (0: the default) of four waves.
int plan_h4_items(Platten *P, int64_t target_wgs) {
    int64_t most = 4;
    auto wgs = [&](int64_t slice) {
        int64_t n = 0;
        for (auto &S : P->h4set) n += (((int64_t)S.n_sims + GRAN2 - 1) / GRAN2 + slice - 1) / slice;
        return (n + WG / WAVE - 1) / (WG / WAVE);
    };
    if (target_wgs <= 0) target_wgs = H4_WGS;
    while (most < H4_SLICE_MAX && wgs(2 * most) >= target_wgs) most *= 2;
    std::vector<H4Item> items;
    int64_t cnt = 0, gs = 0;
    for (size_t i = 0; i < P->h4set.size(); ++i) {
        H4Set &S = P->h4set[i];
        const int64_t ng = ((int64_t)S.n_sims + GRAN2 - 1) / GRAN2;
        // a set's candidate slots (n_slices * h4_cap) must fit its keys' place in the workspace
        int64_t slice = 4;
        while (S.n_sims >= H4_PILOT_MIN_N && slice < most && 2 * slice <= ng) slice *= 2;
        S.slice = (int32_t)slice;
        S.n_slices = (int32_t)((ng + slice - 1) / slice);
        S.cnt_base = cnt;
        cnt += (int64_t)S.n_slices * WAVE;
        gs += S.n_sims;
        for (int64_t s = 0; s < S.n_slices; ++s) {
            H4Item it{};
            it.set = (int32_t)i;
            it.slice = (int32_t)s;
            it.g_begin = (uint32_t)(s * slice);
            it.g_end = (uint32_t)std::min<int64_t>(ng, (s + 1) * slice);
            items.push_back(it);
        }
    }
    // runs: the longest slices that make target_wgs items (a workgroup each)
    std::vector<H4Item> run_items;
    auto run_wgs = [&](int64_t slice) {
        int64_t n = 0;
        for (auto &S : P->h4run) n += (((int64_t)S.n_sims + GRAN2 - 1) / GRAN2 + slice - 1) / slice;
        return n;
    };
    int64_t rs = 16;   // a chunk per wave
    while (rs < H4_SLICE_MAX && run_wgs(2 * rs) >= target_wgs) rs *= 2;
    for (size_t i = 0; i < P->h4run.size(); ++i) {
        const int64_t ng = ((int64_t)P->h4run[i].n_sims + GRAN2 - 1) / GRAN2;
        for (int64_t s = 0; s * rs < ng; ++s) {
            H4Item it{};
            it.set = (int32_t)i;
            it.slice = (int32_t)s;
            it.g_begin = (uint32_t)(s * rs);
            it.g_end = (uint32_t)std::min<int64_t>(ng, (s + 1) * rs);
            run_items.push_back(it);
        }
    }
    P->shape_gen->fetch_add(1);   // plans captured on the old arrays become stale
    if (P->d_h4runitem) CSE_HIP_TRY(hipFree(P->d_h4runitem));
    P->d_h4runitem = nullptr;
    P->n_h4runitem = (int64_t)run_items.size();
    if (P->n_h4runitem)
        if (int e = upload(&P->d_h4runitem, run_items.data(), run_items.size())) return e;
    for (void *q : {(void *)P->d_h4item, (void *)P->d_h4set, (void *)P->d_h4cnt})
        if (q) CSE_HIP_TRY(hipFree(q));
    P->d_h4item = nullptr;
    P->d_h4set = nullptr;
    P->d_h4cnt = nullptr;
    P->n_h4item = (int64_t)items.size();
    P->n_gitems = (P->n_h4item + WG / WAVE - 1) / (WG / WAVE);
    P->group_sims = gs;
    P->tune_wgs = target_wgs;
    CSE_HIP_TRY(dev_malloc((void **)&P->d_h4cnt, (size_t)cnt * sizeof(uint32_t)));
    if (int e = upload(&P->d_h4set, P->h4set.data(), P->h4set.size())) return e;
    return upload(&P->d_h4item, items.data(), items.size());
}

// Workgroup items of the 2-arm kernel: rectangles of 4 row groups x 8 column groups of blocks of equal
// N over ranges of granules.
int plan_group_items(Platten *P, int64_t target_wgs) {
    std::vector<std::vector<int64_t>> groups;   // 32 blocks each (-1: none)
    {
        // rectangles of 4 row groups x 8 column groups of blocks of equal N: block (row r, column
        // c) goes to position 8 (r & 3) + (c & 7) of rectangle (r >> 2, c >> 3); a second block
        // with the same coordinates (two tiles at one grid point) opens another rectangle
        std::map<std::tuple<int64_t, int64_t, int64_t, int64_t>, std::vector<int64_t>> sq;
        for (int64_t b = 0; b < P->n_blocks; ++b) {
            const int64_t r = P->blk_row[b], c = P->blk_col[b];
            const int pos = (int)((r % SQ2R) * SQ2C + c % SQ2C);
            for (int64_t dup = 0;; ++dup) {
                auto &g = sq[std::make_tuple(P->blk_sims[b], r / SQ2R, c / SQ2C, dup)];
                if (g.empty()) g.assign(SQ2R * SQ2C, -1);
                if (g[pos] < 0) {
                    g[pos] = b;
                    break;
                }
            }
        }
        for (auto &kv : sq) groups.push_back(kv.second);
    }
    const int64_t ng = (int64_t)groups.size();
    if (target_wgs == 0) {
        // 64 granules (1,024 simulations) per item: shorter items spend their time in the final
        // atomics, longer ones leave the chip waiting for the rectangles where most quads need the
        // full step; at least 1,024 workgroups while there are granules for them.  1024 x 1024 boxes
        // x 16,384 with 2,048 / 4,096 / 8,192 / 16,384 workgroups: 430 / 362 / 333 / 351 us; 256 x 256
        // triangle x 8,192 with 512 / 1,024 / 2,048: 20.8 / 18.4 / 22.2 us
        int64_t work = 0;
        for (auto &g : groups)
            for (int64_t b : g)
                if (b >= 0) {
                    work += (P->blk_sims[b] + GRAN2 - 1) / GRAN2;
                    break;
                }
        target_wgs = std::min<int64_t>(8192, std::max<int64_t>(1024, work / 64));
    }
    int64_t slices = std::max<int64_t>(1, (target_wgs + ng - 1) / ng);
    // 2-arm items: the kernel's 32-bit sums hold 2^32 / (128 * 163) simulations; below two granules
    // an item's fixed work (the atomics) is most of it
    constexpr int64_t B2_ITEM_MAX = 8192, B2_ITEM_MIN = 2;
    std::vector<SquareItem> si;
    int64_t gs = 0;
    for (auto &g : groups) {
        int64_t first = -1;
        for (int64_t b : g)
            if (b >= 0 && first < 0) first = b;
        const int64_t N = P->blk_sims[first];
        {
            // granules per item: at most B2_ITEM_MAX (the kernel's 32-bit sums)
            const int64_t ng16 = (N + GRAN2 - 1) / GRAN2;
            const int64_t per = std::min<int64_t>(B2_ITEM_MAX, std::max<int64_t>(B2_ITEM_MIN, (ng16 + slices - 1) / slices));
            SquareItem it{};
            for (int c = 0; c < SQ2C; ++c) {   // the columns that hold a block, packed to the front
                int32_t cg = -1;
                for (int r = 0; r < SQ2R; ++r)
                    if (g[r * SQ2C + c] >= 0) cg = P->blk_cg[g[r * SQ2C + c]];
                if (cg < 0) continue;
                it.cg[it.ncg] = cg;
                for (int r = 0; r < SQ2R; ++r) it.blk[r][it.ncg] = (int32_t)g[r * SQ2C + c];
                ++it.ncg;
            }
            for (int c = it.ncg; c < SQ2C; ++c) {   // the rest: the last one's counts, no block
                it.cg[c] = it.cg[it.ncg - 1];
                for (int r = 0; r < SQ2R; ++r) it.blk[r][c] = -1;
            }
            for (int r = 0; r < SQ2R; ++r) {
                it.rg[r] = -1;
                for (int c = 0; c < it.ncg; ++c)
                    if (it.blk[r][c] >= 0) it.rg[r] = P->blk_rg[it.blk[r][c]];
            }
            for (int64_t k0 = 0; k0 < ng16; k0 += per) {
                it.g_begin = (uint32_t)k0;
                it.g_end = (uint32_t)std::min<int64_t>(ng16, k0 + per);
                gs += std::min<int64_t>(N, it.g_end * (int64_t)GRAN2) - (int64_t)it.g_begin * GRAN2;
                si.push_back(it);
            }
        }
    }
    P->shape_gen->fetch_add(1);   // plans captured on the old arrays become stale
    if (P->d_sqitems) CSE_HIP_TRY(hipFree(P->d_sqitems));
    P->d_sqitems = nullptr;
    P->n_gitems = (int64_t)si.size();
    P->group_sims = gs;
    P->tune_wgs = target_wgs;
    return upload(&P->d_sqitems, si.data(), si.size());
}

// Work items of the Phase II/III design: (tile, `chunk` consecutive trials); the posterior kernel's grid
// has `grid` workgroups (-1: two waves on every SIMD).
int plan_queue_items(Platten *P, int32_t chunk, int64_t grid) {
    std::vector<WorkItem> items;
    P->p23_item_off.clear();
    for (int64_t t = 0; t < P->n_tiles; ++t) {
        P->p23_item_off.push_back((int64_t)items.size());
        for (int64_t k0 = 0; k0 < P->tile_N[t]; k0 += chunk) {
            WorkItem w{};
            w.blk = (int32_t)t;
            w.k_begin = (uint32_t)k0;
            w.k_end = (uint32_t)std::min<int64_t>(P->tile_N[t], k0 + chunk);
            items.push_back(w);
        }
    }
    P->p23_item_off.push_back((int64_t)items.size());
    P->shape_gen->fetch_add(1);   // plans captured on the old arrays become stale
    if (P->d_p23items) CSE_HIP_TRY(hipFree(P->d_p23items));
    P->d_p23items = nullptr;
    if (int e = upload(&P->d_p23items, items.data(), items.size())) return e;
    P->p23_chunk = chunk;
    P->p23.items = P->d_p23items;
    P->p23.n_items = (int64_t)items.size();
    P->p23_grid = grid > 0 ? grid : P23_GRID;   // its work is the states, up to HP_SEGS lanes each, not the items
    P->p23_items = std::move(items);
    return CSE_OK;
}

void release_cached_memory() {
    std::vector<int> devices;
    {
        std::lock_guard<std::mutex> g(g_table_mu);
        for (auto &c : g_table_cache)
            if (c.second.p) devices.push_back(c.first);
    }
    for (int d : devices) {
        DeviceGuard guard(d);
        drop_table(d);
    }
}

void free_platten(Platten *P) {
    if (!P) return;
    if (P->shape_gen) P->shape_gen->store(PLATTEN_GONE);   // plans on this platten refuse to replay
    DeviceGuard guard(P->device);   // its work may be in flight while another device is current
    (void)hipDeviceSynchronize();
    void *ptrs[] = {P->d_theta, P->d_N,    P->d_vert_off, P->d_verts,   P->d_key_off,
                    P->d_blocks, P->d_items, P->d_cut_tbl, P->d_S_tbl,  P->d_S_order,
                    P->d_S_group, P->d_keys, P->d_Rw,      P->d_Tw,     P->d_Zw,
                    P->d_apw,    P->d_kw,    P->d_lamw,    P->d_lamg,   P->d_cls_N,
                    P->d_cls_off, P->d_cp_base, P->d_cp_mark, P->d_cp_tbl,  P->d_radii,
                    P->d_is_box, P->d_border, P->d_key_stride, P->d_h4tbl, P->d_tileT, P->d_cfg,
                    P->d_queue,  P->d_p23mem, P->d_p23row, P->d_p23tilerow, P->d_p23counts, P->d_p23items, P->d_gh, P->d_p23stats, P->d_p23look1, P->d_hnodes,
                    P->d_h4run, P->d_h4runitem, P->d_h4bits, P->d_S_pos, P->d_b2br, P->d_b2fb, P->d_b2cut, P->d_grp2, P->d_minpart, P->d_gstart, P->d_gcut, P->d_sqitems,
                    P->d_grp4, P->d_h4rows, P->d_h4set, P->d_h4item, P->d_h4u, P->d_h4eq, P->d_h4at, P->d_h4cnt, P->d_h4fb, P->d_h4plane};
    auto in_arena = [&](void *q) {
        for (auto &a : P->arenas)
            if ((unsigned char *)q >= (unsigned char *)a.first && (unsigned char *)q < (unsigned char *)a.first + a.second)
                return true;
        return false;
    };
    for (void *q : ptrs)
        if (q && !in_arena(q)) (void)hipFree(q);
    for (auto &a : P->arenas) (void)hipFree(a.first);
    P->arenas.clear();
    for (void *q : {(void *)P->d_b2tab, (void *)P->d_b4tab})
        if (q) give_table(P->device, {q, P->table_bytes});
    P->d_b2tab = P->d_b4tab = nullptr;
    for (hipEvent_t e : {P->ev_sim, P->ev_val, P->ev_fork, P->ev_inv})
        if (e) (void)hipEventDestroy(e);
    if (P->side) give_side_stream(P->device, P->side);
    P->side = nullptr;
}

}  // namespace cse
