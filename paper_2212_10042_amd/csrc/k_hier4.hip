// k_hier4.hip -- four Bernoulli arms (arm 0 control) under the hierarchical model of the
// basket case study (Section 10.1): theta_i | mu, s2 ~ N(mu, s2), mu ~ N(-1.34, 100),
// s2 ~ InvGamma(0.0005, 0.000005); statistic of treatment arm i: P(p_i > p_0 | y).
//
// Posterior table (one thread per outcome y in {0..n}^4), float64, by the Laplace node mixture
// of hier_post.hpp; the statistic 1 - P_i is summed directly as sum_j pi_j Phi(-z_j).
// The table holds float32 (1 - P_1, 1 - P_2, 1 - P_3, 0) per outcome, index ((y0 m + y1) m + y2) m + y3.
#include <math.h>

#include <algorithm>

#include "cse_internal.h"
#include "fp64_math.hpp"
#include "hier_post.hpp"
#include "kernels.h"
#include "philox.hpp"

namespace cse {

__global__ __launch_bounds__(128) void k_hier4_table(int n, int64_t n_out, float4 *__restrict__ tbl,
                                                     const HierNode *__restrict__ nodes) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n_out) return;
    const int m = n + 1;
    int y[4];
    {
        int64_t v = idx;
        for (int a = 3; a >= 0; --a) {
            y[a] = (int)(v % m);
            v /= m;
        }
    }
    const double nv[4] = {(double)n, (double)n, (double)n, (double)n};
    double Sc[3];
    hier_complements(y, nv, nodes, Sc);
    float4 o;
    o.x = (float)Sc[0];
    o.y = (float)Sc[1];
    o.z = (float)Sc[2];
    o.w = 0.0f;
    tbl[idx] = o;
}

// Basket design table: float32 (1 - P_0, .., 1 - P_3) per outcome, P_a = P(p_a > p_0a | y).
struct Theta0 {
    double v[4];
};
__global__ __launch_bounds__(128) void k_basket_table(int n, int64_t n_out, Theta0 t0, float4 *__restrict__ tbl,
                                                      const HierNode *__restrict__ nodes) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n_out) return;
    const int m = n + 1;
    int y[4];
    {
        int64_t v = idx;
        for (int a = 3; a >= 0; --a) {
            y[a] = (int)(v % m);
            v /= m;
        }
    }
    double Sc[4];
    basket_posterior(y, (double)n, t0.v, nodes, Sc);
    tbl[idx] = make_float4((float)Sc[0], (float)Sc[1], (float)Sc[2], (float)Sc[3]);
}

hipError_t launch_basket_table(int n, const double *theta0, float4 *tbl, const HierNode *nodes, hipStream_t st) {
    const int64_t m = n + 1;
    const int64_t n_out = m * m * m * m;
    Theta0 t0;
    for (int a = 0; a < 4; ++a) t0.v[a] = theta0[a];
    hipLaunchKernelGGL(k_basket_table, dim3((uint32_t)((n_out + 127) / 128)), dim3(128), 0, st, n, n_out, t0, tbl,
                       nodes);
    return hipGetLastError();
}

// Rejecting outcomes of configuration b = 1..nb (a treatment arm of b with its statistic below the cut;
// the comparison is the one the keyed pass makes): bit y3 of word (b - 1) H4_BITS + (36 y0 + y1) 36 + y2.
__global__ void k_h4_bits(const float4 *__restrict__ tbl, float cut, int nb, uint64_t *__restrict__ bits) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= H4_BITS) return;
    uint64_t w[4] = {0, 0, 0, 0};   // per arm of the row
    for (int y3 = 0; y3 <= NP35; ++y3) {
        const float4 q = tbl[i * (NP35 + 1) + y3];
        w[0] |= (uint64_t)(q.x < cut) << y3;
        w[1] |= (uint64_t)(q.y < cut) << y3;
        w[2] |= (uint64_t)(q.z < cut) << y3;
        w[3] |= (uint64_t)(q.w < cut) << y3;
    }
    for (int b = 1; b <= nb; ++b)
        bits[(b - 1) * H4_BITS + i] = (b & 1 ? w[0] : 0) | (b & 2 ? w[1] : 0) | (b & 4 ? w[2] : 0) | (b & 8 ? w[3] : 0);
}

hipError_t launch_h4_bits(const float4 *tbl, float cut, int nb, uint64_t *bits, hipStream_t st) {
    hipLaunchKernelGGL(k_h4_bits, dim3((uint32_t)((H4_BITS + 255) / 256)), dim3(256), 0, st, tbl, cut, nb, bits);
    return hipGetLastError();
}

hipError_t launch_hier4_table(int n, float4 *tbl, const HierNode *nodes, hipStream_t st) {
    const int64_t m = n + 1;
    const int64_t n_out = m * m * m * m;
    hipLaunchKernelGGL(k_hier4_table, dim3((uint32_t)((n_out + 127) / 128)), dim3(128), 0, st, n, n_out, tbl,
                       nodes);
    return hipGetLastError();
}

__device__ __forceinline__ void wave_sync4() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Statistic planes: S_b = min_{a in b} of the outcome's row, for every configuration b = 1..nb, at the
// outcome's tiled place (H4_SLAB).
__global__ void k_h4_planes(const float4 *__restrict__ tbl, int64_t n, int nb, float *__restrict__ planes) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    constexpr int M1 = NP35 + 1;
    const float4 q = tbl[i];
    const uint32_t y3 = (uint32_t)(i % M1), y2 = (uint32_t)(i / M1 % M1);
    const int64_t at = i / (M1 * M1) * H4_SLAB + 8 * h4_code2(y2) + h4_code3(y3);
    for (int b = 1; b <= nb; ++b) {
        float sb = INFINITY;
        if (b & 1) sb = fminf(sb, q.x);
        if (b & 2) sb = fminf(sb, q.y);
        if (b & 4) sb = fminf(sb, q.z);
        if (b & 8) sb = fminf(sb, q.w);
        planes[(b - 1) * H4_PLANE + at] = sb;
    }
}

hipError_t launch_h4_planes(const float4 *tbl, int nb, float *planes, hipStream_t st) {
    const int64_t n = (int64_t)(NP35 + 1) * (NP35 + 1) * (NP35 + 1) * (NP35 + 1);
    hipLaunchKernelGGL(k_h4_planes, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, st, tbl, n, nb, planes);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Simulation, 4 arms x 35 patients (words a*35 .. a*35+34 for arm a: 35 Philox blocks).
//
// k_h4_count counts every simulation's successes at every distinct threshold of each arm once for the
// whole platten (16^4 boxes: 64 thresholds, where counting per batch of 64 boxes repeated them
// 340-fold) into the count table.
//
// k_h4_tiles (with keys) takes 64 tiles per wave, one per lane, and one simulation at a time for all of
// them: the tile's sums and candidate list are its lane's own, nothing crosses lanes.  Tiles are ordered
// so that a wave mostly holds one pair of thresholds of arms 0 and 1 and 8 x 8 neighbouring ones of
// arms 2 and 3: their outcomes lie in a few lines of the table (tiled for that, H4_SLAB), where one
// lane per simulation touched one line per lane.  Four simulations share the arithmetic on packed
// counts; per simulation the table offset is one packed 16-bit dot product.  A calibration stores
// only candidate keys (k_h4_pilot).
// Bound by the gathers' addresses (40 cache lines looked up per instruction).  16^4 boxes x 32,768
// simulations, 4-arm calibration: counts 0.012, pilot 0.155, tiles 2.13 ms (4.40 with Philox words
// and counts per batch of 64 boxes, lane = simulation, and 7.9 GB of keys stored) and the selection
// 1.52 -> 0.56 ms.  Rows of 36 or 64 floats instead of 4 x 8 tiles: 2.33 and 2.22 ms.
//
// k_h4_runs (without keys) takes up to 8 tiles per lane that differ in arm 3's threshold alone.
// ------------------------------------------------------------------------------------------
constexpr int H4C_NB = NP35;   // Philox blocks of a simulation
__global__ __launch_bounds__(WG) void k_h4_count(const Grp4 *__restrict__ grp, int32_t n_grp, uint32_t win_b,
                                                 uint32_t key0, uint32_t key1, uint2 *__restrict__ tab) {
    constexpr int NWV = WG / WAVE;
    __shared__ uint32_t words[4 * H4C_NB][WAVE];
    __shared__ uint2 tr[NWV][WAVE];
    const int lane = threadIdx.x & (WAVE - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t k0 = win_b * GRAN2 + blockIdx.x * WAVE;
    for (int b = wv; b < H4C_NB; b += NWV) {
        const u32x4 w = philox_block((uint32_t)b, k0 + (uint32_t)lane, key0, key1);
        words[4 * b + 0][lane] = w.x;
        words[4 * b + 1][lane] = w.y;
        words[4 * b + 2][lane] = w.z;
        words[4 * b + 3][lane] = w.w;
    }
    __syncthreads();
    for (int g = (int)blockIdx.y * NWV + wv; g < n_grp; g += (int)gridDim.y * NWV) {   // uniform over the wave
        const Grp4 *__restrict__ G = grp + g;
        const uint32_t n = (uint32_t)G->n_sims;
        if (k0 >= n) continue;
        const int arm = G->arm;
        uint32_t T[8], y[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            T[u] = G->T[u];
            y[u] = 0u;
        }
        const uint32_t(*w)[WAVE] = words + arm * NP35;
#pragma unroll 7
        for (int j = 0; j < NP35; ++j) {
            const uint32_t x = w[j][lane];
#pragma unroll
            for (int u = 0; u < 8; ++u) y[u] += (x < T[u]) ? 1u : 0u;
        }
        // (simulation, threshold) bytes -> threshold-major granules: lane = granule q of the chunk,
        // threshold t, half h of its 16 simulations
        tr[wv][lane] = make_uint2(y[0] | (y[1] << 8) | (y[2] << 16) | (y[3] << 24),
                                  y[4] | (y[5] << 8) | (y[6] << 16) | (y[7] << 24));
        wave_sync4();
        const int q = lane >> 4, t = (lane >> 1) & 7, h = lane & 1;
        const uint8_t *src = reinterpret_cast<const uint8_t *>(&tr[wv][16 * q + 8 * h]) + t;
        uint32_t b[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) b[i] = src[8 * i];
        wave_sync4();
        const uint32_t kq = k0 + (uint32_t)(16 * q);   // the granule's first simulation
        if (kq >= n || t >= G->n_thr) continue;
        const int64_t stride = G->stride;
        uint2 *__restrict__ dst = tab + (G->row + t * stride + (int64_t)(kq / GRAN2 - win_b)) * 2 + h;
        dst[0] = make_uint2(b[0] | (b[1] << 8) | (b[2] << 16) | (b[3] << 24), b[4] | (b[5] << 8) | (b[6] << 16) | (b[7] << 24));
        if (arm >= 2) {   // the code rows
#pragma unroll
            for (int i = 0; i < 8; ++i) b[i] = arm == 2 ? h4_code2(b[i]) : h4_code3(b[i]);
            dst[16 * stride] =
                make_uint2(b[0] | (b[1] << 8) | (b[2] << 16) | (b[3] << 24), b[4] | (b[5] << 8) | (b[6] << 16) | (b[7] << 24));
        }
    }
}

typedef unsigned short us2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ us2 as_us2(uint32_t v) { return __builtin_bit_cast(us2, v); }
__device__ __forceinline__ uint32_t as_u32(us2 v) { return __builtin_bit_cast(uint32_t, v); }
// Table offsets of four simulations, whose counts (or codes) are the bytes of y0, y1, y2 and y3:
// w01 (36 y0 + y1) + w23 (m2 y2 + y3) + base.
__device__ __forceinline__ void h4_offsets(uint32_t y0, uint32_t y1, uint32_t y2, uint32_t y3, uint16_t m2, uint32_t w,
                                           uint32_t base, uint32_t off[4]) {
    auto ev = [](uint32_t v) { return as_us2(v & 0x00FF00FFu); };                               // simulations 0, 2
    auto od = [](uint32_t v) { return as_us2(__builtin_amdgcn_perm(0u, v, 0x0C030C01u)); };     // simulations 1, 3
    const us2 c36 = {(unsigned short)(NP35 + 1), (unsigned short)(NP35 + 1)}, cm = {m2, m2};
    const uint32_t ae = as_u32(ev(y0) * c36 + ev(y1)), ao = as_u32(od(y0) * c36 + od(y1));
    const uint32_t be = as_u32(ev(y2) * cm + ev(y3)), bo = as_u32(od(y2) * cm + od(y3));
    // (low or high halves of a and b side by side) . (w01, w23)
    off[0] = __builtin_amdgcn_udot2(as_us2(__builtin_amdgcn_perm(be, ae, 0x05040100u)), as_us2(w), base, false);
    off[1] = __builtin_amdgcn_udot2(as_us2(__builtin_amdgcn_perm(bo, ao, 0x05040100u)), as_us2(w), base, false);
    off[2] = __builtin_amdgcn_udot2(as_us2(__builtin_amdgcn_perm(be, ae, 0x07060302u)), as_us2(w), base, false);
    off[3] = __builtin_amdgcn_udot2(as_us2(__builtin_amdgcn_perm(bo, ao, 0x07060302u)), as_us2(w), base, false);
}
__device__ __forceinline__ uint32_t u4_get(const uint4 &v, int i) {
    return i == 0 ? v.x : (i == 1 ? v.y : (i == 2 ? v.z : v.w));
}
constexpr uint32_t H4_W_PLANE = (uint32_t)(4 * H4_SLAB) | (4u << 16);            // byte offsets into a plane (codes, m2 = 8)
static_assert(4 * H4_SLAB < 65536 && 15 * 4 * H4_PLANE < (1ll << 32), "16-bit weights, 32-bit offsets");

// A set's count rows in LDS, a chunk (64 simulations) at a time: the distinct rows are loaded once for
// the wave, 16 rows per instruction, and each lane reads its own from LDS (a global 16-byte load per
// lane and arm took 63 cycles whether the lanes' addresses agreed or not, and 960 of 1,640 us on the
// basket's 16^4 boxes with one tile per lane).  The next chunk's first H4_AHEAD * 16 rows are loaded ahead.
constexpr int H4_AHEAD = 3;
struct H4Rows {
    const uint4 *__restrict__ tab;
    const uint32_t *__restrict__ rows;
    uint4 *__restrict__ lds;
    int32_t n;
    const uint4 *src[H4_AHEAD];   // this lane's piece of chunk 0 of the rows loaded ahead (past the list: its last row)
    uint4 nx[H4_AHEAD];
    __device__ __forceinline__ H4Rows(const uint4 *__restrict__ tab_, const uint32_t *__restrict__ rows_, int32_t n_,
                                      uint4 *lds_)
        : tab(tab_), rows(rows_), lds(lds_), n(n_) {
        const int lane = threadIdx.x & (WAVE - 1);
#pragma unroll
        for (int i = 0; i < H4_AHEAD; ++i) src[i] = tab + rows[min(16 * i + (lane >> 2), n - 1)] + (lane & 3);
    }
    __device__ __forceinline__ void load(uint32_t chunk) {
#pragma unroll
        for (int i = 0; i < H4_AHEAD; ++i) nx[i] = src[i][4 * chunk];
    }
    __device__ __forceinline__ void store(uint32_t chunk) {   // the loaded chunk and its further rows into LDS
        const int lane = threadIdx.x & (WAVE - 1);
        wave_sync4();
#pragma unroll
        for (int i = 0; i < H4_AHEAD; ++i) {
            const int r = 16 * i + (lane >> 2);
            if (r < n) lds[r * H4_ROW_LDS + (lane & 3)] = nx[i];
        }
        for (int r = 16 * H4_AHEAD + (lane >> 2); r < n; r += 16)
            lds[r * H4_ROW_LDS + (lane & 3)] = tab[rows[r] + 4 * chunk + (lane & 3)];
        wave_sync4();
    }
};

// Upper bound of each tile's k-th smallest key from the first h4_pilot(N) simulations: about the order
// statistic of rank r = mu + z sd + z^2 / 6 + 1, mu = m k / N (z = 6 by default; the z^2 / 6 is the
// skewness of a Poisson count: without it and at z = 5 one seed in three left some of the 60,112
// tiles of 16^4 boxes short).  A histogram finds the bin of that order statistic, 8 bins per octave
// from 2^-20 to 1/4, then 256 per unit up to 1 (keys of tiles deep in the null crowd towards 1); the
// bound is its upper edge, unless that admits too many pilot keys: then the bin is divided
// again, down to a single value where the statistic has an atom there (few distinct outcomes), and
// the tile's keys equal to the bound are counted, not kept.  One workgroup per set, lane = tile, its
// four waves share the pilot's simulations.
constexpr int H4P_LOG = 18 * 8, H4P_BINS = H4P_LOG + 192 + 1;
constexpr uint32_t H4P_BIN0 = (127u - 20u) << 3;
// LDS of a workgroup of four waves (160 KB): the rows of a set, and the pilot's static arrays (histogram, ranges,
// segments) or the keys' transposes of the every-key pass; sets of runs hold as many rows as fit without either.
constexpr int H4_LDS = 160 << 10, H4P_STATIC = H4P_BINS * WAVE / 2 * 4 + WAVE * 8 + WG * 4 + 256;
static_assert(4 * H4_SET_ROWS * H4_ROW_LDS * 16 + H4P_STATIC <= H4_LDS, "the pilot fits");
static_assert((4 * H4_SET_ROWS + WG) * H4_ROW_LDS * 16 <= H4_LDS, "the every-key pass fits");
static_assert(4 * H4_ROWS * WAVE * H4_ROW_LDS * 16 <= H4_LDS, "runs fit");
__device__ __forceinline__ int h4p_bin(float v) {   // v in [0, 1]
    const int lo = max((int)(__float_as_uint(v) >> 20) - (int)H4P_BIN0, 0);
    const int hi = H4P_LOG - 64 + (int)(v * 256.0f);
    return v < 0.25f ? lo : min(hi, H4P_BINS - 1);
}
__device__ __forceinline__ float h4p_edge(int b) {   // upper edge: every key of the bin lies below it
    return b < H4P_LOG ? __uint_as_float(((uint32_t)b + 1u + H4P_BIN0) << 20) : 0.25f + (float)(b + 1 - H4P_LOG) * (1.0f / 256.0f);
}
__global__ __launch_bounds__(WG) void k_h4_pilot(const H4Set *__restrict__ sets, const uint32_t *__restrict__ rows,
                                                 int32_t max_rows, const uint4 *__restrict__ tab,
                                                 const float *__restrict__ planes, const int32_t *__restrict__ kk,
                                                 float margin, float *__restrict__ U, uint32_t *__restrict__ eq,
                                                 uint32_t *__restrict__ fb) {
    constexpr int NWV = WG / WAVE;
    __shared__ uint32_t hist[H4P_BINS * WAVE / 2];   // 16-bit counts, two lanes per word
    __shared__ uint2 range[WAVE];                    // per tile: the keys' bits [x, y) being divided
    __shared__ uint32_t more;
    __shared__ float part[NWV][WAVE];                // keys per segment of the bins
    const int lane = threadIdx.x & (WAVE - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const H4Set *__restrict__ S = sets + blockIdx.x;
    if (blockIdx.x == 0 && threadIdx.x == 0) fb[0] = 0u;
    const int32_t N = S->n_sims;
    const int32_t t = S->tile[lane];
    const int32_t k = t >= 0 ? kk[t] : 0;
    if (wv == 0 && t >= 0) eq[t] = 0u;
    if (N < H4_PILOT_MIN_N) {   // uniform: every key is a candidate
        if (wv == 0 && t >= 0) U[t] = INFINITY;
        return;
    }
    const bool sel = k >= 1 && k <= N;
    const int m = h4_pilot(N), nch = m / WAVE;
    const uint32_t base = (S->cfg[lane] - 1u) * (uint32_t)(4 * H4_PLANE);
    extern __shared__ uint4 h4_lds[];
    H4Rows rr(tab, rows + S->row_at, S->n_rows, h4_lds + (size_t)wv * max_rows * H4_ROW_LDS);
    const uint4 *__restrict__ l0 = rr.lds + S->row[0][lane] * H4_ROW_LDS, *__restrict__ l1 = rr.lds + S->row[1][lane] * H4_ROW_LDS,
                *__restrict__ l2 = rr.lds + S->row[4][lane] * H4_ROW_LDS, *__restrict__ l3 = rr.lds + S->row[5][lane] * H4_ROW_LDS;
    const float pr = (float)k / (float)N, mean = pr * (float)m;
    // at most a fifth of the pilot: a slice has room for half of its keys (a wide margin, CSE_OPT_H4_MARGIN, ends there)
    const float rank = fminf(mean + margin * sqrtf(mean * (1.0f - pr)) + margin * margin * (1.0f / 6.0f) + 1.0f, 0.2f * (float)m);
    // pilot keys the bound may admit before its bin is divided: those of 1,800 candidates or a fifth of the
    // pilot, or a quarter over rank.  (Without the fifth, tiles deep in the null, whose keys crowd in one bin,
    // admitted nearly all keys of up to 2,048 simulations, so that slices overflowed and all was regenerated:
    // 6^4 boxes x 1,500 721 us, 150 so.)
    const float most = fmaxf(1.25f * rank + 8.0f, fminf(1800.0f * (float)m / (float)N, 0.2f * (float)m));
    uint2 r = make_uint2(0u, 0xFFFFFFFFu);    // first pass: the fixed bins
    float below = 0.0f;                       // pilot keys below the range (wave 0)
    bool open = sel && wv == 0;               // wave 0: the tile's bound is not final
    for (int pass = 0;; ++pass) {
        for (int i = threadIdx.x; i < H4P_BINS * WAVE / 2; i += WG) hist[i] = 0u;
        if (threadIdx.x == 0) more = 0u;
        if (pass > 0) r = range[lane];
        // later passes: bins of 2^sh consecutive floats, at most 256
        const uint32_t width = r.y - r.x, sh = width > 256u ? 24u - (uint32_t)__builtin_clz(width - 1u) : 0u;
        __syncthreads();
        if (wv < nch) rr.load(wv);
        for (int c = wv; c < nch; c += NWV) {
            rr.store(c);
            if (c + NWV < nch) rr.load(c + NWV);
            for (int g = 0; g < 4; ++g) {
                const uint4 y0 = l0[g], y1 = l1[g], y2 = l2[g], y3 = l3[g];
                float v[GRAN2];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    uint32_t off[4];
                    h4_offsets(u4_get(y0, q), u4_get(y1, q), u4_get(y2, q), u4_get(y3, q), 8, H4_W_PLANE, base, off);
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        v[4 * q + j] = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(planes) + off[j]);
                }
#pragma unroll
                for (int j = 0; j < GRAN2; ++j) {
                    const uint32_t bits = __float_as_uint(v[j]);
                    if (pass == 0 || (bits >= r.x && bits < r.y)) {
                        const int b = pass == 0 ? h4p_bin(v[j]) : (int)((bits - r.x) >> sh);
                        atomicAdd(&hist[b * (WAVE / 2) + (lane >> 1)], 1u << (16 * (lane & 1)));
                    }
                }
            }
        }
        __syncthreads();
        // each wave sums a segment of the bins per tile, wave 0 finds the segment and then the bin (one walk
        // over 337 bins: 180 us at 16^4 boxes, 155 so)
        const int nb = pass == 0 ? H4P_BINS : 256, seg = (nb + NWV - 1) / NWV;
        auto bin = [&](int b) { return (float)((hist[b * (WAVE / 2) + (lane >> 1)] >> (16 * (lane & 1))) & 0xFFFFu); };
        {
            float c = 0.0f;   // whole numbers below 2^24: exact in any order
            const int e = min(nb, (wv + 1) * seg);
#pragma unroll 4
            for (int b = wv * seg; b < e; ++b) c += bin(b);
            part[wv][lane] = c;
        }
        __syncthreads();
        if (open) {
            float run = below;
            int b = 0;
            for (int w = 0; w < NWV && run + part[w][lane] < rank; ++w) {
                run += part[w][lane];
                b += seg;
            }
            b = min(b, nb);
            float c = 0.0f;
            for (; b < nb; ++b) {
                c = bin(b);
                if (run + c >= rank) break;
                run += c;
            }
            float u = INFINITY;   // fewer than r pilot keys: every key is a candidate
            open = false;
            if (b < nb) {
                if (pass == 0) {
                    u = h4p_edge(b);
                    r = make_uint2(b == 0 ? 0u : __float_as_uint(h4p_edge(b - 1)), __float_as_uint(u));
                } else {
                    r.x += (uint32_t)b << sh;
                    r.y = min(r.y, r.x + (1u << sh));
                    u = __uint_as_float(r.y);
                }
                if (run + c > most) {
                    if (r.y - r.x <= 1u) u = __uint_as_float(r.x);   // one value: its keys are counted
                    else open = true;
                }
                below = run;
            }
            if (open) atomicAdd(&more, 1u);
            else U[t] = u;
        }
        if (wv == 0) range[lane] = open ? r : make_uint2(0u, 0u);
        __syncthreads();
        if (more == 0u) break;   // uniform
        __syncthreads();         // `more` is read before the next pass clears it
    }
    if (wv == 0 && t >= 0 && !sel) U[t] = -INFINITY;   // no selection
}

// Rejection counts and score sums with keys, from the statistic planes: every key stored, or (CAND) the
// keys below the tile's bound U as candidates, those equal to it counted.
template <bool CAND, bool SCORE>
__global__ __launch_bounds__(WG) void k_h4_tiles(const H4Set *__restrict__ sets, const H4Item *__restrict__ items,
                                                 int64_t n_items, const uint32_t *__restrict__ rows, int32_t max_rows,
                                                 const uint4 *__restrict__ tab, uint32_t win_b,
                                                 uint32_t win_e,
                                                 const float *__restrict__ planes, float cut,
                                                 uint32_t *__restrict__ R, unsigned long long *__restrict__ sumT,
                                                 float *__restrict__ keys, const float *__restrict__ U,
                                                 uint32_t *__restrict__ eq, uint32_t *__restrict__ cnt) {
    constexpr uint32_t H = 0x80808080u;
    const int lane = threadIdx.x & (WAVE - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t it = (int64_t)blockIdx.x * (WG / WAVE) + wv;
    if (it >= n_items) return;
    const H4Item *__restrict__ I = items + it;
    const uint32_t gb = max(I->g_begin, win_b), ge = min(I->g_end, win_e);
    if (gb >= ge) return;
    const H4Set *__restrict__ S = sets + I->set;
    const int32_t N = S->n_sims, t = S->tile[lane];
    const uint32_t cfg = S->cfg[lane];
    extern __shared__ uint4 h4_lds[];
    H4Rows rr(tab, rows + S->row_at, S->n_rows, h4_lds + (size_t)wv * max_rows * H4_ROW_LDS);
    auto lrow = [&](int a) { return rr.lds + S->row[a][lane] * H4_ROW_LDS; };
    const uint4 *__restrict__ l0 = lrow(0), *__restrict__ l1 = lrow(1), *__restrict__ l2 = lrow(2),
                *__restrict__ l3 = lrow(3), *__restrict__ c2 = lrow(4), *__restrict__ c3 = lrow(5);
    const uint32_t base = (cfg - 1u) * (uint32_t)(4 * H4_PLANE);
    const float bound = CAND ? (t >= 0 ? U[t] : -INFINITY) : 0.0f;
    // CAND: keys at or above it matter to nothing (the float after the bound: keys equal to it count)
    const float look = fmaxf(cut, bound >= 0.0f && bound < INFINITY ? __uint_as_float(__float_as_uint(bound) + 1u) : bound);
    uint32_t ncand = 0u, neq = 0u, cap = 0u;
    float *__restrict__ kp = keys;
    if (!CAND) kp = keys + S->key_base;
    if (CAND) {
        cap = (uint32_t)h4_cap(N, S->slice);
        kp = keys + S->key_base + ((int64_t)lane * S->n_slices + I->slice) * cap;
    }
    const int64_t kstride = (int64_t)S->n_lanes * WAVE;
    uint32_t aR = 0u, a0 = 0u, a1 = 0u, a2 = 0u, a3 = 0u;
    auto add = [&](uint32_t f, uint32_t y0, uint32_t y1, uint32_t y2, uint32_t y3) {   // f: 128 per rejecting simulation
        aR += (uint32_t)__popc(f);
        if (SCORE) {
            a0 = __builtin_amdgcn_udot4(f, y0, a0, false);
            a1 = __builtin_amdgcn_udot4(f, y1, a1, false);
            a2 = __builtin_amdgcn_udot4(f, y2, a2, false);
            a3 = __builtin_amdgcn_udot4(f, y3, a3, false);
        }
    };
    rr.load((gb - win_b) / 4);   // items and windows begin at chunks
    for (uint32_t g0 = gb; g0 < ge; g0 += 4) {
    rr.store((g0 - win_b) / 4);
    if (g0 + 4 < ge) rr.load((g0 + 4 - win_b) / 4);
    for (uint32_t i = 0; i < 4; ++i) {
        const uint32_t g = g0 + i;
        if (g >= ge) break;   // uniform
        const uint4 y0 = l0[i], y1 = l1[i];
        uint4 y2 = make_uint4(0u, 0u, 0u, 0u), y3 = y2, e2 = y2, e3 = y2;
        if (SCORE) {
            y2 = l2[i];
            y3 = l3[i];
        }
        e2 = c2[i];
        e3 = c3[i];
        const int nv = N - (int)(g * GRAN2);   // simulations from this granule on (uniform)
        float v[GRAN2];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t off[4];
            h4_offsets(u4_get(y0, q), u4_get(y1, q), u4_get(e2, q), u4_get(e3, q), 8, H4_W_PLANE, base, off);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                v[4 * q + j] = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(planes) + off[j]);
        }
        if (!CAND) {
            // 16 keys of each of 64 tiles, through LDS: four lanes store a tile's 64 bytes (a lane's own 16 keys
            // in four stores of 16 bytes, each to a line of its own: 5.4 ms where this takes 3.8)
            uint4 *__restrict__ tr = h4_lds + (size_t)(WG / WAVE) * max_rows * H4_ROW_LDS + (size_t)wv * WAVE * H4_ROW_LDS;
            wave_sync4();
#pragma unroll
            for (int q = 0; q < 4; ++q)
                tr[lane * H4_ROW_LDS + q] = make_uint4(__float_as_uint(v[4 * q]), __float_as_uint(v[4 * q + 1]),
                                                       __float_as_uint(v[4 * q + 2]), __float_as_uint(v[4 * q + 3]));
            wave_sync4();
            float *__restrict__ kc = kp + (int64_t)(g / 4) * kstride + (g % 4) * GRAN2;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int l = 16 * r + (lane >> 2);
                if (l < S->n_lanes) *reinterpret_cast<uint4 *>(kc + l * WAVE + 4 * (lane & 3)) = tr[l * H4_ROW_LDS + (lane & 3)];
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int n4 = nv - 4 * q;   // uniform
            const uint32_t valid = n4 >= 4 ? H : (n4 <= 0 ? 0u : H >> (8 * (4 - n4)));
            uint32_t f = 0u;
            const float *vq = v + 4 * q;
            const bool any = fminf(fminf(vq[0], vq[1]), fminf(vq[2], vq[3])) < (CAND ? look : cut);
            if (__ballot(any) == 0ull) continue;   // rejections and candidates are a few per cent
#pragma unroll
            for (int j = 0; j < 4; ++j) f |= vq[j] < cut ? 0x80u << (8 * j) : 0u;
            f &= valid;
            add(f, u4_get(y0, q), u4_get(y1, q), u4_get(y2, q), u4_get(y3, q));
            if (CAND) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (vq[j] <= bound && j < n4) {
                        if (vq[j] == bound) {
                            ++neq;
                        } else {
                            if (ncand < cap) kp[ncand] = vq[j];
                            ++ncand;
                        }
                    }
            }
        }
    }
    }
    if (t < 0) return;
    if (CAND) {
        cnt[S->cnt_base + (int64_t)I->slice * WAVE + lane] = ncand;
        if (neq) atomicAdd(&eq[t], neq);
    }
    if (aR) {
        atomicAdd(&R[t], aR);
        if (SCORE) {   // the sums of two arms in the halves of one 64-bit word (at most 35 * 2^24 each)
            atomicAdd(&sumT[2 * (int64_t)t], (unsigned long long)(a0 >> 7) | ((unsigned long long)(a1 >> 7) << 32));
            atomicAdd(&sumT[2 * (int64_t)t + 1], (unsigned long long)(a2 >> 7) | ((unsigned long long)(a3 >> 7) << 32));
        }
    }
}

// Rejection counts and score sums of runs: a lane takes up to 8 tiles that differ in arm 3's threshold
// alone, so one gather per simulation (the rejecting y3 of its y0, y1, y2 and configuration, as bits)
// serves them all, and each tile tests its own y3 in registers.  The four waves of a workgroup take
// chunks of 64 simulations in turn and add up in LDS.  Bound by vector instructions (four per tile and
// simulation, 58% of the issue slots with three waves per SIMD; four waves spill).  Basket, 16^4 boxes
// x 32,768 simulations: 1.37 ms with one byte gathered per tile and simulation, 0.42 ms so (0.58 without
// pieces of one length together, 0.50 with a wave's sums added to memory by itself).  Runs of one tile
// are still faster than lanes of one tile (0.21 and 0.35 ms at 1,899 tiles x 131,072 simulations): the
// words of one pair of thresholds of arms 0 and 1 lie in a line or two.
template <bool SCORE>
__global__ __launch_bounds__(WG) void k_h4_runs(const H4Run *__restrict__ sets, const H4Item *__restrict__ items,
                                                const uint32_t *__restrict__ rows, int32_t max_rows,
                                                const uint4 *__restrict__ tab, uint32_t win_b, uint32_t win_e,
                                                const uint64_t *__restrict__ bits, uint32_t *__restrict__ R,
                                                unsigned long long *__restrict__ sumT) {
    constexpr uint32_t ONE = 0x01010101u;
    constexpr uint32_t W = (uint32_t)(8 * (NP35 + 1)) | (8u << 16);   // bytes per (36 y0 + y1) and per y2
    const int lane = threadIdx.x & (WAVE - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const H4Item *__restrict__ I = items + blockIdx.x;
    const uint32_t gb = max(I->g_begin, win_b), ge = min(I->g_end, win_e);
    if (gb >= ge) return;   // the whole workgroup
    const H4Run *__restrict__ S = sets + I->set;
    const int32_t N = S->n_sims, n_run = S->n_run;
    extern __shared__ uint4 h4_lds[];
    H4Rows rr(tab, rows + S->row_at, S->n_rows, h4_lds + (size_t)wv * max_rows * H4_ROW_LDS);
    auto lrow = [&](int a) { return rr.lds + S->row[a][lane] * H4_ROW_LDS; };
    const uint4 *__restrict__ l0 = lrow(0), *__restrict__ l1 = lrow(1), *__restrict__ l2 = lrow(2);
    const uint4 *__restrict__ l3[H4_RUN];
#pragma unroll
    for (int r = 0; r < H4_RUN; ++r) l3[r] = lrow(3 + r);
    const uint32_t base = (S->cfg[lane] - 1u) * (uint32_t)(8 * H4_BITS);
    uint32_t aR[H4_RUN], a0[H4_RUN], a1[H4_RUN], a2[H4_RUN], a3[H4_RUN];
#pragma unroll
    for (int r = 0; r < H4_RUN; ++r) aR[r] = a0[r] = a1[r] = a2[r] = a3[r] = 0u;
    const uint32_t gw = gb + 4u * (uint32_t)wv;   // items and windows begin at chunks; the waves take them in turn
    if (gw < ge) rr.load((gw - win_b) / 4);
    for (uint32_t g0 = gw; g0 < ge; g0 += WG / WAVE * 4) {
        rr.store((g0 - win_b) / 4);
        if (g0 + WG / WAVE * 4 < ge) rr.load((g0 + WG / WAVE * 4 - win_b) / 4);
#pragma unroll 1
        for (uint32_t i = 0; i < 4; ++i) {
            const uint32_t g = g0 + i;
            if (g >= ge) break;   // uniform
            const uint4 y0 = l0[i], y1 = l1[i], y2 = l2[i];
            uint64_t m[GRAN2];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t off[4];
                h4_offsets(u4_get(y0, q), u4_get(y1, q), 0u, u4_get(y2, q), 0, W, base, off);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    m[4 * q + j] = *reinterpret_cast<const uint64_t *>(reinterpret_cast<const char *>(bits) + off[j]);
            }
            const int nv = N - (int)(g * GRAN2);   // simulations from this granule on (uniform)
#pragma unroll
            for (int r = 0; r < H4_RUN; ++r) {
                if (r >= n_run) break;   // uniform
                const uint4 y3 = l3[r][i];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int n4 = nv - 4 * q;
                    const uint32_t valid = n4 >= 4 ? ONE : (n4 <= 0 ? 0u : ONE >> (8 * (4 - n4)));
                    const uint32_t w = u4_get(y3, q);
                    // shifts by the byte in the low 6 bits: counts are at most 35
                    const uint32_t x0 = (uint32_t)(m[4 * q] >> (w & 63u)), x1 = (uint32_t)(m[4 * q + 1] >> ((w >> 8) & 63u)),
                                   x2 = (uint32_t)(m[4 * q + 2] >> ((w >> 16) & 63u)), x3 = (uint32_t)(m[4 * q + 3] >> (w >> 24));
                    const uint32_t x01 = __builtin_amdgcn_perm(x1, x0, 0x0C0C0400u), x23 = __builtin_amdgcn_perm(x3, x2, 0x04000C0Cu);
                    const uint32_t f = (x01 | x23) & valid;
                    aR[r] += (uint32_t)__popc(f);
                    if (SCORE) {
                        a0[r] = __builtin_amdgcn_udot4(f, u4_get(y0, q), a0[r], false);
                        a1[r] = __builtin_amdgcn_udot4(f, u4_get(y1, q), a1[r], false);
                        a2[r] = __builtin_amdgcn_udot4(f, u4_get(y2, q), a2[r], false);
                        a3[r] = __builtin_amdgcn_udot4(f, w, a3[r], false);
                    }
                }
            }
        }
    }
    // the waves' sums through LDS: one addition to memory per tile and workgroup
    constexpr int V = SCORE ? 5 : 1;
    uint32_t *__restrict__ red = reinterpret_cast<uint32_t *>(h4_lds);
    __syncthreads();
    for (int i = threadIdx.x; i < V * H4_RUN * WAVE; i += WG) red[i] = 0u;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < H4_RUN; ++r) {
        if (aR[r] == 0u) continue;
        uint32_t *__restrict__ w = red + V * r * WAVE + lane;
        atomicAdd(&w[0], aR[r]);
        if (SCORE) {
            atomicAdd(&w[WAVE], a0[r]);
            atomicAdd(&w[2 * WAVE], a1[r]);
            atomicAdd(&w[3 * WAVE], a2[r]);
            atomicAdd(&w[4 * WAVE], a3[r]);
        }
    }
    __syncthreads();
    for (int r = wv; r < n_run; r += WG / WAVE) {
        const uint32_t *__restrict__ w = red + V * r * WAVE + lane;
        const int32_t t = S->tile[r][lane];
        if (t < 0 || w[0] == 0u) continue;
        atomicAdd(&R[t], w[0]);
        if (SCORE) {   // the sums of two arms in the halves of one 64-bit word (at most 35 * 2^24 each)
            atomicAdd(&sumT[2 * (int64_t)t], (unsigned long long)w[WAVE] | ((unsigned long long)w[2 * WAVE] << 32));
            atomicAdd(&sumT[2 * (int64_t)t + 1], (unsigned long long)w[3 * WAVE] | ((unsigned long long)w[4 * WAVE] << 32));
        }
    }
}

hipError_t launch_hier4(const Platten &P, uint64_t seed, uint32_t *R, unsigned long long *sumT, float *keys,
                        const int32_t *k, hipStream_t st) {
    if (P.n_h4item == 0) return hipSuccess;
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    const float cut = (float)P.design.cut;
    const uint32_t total = (uint32_t)((P.max_N + GRAN2 - 1) / GRAN2);
    const dim3 grid((uint32_t)((P.n_h4item + WG / WAVE - 1) / (WG / WAVE)));
    const size_t lds = (size_t)(WG / WAVE) * P.h4_max_rows * H4_ROW_LDS * sizeof(uint4);
#define CSE_H4_LAUNCH(M, SC)                                                                                          \
    hipLaunchKernelGGL((k_h4_tiles<M, SC>), grid, dim3(WG), (M) ? lds : lds + (size_t)WG * H4_ROW_LDS * sizeof(uint4), st, P.d_h4set, P.d_h4item, P.n_h4item, P.d_h4rows,     \
                       P.h4_max_rows, P.d_b4tab, wb,                                                                  \
                       we, P.d_h4plane, cut, R, sumT, keys, P.d_h4u, P.d_h4eq, P.d_h4cnt)
#define CSE_H4_SC(M)             \
    if (sumT)                    \
        CSE_H4_LAUNCH(M, true);  \
    else                         \
        CSE_H4_LAUNCH(M, false)
    for (uint32_t wb = 0; wb < total; wb += (uint32_t)P.b4_win) {
        const uint32_t we = std::min<uint32_t>(total, wb + (uint32_t)P.b4_win);
        const uint32_t chunks = (we - wb + 3) / 4;
        const uint32_t per = (uint32_t)((P.n_grp4 + WG / WAVE - 1) / (WG / WAVE));
        const uint32_t split = std::min<uint32_t>(per, std::max<uint32_t>(1u, 2048u / chunks));
        hipLaunchKernelGGL(k_h4_count, dim3(chunks, split), dim3(WG), 0, st, P.d_grp4, P.n_grp4, wb, k0, k1,
                           (uint2 *)P.d_b4tab);
        if (keys && k && wb == 0)
            hipLaunchKernelGGL(k_h4_pilot, dim3((uint32_t)P.n_h4set), dim3(WG), lds, st, P.d_h4set, P.d_h4rows,
                               P.h4_max_rows, P.d_b4tab, P.d_h4plane, k, P.h4_margin, P.d_h4u, P.d_h4eq, P.d_h4fb);
        if (keys) {
            if (k) {
                CSE_H4_SC(true);
            } else {
                CSE_H4_SC(false);
            }
            continue;
        }
        const dim3 rgrid((uint32_t)P.n_h4runitem);
        const size_t rlds = std::max((size_t)(WG / WAVE) * P.h4_run_rows * H4_ROW_LDS * sizeof(uint4),
                                     (size_t)5 * H4_RUN * WAVE * sizeof(uint32_t));
        if (sumT)
            hipLaunchKernelGGL(k_h4_runs<true>, rgrid, dim3(WG), rlds, st, P.d_h4run, P.d_h4runitem, P.d_h4rows,
                               P.h4_run_rows, P.d_b4tab, wb, we, P.d_h4bits, R, sumT);
        else
            hipLaunchKernelGGL(k_h4_runs<false>, rgrid, dim3(WG), rlds, st, P.d_h4run, P.d_h4runitem, P.d_h4rows,
                               P.h4_run_rows, P.d_b4tab, wb, we, P.d_h4bits, R, sumT);
    }
#undef CSE_H4_SC
#undef CSE_H4_LAUNCH
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Plain forward path: one launch per tile (box centre, configuration b), one simulation per
// thread, each thread drawing its own 140 words; the baseline the fused kernel is timed against.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(WG) void k_hier4_plain(uint32_t T0, uint32_t T1, uint32_t T2, uint32_t T3,
                                                    uint32_t bmask, uint32_t n_sims, uint32_t key0,
                                                    uint32_t key1, const float4 *__restrict__ tbl,
                                                    float cut, uint32_t *__restrict__ R_tile) {
    constexpr int NP = NP35;
    constexpr int M1 = NP + 1;
    __shared__ uint32_t s_cnt;
    if (threadIdx.x == 0) s_cnt = 0u;
    __syncthreads();
    const uint32_t k = blockIdx.x * WG + threadIdx.x;
    uint32_t r = 0u;
    if (k < n_sims) {
        int y[4] = {0, 0, 0, 0};
        const uint32_t T[4] = {T0, T1, T2, T3};
#pragma unroll
        for (int b = 0; b < NP; ++b) {   // 4 * 35 words = 35 blocks
            const u32x4 w = philox_block((uint32_t)b, k, key0, key1);
#pragma unroll
            for (int l = 0; l < 4; ++l) {
                const int widx = 4 * b + l;
                const int a = widx / NP;
                y[a] += (u32x4_get(w, l) < T[a]) ? 1 : 0;
            }
        }
        const float4 q = tbl[((y[0] * M1 + y[1]) * M1 + y[2]) * M1 + y[3]];
        float sb = INFINITY;
        if (bmask & 1u) sb = fminf(sb, q.x);
        if (bmask & 2u) sb = fminf(sb, q.y);
        if (bmask & 4u) sb = fminf(sb, q.z);
        if (bmask & 8u) sb = fminf(sb, q.w);   // basket design only (arm 3 is a hypothesis)
        r = (sb < cut) ? 1u : 0u;
    }
    const unsigned long long m = __ballot(r);
    if ((threadIdx.x & (WAVE - 1)) == 0) atomicAdd(&s_cnt, (uint32_t)__popcll(m));
    __syncthreads();
    if (threadIdx.x == 0 && s_cnt) atomicAdd(R_tile, s_cnt);
}

hipError_t launch_hier4_plain(const Platten &P, uint64_t seed, int64_t t, uint32_t *R_tile, hipStream_t st) {
    const uint32_t N = (uint32_t)P.tile_N[t];
    const uint32_t grid = (N + WG - 1) / WG;
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    const uint32_t *T = &P.tile_T[t * 4];
    hipLaunchKernelGGL(k_hier4_plain, dim3(grid), dim3(WG), 0, st, T[0], T[1], T[2], T[3],
                       (uint32_t)P.tile_cfg[t], N, k0, k1, P.d_h4tbl, (float)P.design.cut, R_tile);
    return hipGetLastError();
}

}  // namespace cse
