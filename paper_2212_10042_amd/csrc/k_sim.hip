// k_sim.hip -- Monte Carlo kernels of the z-test and the 2-arm design for gfx950.
//
// A simulation's random words do not depend on the tile (common random numbers, Section 7.3), so
// what depends on the words alone is formed once and shared by every tile: the z-test's normal
// draw, and the 2-arm design's success counts at each distinct threshold.  The per-tile work is
// the decision and its sums: rejection counts R and score sums (sufficient statistic over
// rejections, Example 1).
#include <algorithm>

#include "cse_internal.h"
#include "kernels.h"
#include "philox.hpp"

namespace cse {

// Lanes of one wave exchange values through LDS between these two points.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ------------------------------------------------------------------------------------
// 2-arm binomial, n = 35 per arm, pooled z.  Words 0..34 are arm 0, 35..69 arm 1
// (18 Philox blocks).  Two kernels:
//
// k_b2_count: the success counts of every simulation at every threshold group (8 neighbouring
// distinct thresholds of one arm), once for the whole platten: 16,384 simulations at 2 x 1,024
// thresholds are 1.2e9 word comparisons, where counting per rectangle of tiles repeats them for
// every rectangle (1024 x 1024 boxes: 32-fold).  A workgroup takes one chunk of 64 simulations
// (one per lane): its words go to LDS once, then each wave counts threshold groups and writes them
// to the count table (Grp2: bytes, 16 simulations of a threshold contiguous) and, for a
// calibration, to the workspace the selection reads (8 bytes per simulation and group, and once more
// the counts at the group's first and last threshold, 2 bytes).
//
// k_b2_tiles: per (simulation, tile) the decision y1 >= c(y0) and its sums, four simulations per
// instruction.  A wave takes 8 arm-0 thresholds (wave-uniform, so their counts and cut points are
// scalar loads) against 64 arm-1 thresholds, one per lane, so a lane's 8 tiles keep their sums in
// registers and nothing crosses lanes.  With y1 + 128 and c in the bytes of two words, bit 7 of
// each byte of their difference is the decision (y1 + 128 - c lies in [64, 163]: no borrow);
// masked to those bits it is the weight (128 or 0) of three accumulations: a bit count for R and
// two 4-byte dot products for the sums of y0 and y1: 5 instructions per 4 simulations and tile.
// A quad (4 simulations) that none of the wave's 512 tiles rejects, or that all of them reject, is
// recognised by its extremes and takes none or 9 instructions instead of 40: far from the power
// curve's slope that is nearly every quad.  The sums of y0 and y1 (at most 35 * 2^24 each) go to
// memory as the halves of one 64-bit atomic.
//
// Bound by VALU issue on large grids, by the atomics and load latency on small ones.  1024 x 1024
// boxes x 16,384 simulations: counts 0.08 ms and sums 0.33 ms (0.61 with the 5 instructions for
// every quad: 89% of the VALU issue peak), where one kernel that counted per square of batches and
// decided one simulation at a time took 5.06 ms and wrote 4.3 GB of records for the selection to
// read back; 256 x 256 lower triangle x 8,192: 0.168 -> 0.017 + 0.018 ms.
// ------------------------------------------------------------------------------------
template <bool RECS>
__global__ __launch_bounds__(WG) void k_b2_count(const Grp2 *__restrict__ grp, int32_t n_grp, uint32_t win_b,
                                                 uint32_t win_e, uint32_t key0, uint32_t key1,
                                                 const int32_t *__restrict__ cut_tbl, uint2 *__restrict__ tab,
                                                 uint2 *__restrict__ recs, uint16_t *__restrict__ ext) {
    constexpr int NB = (2 * NP35 + 3) / 4;
    constexpr int NWV = WG / WAVE;
    __shared__ uint32_t words[4 * NB][WAVE];
    __shared__ uint8_t s_cut[WAVE];
    __shared__ uint2 tr[NWV][WAVE];
    const int lane = threadIdx.x & (WAVE - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t k0 = win_b * GRAN2 + blockIdx.x * WAVE;
    const uint32_t k = k0 + (uint32_t)lane;
    if (threadIdx.x < WAVE) s_cut[threadIdx.x] = threadIdx.x <= NP35 ? (uint8_t)cut_tbl[threadIdx.x] : (uint8_t)64;
    for (int b = wv; b < NB; b += NWV) {
        const u32x4 w = philox_block((uint32_t)b, k, key0, key1);
        words[4 * b + 0][lane] = w.x;
        words[4 * b + 1][lane] = w.y;
        words[4 * b + 2][lane] = w.z;
        words[4 * b + 3][lane] = w.w;
    }
    __syncthreads();
    for (int g = (int)blockIdx.y * NWV + wv; g < n_grp; g += (int)gridDim.y * NWV) {   // uniform over the wave
        const Grp2 *__restrict__ G = grp + g;
        const uint32_t n = (uint32_t)G->n_sims;
        if (k0 >= n) continue;
        const int arm = G->arm;
        uint32_t T[B2U], y[B2U];
#pragma unroll
        for (int u = 0; u < B2U; ++u) {
            T[u] = G->T[u];
            y[u] = 0u;
        }
        const uint32_t(*w)[WAVE] = words + arm * NP35;
#pragma unroll 7
        for (int j = 0; j < NP35; ++j) {
            const uint32_t x = w[j][lane];
#pragma unroll
            for (int u = 0; u < B2U; ++u) y[u] += (x < T[u]) ? 1u : 0u;
        }
        const uint2 c8 = make_uint2(y[0] | (y[1] << 8) | (y[2] << 16) | (y[3] << 24),
                                    y[4] | (y[5] << 8) | (y[6] << 16) | (y[7] << 24));
        if (RECS) {   // chunks are padded: past n_sims too
            recs[G->rec + k] = c8;
            ext[G->rec + k] = (uint16_t)(y[0] | (y[B2U - 1] << 8));
        }
        // (simulation, threshold) bytes -> threshold-major granules: lane = granule q of the chunk,
        // threshold t, half h of its 16 simulations
        tr[wv][lane] = c8;
        wave_sync();
        const int q = lane >> 4, t = (lane >> 1) & 7, h = lane & 1;
        const uint8_t *src = reinterpret_cast<const uint8_t *>(&tr[wv][16 * q + 8 * h]) + t;
        uint32_t b[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) b[i] = src[8 * i];
        wave_sync();
        const uint32_t kq = k0 + (uint32_t)(16 * q);   // the granule's first simulation
        if (kq >= n) continue;
        const int64_t gi = (int64_t)(kq / GRAN2 - win_b);
        uint2 *__restrict__ dst = tab + (G->unit + gi * (arm ? 1 : 2)) * (UNIT2 / 8) + 2 * t + h;
        const uint2 v = make_uint2(b[0] | (b[1] << 8) | (b[2] << 16) | (b[3] << 24),
                                   b[4] | (b[5] << 8) | (b[6] << 16) | (b[7] << 24));
        if (arm) {
            dst[0] = make_uint2(v.x | 0x80808080u, v.y | 0x80808080u);
        } else {
            dst[0] = v;
            uint32_t c[8];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                c[i] = kq + (uint32_t)(8 * h + i) < n ? (uint32_t)s_cut[b[i]] : 64u;
            dst[UNIT2 / 8] = make_uint2(c[0] | (c[1] << 8) | (c[2] << 16) | (c[3] << 24),
                                        c[4] | (c[5] << 8) | (c[6] << 16) | (c[7] << 24));
        }
    }
}

__global__ __launch_bounds__(WG) void k_b2_tiles(const Blk2 *__restrict__ blocks, const SquareItem *__restrict__ items,
                                                 const Grp2 *__restrict__ grp, const uint4 *__restrict__ tab,
                                                 uint32_t win_b, uint32_t win_e, uint32_t *__restrict__ R,
                                                 unsigned long long *__restrict__ sumT) {
    static_assert(SQ2R == WG / WAVE && SQ2C * B2V == WAVE, "one wave per row group, one lane per arm-1 threshold");
    constexpr uint32_t H = 0x80808080u;
    constexpr int U4 = UNIT2 / 16;   // uint4 per unit
    const int lane = threadIdx.x & (WAVE - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const SquareItem *__restrict__ I = items + blockIdx.x;
    const int32_t rg = I->rg[wv];
    const uint32_t gb = max(I->g_begin, win_b), ge = min(I->g_end, win_e);
    if (rg < 0 || gb >= ge) return;
    const int32_t blk = I->blk[wv][lane >> 3];
    const uint4 *__restrict__ pa = tab + (grp[rg].unit + 2 * (int64_t)(gb - win_b)) * U4;
    const uint4 *__restrict__ pb = tab + (grp[I->cg[lane >> 3]].unit + (int64_t)(gb - win_b)) * U4 + (lane & 7);
    uint32_t aR[B2U], a0[B2U], a1[B2U];
#pragma unroll
    for (int u = 0; u < B2U; ++u) aR[u] = a0[u] = a1[u] = 0u;
    // simulations of the quads that every tile rejects, and their sums
    uint32_t all = 0u, a1all = 0u, a0all[B2U];
#pragma unroll
    for (int u = 0; u < B2U; ++u) a0all[u] = 0u;
    uint32_t h = H;
    asm("" : "+v"(h));   // the weight in a vector register, beside a scalar operand
    for (uint32_t g = gb; g < ge; ++g, pa += 2 * U4, pb += U4) {
        const uint4 y1 = *pb;
        uint4 y0[B2U], c0[B2U];
#pragma unroll
        for (int u = 0; u < B2U; ++u) {
            y0[u] = pa[u];
            c0[u] = pa[U4 + u];
        }
        // the granule's scalar loads issued together, ahead of the branches (not one by one inside)
#pragma unroll
        for (int u = 0; u < B2U; ++u)
            asm volatile("" ::"s"(y0[u].x), "s"(y0[u].y), "s"(y0[u].z), "s"(y0[u].w), "s"(c0[u].x), "s"(c0[u].y),
                         "s"(c0[u].z), "s"(c0[u].w));
        auto quad = [&](uint32_t v, auto part) {
            // counts and cut points ascend with the threshold: lane 63 has the largest y1, row 0 the
            // smallest c, and the other way round
            const uint32_t hi = (__builtin_amdgcn_readlane(v, WAVE - 1) - part(c0[0])) & H;
            const uint32_t lo = (__builtin_amdgcn_readlane(v, 0) - part(c0[B2U - 1])) & H;
            if (hi != 0u && lo != H) {
#pragma unroll
                for (int u = 0; u < B2U; ++u) {
                    const uint32_t m = (v - part(c0[u])) & H;
                    aR[u] += (uint32_t)__popc(m);
                    a0[u] = __builtin_amdgcn_udot4(m, part(y0[u]), a0[u], false);
                    a1[u] = __builtin_amdgcn_udot4(m, v, a1[u], false);
                }
            }
            if (lo == H) {
                all += 4u;
                a1all = __builtin_amdgcn_udot4(v, H, a1all, false);
#pragma unroll
                for (int u = 0; u < B2U; ++u) a0all[u] = __builtin_amdgcn_udot4(h, part(y0[u]), a0all[u], false);
            }
        };
        quad(y1.x, [](const uint4 &q) { return q.x; });
        quad(y1.y, [](const uint4 &q) { return q.y; });
        quad(y1.z, [](const uint4 &q) { return q.z; });
        quad(y1.w, [](const uint4 &q) { return q.w; });
    }
    if (blk < 0) return;
#pragma unroll
    for (int u = 0; u < B2U; ++u) {
        const int32_t t = blocks[blk].tile[u * B2V + (lane & 7)];
        const uint32_t r = aR[u] + all;
        if (t >= 0 && r) {
            atomicAdd(&R[t], r);
            const uint32_t s0 = (a0[u] + a0all[u]) >> 7, s1 = ((a1[u] + a1all) >> 7) - 128u * r;
            atomicAdd(&sumT[t], (unsigned long long)s0 | ((unsigned long long)s1 << 32));
        }
    }
}


// ------------------------------------------------------------------------------------
// z-test: X = theta + Z, Z from words 0 and 1 by Box-Muller in float32,
// u = ((word >> 9) + 1/2) 2^-23.  Reject X > cut; score term X - theta = Z; key S = -X.
// Score sums are carried in 64-bit fixed point (2^-32) so the cross-wave sum is exact.
// ------------------------------------------------------------------------------------
__device__ __forceinline__ float unit23(uint32_t w) {
    return ((float)(w >> 9) + 0.5f) * (1.0f / 8388608.0f);
}

template <bool KEYS>
__global__ __launch_bounds__(WG) void k_ztest1(const Blk1 *__restrict__ blocks,
                                               const WorkItem *__restrict__ items, int64_t n_items,
                                               uint32_t key0, uint32_t key1, float cut,
                                               uint32_t *__restrict__ R,
                                               unsigned long long *__restrict__ sumZfx,
                                               float *__restrict__ keys) {
    constexpr int NT = B1T;
    __shared__ uint32_t xbuf[WG / WAVE][NT][WAVE + 1];
    const int lane = threadIdx.x & (WAVE - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t it = (int64_t)blockIdx.x * (WG / WAVE) + wv;
    if (it >= n_items) return;
    const WorkItem W = items[it];
    const Blk1 *__restrict__ B = blocks + W.blk;
    const uint32_t n_sims = (uint32_t)B->n_sims;
    const int64_t key_base = B->key_base;

    uint32_t accR[NT];
    float accZ[NT];
#pragma unroll
    for (int s = 0; s < NT; ++s) {
        accR[s] = 0u;
        accZ[s] = 0.0f;
    }
    uint32_t totR = 0u;
    long long totZ = 0;

    auto flush = [&]() {
#pragma unroll
        for (int s = 0; s < NT; ++s) xbuf[wv][s][lane] = accR[s];
        wave_sync();
        for (int l = 0; l < WAVE; ++l) totR += xbuf[wv][lane][l];
        wave_sync();
#pragma unroll
        for (int s = 0; s < NT; ++s) xbuf[wv][s][lane] = __float_as_uint(accZ[s]);
        wave_sync();
        for (int l = 0; l < WAVE; ++l)
            totZ += (long long)__double2ll_rn((double)__uint_as_float(xbuf[wv][lane][l]) * 4294967296.0);
        wave_sync();
#pragma unroll
        for (int s = 0; s < NT; ++s) {
            accR[s] = 0u;
            accZ[s] = 0.0f;
        }
    };

    int since = 0;
    for (uint32_t k0 = W.k_begin; k0 < W.k_end; k0 += WAVE) {
        const uint32_t k = k0 + (uint32_t)lane;
        const bool act = k < W.k_end;
        const u32x4 w = philox_block(0u, k, key0, key1);
        const float u0 = unit23(w.x), u1 = unit23(w.y);
        const float Z = sqrtf(-2.0f * logf(u0)) * cospif(2.0f * u1);
#pragma unroll
        for (int s = 0; s < NT; ++s) {
            const float X = B->theta[s] + Z;
            const bool r = act && (X > cut);
            accR[s] += r ? 1u : 0u;
            accZ[s] += r ? Z : 0.0f;
            if (KEYS && act && B->tile[s] >= 0) keys[key_base + (int64_t)s * n_sims + k] = -X;
        }
        if (++since == 16) {
            flush();
            since = 0;
        }
    }
    flush();
    const int32_t tile = B->tile[lane];
    if (tile >= 0) {
        atomicAdd(&R[tile], totR);
        atomicAdd(&sumZfx[tile], (unsigned long long)totZ);
    }
}

// ------------------------------------------------------------------------------------
// The plain forward-only path: one launch per tile, one simulation per thread, the tile's
// own thresholds, no sharing across tiles, rejection count only.
// ------------------------------------------------------------------------------------
__global__ __launch_bounds__(WG) void k_binom2_plain(uint32_t T0, uint32_t T1, uint32_t n_sims,
                                                     uint32_t key0, uint32_t key1,
                                                     const int32_t *__restrict__ cut_tbl,
                                                     uint32_t *__restrict__ R_tile) {
    constexpr int NW = 2 * NP35;
    constexpr int NB = (NW + 3) / 4;
    __shared__ uint32_t s_cnt;
    if (threadIdx.x == 0) s_cnt = 0u;
    __syncthreads();
    const uint32_t k = blockIdx.x * WG + threadIdx.x;
    uint32_t r = 0u;
    if (k < n_sims) {
        int y0 = 0, y1 = 0;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const u32x4 w = philox_block((uint32_t)b, k, key0, key1);
#pragma unroll
            for (int l = 0; l < 4; ++l) {
                const int widx = 4 * b + l;
                const uint32_t x = u32x4_get(w, l);
                if (widx < NP35)
                    y0 += (x < T0) ? 1 : 0;
                else if (widx < NW)
                    y1 += (x < T1) ? 1 : 0;
            }
        }
        r = (y1 >= cut_tbl[y0]) ? 1u : 0u;
    }
    const unsigned long long m = __ballot(r);
    if ((threadIdx.x & (WAVE - 1)) == 0) atomicAdd(&s_cnt, (uint32_t)__popcll(m));
    __syncthreads();
    if (threadIdx.x == 0 && s_cnt) atomicAdd(R_tile, s_cnt);
}

__global__ __launch_bounds__(WG) void k_ztest1_plain(float theta, float cut, uint32_t n_sims,
                                                     uint32_t key0, uint32_t key1,
                                                     uint32_t *__restrict__ R_tile) {
    __shared__ uint32_t s_cnt;
    if (threadIdx.x == 0) s_cnt = 0u;
    __syncthreads();
    const uint32_t k = blockIdx.x * WG + threadIdx.x;
    uint32_t r = 0u;
    if (k < n_sims) {
        const u32x4 w = philox_block(0u, k, key0, key1);
        const float Z = sqrtf(-2.0f * logf(unit23(w.x))) * cospif(2.0f * unit23(w.y));
        r = (theta + Z > cut) ? 1u : 0u;
    }
    const unsigned long long m = __ballot(r);
    if ((threadIdx.x & (WAVE - 1)) == 0) atomicAdd(&s_cnt, (uint32_t)__popcll(m));
    __syncthreads();
    if (threadIdx.x == 0 && s_cnt) atomicAdd(R_tile, s_cnt);
}

// ------------------------------------------------------------------------------ launchers
hipError_t launch_binom2(const Platten &P, uint64_t seed, uint32_t *R, unsigned long long *sumT,
                         uint2 *recs, hipStream_t st) {
    if (P.n_gitems <= 0) return hipSuccess;
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    const uint32_t total = (uint32_t)((P.max_N + GRAN2 - 1) / GRAN2);
    for (uint32_t wb = 0; wb < total; wb += (uint32_t)P.b2_win) {
        const uint32_t we = std::min<uint32_t>(total, wb + (uint32_t)P.b2_win);
        // counting: enough workgroups to fill the chip, each chunk's words drawn once per workgroup
        const uint32_t chunks = (we - wb + 3) / 4;
        const uint32_t per = (uint32_t)((P.n_grp2 + WG / WAVE - 1) / (WG / WAVE));
        const uint32_t split = std::min<uint32_t>(per, std::max<uint32_t>(1u, 4096u / chunks));
        if (recs)
            hipLaunchKernelGGL(k_b2_count<true>, dim3(chunks, split), dim3(WG), 0, st, P.d_grp2, P.n_grp2, wb, we, k0,
                               k1, P.d_cut_tbl, (uint2 *)P.d_b2tab, recs, (uint16_t *)(recs ? recs + P.b2_recs : nullptr));
        else
            hipLaunchKernelGGL(k_b2_count<false>, dim3(chunks, split), dim3(WG), 0, st, P.d_grp2, P.n_grp2, wb, we, k0,
                               k1, P.d_cut_tbl, (uint2 *)P.d_b2tab, recs, (uint16_t *)(recs ? recs + P.b2_recs : nullptr));
        hipLaunchKernelGGL(k_b2_tiles, dim3((uint32_t)P.n_gitems), dim3(WG), 0, st, (const Blk2 *)P.d_blocks,
                           P.d_sqitems, P.d_grp2, P.d_b2tab, wb, we, R, sumT);
    }
    return hipGetLastError();
}

hipError_t launch_ztest1(const Platten &P, uint64_t seed, uint32_t *R, unsigned long long *sumZfx,
                         float *keys, hipStream_t st) {
    const int64_t grid = (P.n_items + (WG / WAVE) - 1) / (WG / WAVE);
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    const float cut = (float)P.design.cut;
    if (keys)
        hipLaunchKernelGGL(k_ztest1<true>, dim3((uint32_t)grid), dim3(WG), 0, st,
                           (const Blk1 *)P.d_blocks, P.d_items, P.n_items, k0, k1, cut, R, sumZfx,
                           keys);
    else
        hipLaunchKernelGGL(k_ztest1<false>, dim3((uint32_t)grid), dim3(WG), 0, st,
                           (const Blk1 *)P.d_blocks, P.d_items, P.n_items, k0, k1, cut, R, sumZfx,
                           keys);
    return hipGetLastError();
}

hipError_t launch_plain_tile(const Platten &P, uint64_t seed, int64_t t, uint32_t T0, uint32_t T1,
                             uint32_t *R_tile, hipStream_t st) {
    const uint32_t N = (uint32_t)P.tile_N[t];
    const uint32_t grid = (N + WG - 1) / WG;
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    if (P.design.kind == CSE_ZTEST1)
        hipLaunchKernelGGL(k_ztest1_plain, dim3(grid), dim3(WG), 0, st, (float)P.tile_theta[t],
                           (float)P.design.cut, N, k0, k1, R_tile);
    else
        hipLaunchKernelGGL(k_binom2_plain, dim3(grid), dim3(WG), 0, st, T0, T1, N, k0, k1,
                           P.d_cut_tbl, R_tile);
    return hipGetLastError();
}

}  // namespace cse
