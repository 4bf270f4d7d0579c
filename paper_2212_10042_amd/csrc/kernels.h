// kernels.h -- launchers of the device kernels (library-internal).
#pragma once
#include "cse_internal.h"

namespace cse {

// counts of every threshold group into the count table (and, when recs is not NULL, the calibration
// workspace), then the per-tile sums
hipError_t launch_binom2(const Platten &P, uint64_t seed, uint32_t *R, unsigned long long *sumT,
                         uint2 *recs, hipStream_t st);
hipError_t launch_ztest1(const Platten &P, uint64_t seed, uint32_t *R, unsigned long long *sumZfx,
                         float *keys, hipStream_t st);
hipError_t launch_plain_tile(const Platten &P, uint64_t seed, int64_t t, uint32_t T0, uint32_t T1,
                             uint32_t *R_tile, hipStream_t st);
hipError_t launch_bound(const Platten &P, int mode, const uint32_t *R, const double *a_in,
                        double level, double *out, double *q_out, int32_t *k_out, double *cp_out,
                        hipStream_t st);
hipError_t launch_select(const Platten &P, const void *keys, const int32_t *k, double *lam, int32_t *rej_at,
                         hipStream_t st);
hipError_t launch_b2_bracket(const Platten &P, const int32_t *k, hipStream_t st);
hipError_t launch_min(const Platten &P, const double *v, const int32_t *in_null, int64_t n, double *out,
                      hipStream_t st);
hipError_t launch_tiebreak(const Platten &P, uint64_t seed, const int32_t *k, const double *lam, int32_t *rej_at,
                           uint32_t *c_tile, hipStream_t st);
hipError_t launch_min_pair(const Platten &P, const double *v, const uint32_t *c, const int32_t *in_null, int64_t n,
                           double *out_v, uint32_t *out_c, hipStream_t st);
hipError_t launch_confset(const Platten &P, const double *s_obs, int64_t s_stride, const double *lam,
                          const double *coef, int link, int32_t *keep, double *e_lo, double *e_hi,
                          double *e_range, hipStream_t st);
hipError_t launch_finish(const Platten &P, const uint32_t *R, const unsigned long long *sumT,
                         const unsigned long long *sumZfx, int32_t *R_out, int64_t *T_out,
                         double *Z_out, double *grad, hipStream_t st);
hipError_t launch_zero(void *p, size_t bytes, hipStream_t st);
hipError_t launch_taylor(const Platten &P, const double *f, const double *g, double *bound, int32_t *vertex,
                         double *point, hipStream_t st);
hipError_t launch_hier4_table(int n, float4 *tbl, const HierNode *nodes, hipStream_t st);
hipError_t launch_basket_table(int n, const double *theta0, float4 *tbl, const HierNode *nodes, hipStream_t st);
hipError_t launch_h4_planes(const float4 *tbl, int nb, float *planes, hipStream_t st);
// counts of every threshold group, then the per-tile sums; keys: NULL, or every float32 key, or (k
// given, after k is known on the stream) the candidate keys of the tiles' k-th smallest
hipError_t launch_h4_bits(const float4 *tbl, float cut, int nb, uint64_t *bits, hipStream_t st);
hipError_t launch_hier4(const Platten &P, uint64_t seed, uint32_t *R, unsigned long long *sumT, float *keys,
                        const int32_t *k, hipStream_t st);
// lambda*_i and the count below it from the candidates (exact; a tile whose k-th key is not among
// them regenerates its keys from the counter-based generator)
hipError_t launch_h4_select(const Platten &P, uint64_t seed, const float *keys, const int32_t *k, double *lam,
                            int32_t *rej_at, hipStream_t st);
hipError_t launch_phase23(const Platten &P, uint64_t seed, uint32_t *R, unsigned long long *sumT, float *keys,
                          hipStream_t st);
hipError_t launch_p23_look1(const Platten &P, hipStream_t st);
// the same over a caller-made item list (device and host copies), which fits the platten's chunks
hipError_t launch_phase23_list(const Platten &P, uint64_t seed, const WorkItem *d_items, const WorkItem *h_items,
                               int64_t n_items, int64_t grid, uint32_t *R, unsigned long long *sumT, float *keys,
                               unsigned long long *stats, hipStream_t st);
hipError_t launch_phase23_tile(const Platten &P, uint64_t seed, int64_t t, uint32_t *R_tile, hipStream_t st);
hipError_t launch_hier4_plain(const Platten &P, uint64_t seed, int64_t t, uint32_t *R_tile, hipStream_t st);

}  // namespace cse
