// cse_internal.h -- data structures shared by the files of libcse.so (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <memory>
#include <string>
#include <vector>

#include "cse.h"

namespace cse {

constexpr int WAVE = 64;
constexpr int WG = 256;              // 4 waves per workgroup
constexpr int MAX_D = 4;
constexpr int NP35 = 35;             // patients per arm of the binomial designs
constexpr int P23_NMAX_ARM = 350;    // embedded patients per arm of the Phase II/III design
constexpr uint64_t PLATTEN_GONE = ~0ull;   // shape generation of a destroyed platten
constexpr int MIN_PARTS = 256;            // partial minima of the large min reductions

// ---- tile batches ("blocks"): each wave owns one block for a range of simulations ----
// 2-arm designs: an 8 x 8 product of distinct arm-0 and arm-1 thresholds, so one
// simulation's success counts at 16 thresholds serve 64 tiles (common random numbers).
constexpr int B2U = 8, B2V = 8;
struct Blk2 {
    uint32_t T0[B2U];          // arm-0 Bernoulli thresholds (uint32, see platten.cpp)
    uint32_t T1[B2V];          // arm-1 thresholds
    int32_t tile[B2U * B2V];   // tile id of slot (u, v) = u * B2V + v, or -1
    int32_t n_sims;            // simulations of every tile of this block
    int32_t pad;
    int64_t rec0, rec1;        // calibration counts: simulation k's arm-0 counts at the block's 8
                               // thresholds are the bytes of entry rec0 + k, its arm-1 counts those
                               // of rec1 + k (Grp2's rec of its two threshold groups)
};
// Threshold group of a 2-arm platten: 8 neighbouring distinct thresholds of one arm, counted once
// per simulation for every block that has them (one row or column of the 8 x 8 grid of blocks of
// one simulation count).
//  * unit: first 128-byte unit of the group in the count table.  A granule (16 simulations) takes
//    one unit for arm 1, the counts y1 + 128 as bytes, threshold-major ([8][16]), and two units for
//    arm 0, the counts y0 and then the design's cut points c(y0) (64, no rejection, past n_sims).
//  * rec: first entry (8 bytes: one simulation's counts at the 8 thresholds) in the calibration
//    workspace, simulations padded to whole chunks of 64.
struct Grp2 {
    uint32_t T[B2U];
    int32_t arm;
    int32_t n_sims;
    int64_t unit;
    int64_t rec;
};
constexpr int GRAN2 = 16;              // simulations per granule of the count table
constexpr int UNIT2 = B2U * GRAN2;     // bytes per unit
constexpr int64_t B2_TABLE_MAX = (int64_t)128 << 20;   // count-table bytes (more: simulation windows)
constexpr int REC2_BYTES = 16;   // calibration workspace as documented: bytes per (simulation, batch)
// calibration workspace: all groups' 8-byte entries, then once more each entry's first and last
// count as 2 bytes (the selection's first pass reads only those)
constexpr int B2_REC_BYTES = 8 + 2;

// z-test: 64 tiles share each simulation's normal draw.
constexpr int B1T = 64;
struct Blk1 {
    float theta[B1T];
    int32_t tile[B1T];
    int32_t n_sims;
    int32_t pad;
    int64_t key_base;          // keys of slot s live at key_base + s * n_sims + k
};

// 4-arm designs.  Threshold group: up to 8 neighbouring distinct thresholds of one arm among the tiles
// of one simulation count, counted once per simulation for all of them.  Threshold t has a row of
// the count table, one 16-byte unit per granule (16 simulations, one byte each), at row + t *
// stride; arms 2 and 3 have a second row, 8 * stride further on, with the counts' codes for the
// statistic's table (h4_code2, h4_code3).
struct Grp4 {
    uint32_t T[8];
    int32_t arm;
    int32_t n_sims;
    int32_t n_thr;
    int32_t pad;
    int64_t row;      // units
    int64_t stride;   // units: granules of a window
};
// A wave's 64 tiles, one per lane (lanes past n_lanes repeat lane 0's rows and have no tile).  The
// distinct count-table rows of the set are listed from row_at on; a lane's four count rows and two
// code rows (arms 2 and 3) are places in that list.
constexpr int H4_ROWS = 6;
constexpr int H4_SET_ROWS = 368;   // distinct rows of a set at most: four waves' rows beside the pilot's histogram in LDS
struct H4Set {
    int32_t tile[64];
    uint16_t row[H4_ROWS][64];
    uint32_t cfg[64];       // null configuration b
    int32_t n_sims;
    int32_t n_lanes;
    int32_t slice;          // granules per item
    int32_t n_slices;
    int32_t n_rows;
    int32_t pad;
    int64_t row_at;
    int64_t key_base;       // key of lane l, simulation k at key_base + (k / 64) * 64 n_lanes + 64 l + k % 64
    int64_t cnt_base;       // candidates kept by lane l in slice s: entry cnt_base + 64 s + l
};
constexpr int H4_ROW_LDS = 5;   // 16-byte units of a staged row: a chunk's four and one of padding (no bank conflicts)
// Wave item: the granules [g_begin, g_end) of a set (its slice `slice`).
struct H4Item {
    int32_t set;
    int32_t slice;
    uint32_t g_begin;
    uint32_t g_end;
};
// Runs of tiles that differ only in arm 3's threshold (and are of one configuration): up to H4_RUN
// tiles per lane, 64 runs to a set.  row: places of the count rows of arms 0, 1 and 2 and of each tile's
// arm 3 in the set's list.
constexpr int H4_RUN = 8;
constexpr int64_t H4_BITS = (int64_t)(NP35 + 1) * (NP35 + 1) * (NP35 + 1);
struct H4Run {
    int32_t tile[H4_RUN][64];
    uint16_t row[3 + H4_RUN][64];
    uint32_t cfg[64];
    int32_t n_sims;
    int32_t n_run;          // tiles of the longest run
    int32_t n_rows;
    int32_t pad;
    int64_t row_at;
};
// Table of the statistic S_b of each configuration b, one plane per b: outcome (y0, y1, y2, y3) at
// ((36 y0 + y1) * H4_SLAB + 8 code2(y2) + code3(y3)), so that 4 x 8 neighbouring (y2, y3) share a
// 128-byte line.
constexpr int H4_SLAB = 9 * 5 * 32;
constexpr int64_t H4_PLANE = (int64_t)(NP35 + 1) * (NP35 + 1) * H4_SLAB;   // floats
__host__ __device__ inline uint32_t h4_code2(uint32_t y) { return 20u * (y >> 2) + (y & 3u); }
__host__ __device__ inline uint32_t h4_code3(uint32_t y) { return ((y >> 3) << 5) + (y & 7u); }
// Calibration of the 4-arm designs from candidate keys: a pilot over the first h4_pilot(N)
// simulations of a set gives each tile an upper bound of its k-th smallest key; the pass over all
// simulations keeps only the keys below it.
constexpr int64_t H4_SLICE_MAX = 256;    // granules per item at most (4,096 simulations)
constexpr int64_t H4_TABLE_MAX = (int64_t)4 << 30;   // count-table bytes of windows of H4_SLICE_MAX granules (more: shorter ones)
constexpr int64_t H4_WGS = 2048;         // workgroups of four waves, default
constexpr int H4_PILOT_MIN_N = 1024;     // fewer simulations: every key is kept
constexpr int H4_PILOT_MAX = 2048;
constexpr int H4_CAND_MAX = 3072;        // candidates a wave selects in LDS (more: the workgroup)
constexpr int64_t H4_CAND_KEYS = (int64_t)64 << 20;   // keys of the platten from which candidates are kept
constexpr double H4_CAND_ALPHA = 0.05;   // and largest alpha: the rank stays below a fifth of every pilot
// candidate slots of a tile per slice of `slice` granules (a pilot leaves an eighth of the keys at most;
// a set's slots fit its keys' place in the workspace)
__host__ __device__ inline int h4_cap(int n, int slice) { return n < H4_PILOT_MIN_N ? slice * GRAN2 : slice * GRAN2 / 2; }
__host__ __device__ inline int h4_pilot(int n) {   // a multiple of 64
    const int m = n / 16 / 64 * 64;
    return m < 256 ? 256 : (m > H4_PILOT_MAX ? H4_PILOT_MAX : m);
}

// Work item: one wave simulates sims [k_begin, k_end) of block blk.
struct WorkItem {
    int32_t blk;
    uint32_t k_begin;
    uint32_t k_end;
    int32_t pad;
};

// Workgroup item of the 2-arm kernel: wave w takes the 8 thresholds of row group rg[w] (-1: none)
// against the up to 64 thresholds of the column groups cg[0..7] (ascending; the first ncg are
// valid) over the granules [g_begin, g_end); blk[w][c] is the batch of (rg[w], cg[c]), or -1.
constexpr int SQ2R = 4, SQ2C = 8;
struct SquareItem {
    int32_t rg[SQ2R];
    int32_t cg[SQ2C];
    int32_t blk[SQ2R][SQ2C];
    int32_t ncg;
    uint32_t g_begin;
    uint32_t g_end;
    int32_t pad;
};

// Per-node constants of the hierarchical posterior (90 nodes equally spaced in log s2 on
// [log 1e-6, log 1e3]), computed once on the host: log s2, s2, 1/s2, c = 100 / (s2 + 400),
// beta = c / s2, and lconst = log|Q|/2 + log of the inverse-gamma density of s2 + log of the
// trapezoid weight in log s2 times s2.
constexpr int HIER_NODES = 90;
struct HierNode {
    double ls2, s2, inv_s2, c, beta, lconst;
};

// Arguments of the Phase II/III kernel (device pointers owned by the platten, except the
// outputs filled in per launch).
struct P23Args {
    const WorkItem *items;          // (tile in blk, simulation range) queue entries
    int64_t n_items;
    uint32_t *counter;              // queue head, zeroed before each launch
    const uint32_t *tileT;          // [n_tiles][4] Bernoulli thresholds
    const int32_t *cfg;             // [n_tiles] null configuration b
    const int64_t *key_off;         // [n_tiles] first key of the tile (keys contiguous per tile)
    uint32_t key0, key1;            // Philox key (seed)
    float cut;                      // lambda of the final analysis (the design's fixed rule)
    int32_t pad;
    uint32_t *R;                    // [n_tiles] rejections at cut
    unsigned long long *sumT;       // [n_tiles][8] sums of observed y_a, then n_a, over rejections
    float *keys;                    // calibration keys S or NULL
    unsigned long long *stats;      // NULL or [4]: trials, Phase II / Phase III posterior looks, Newton steps
    const double *gh;               // Gauss-Hermite rule (weight e^{-x^2}): nodes [16], weights [16]
    const HierNode *nodes;          // per-node constants of the hierarchical posterior [90]
    const uint8_t *look1;           // decision code of the first look per outcome, 51^4 entries
    const uint16_t *counts;         // count table, or NULL: trials draw their own words
    const uint2 *tile_row;          // [n_tiles][4] (at, stride) of the tile's four rows
    double sqrt_pi, z95;            // sqrt(pi), Phi^{-1}(0.95)
};

// Phase II/III design, count table: the successes among the first n words of an arm's stream, for
// every distinct threshold of the arm and every sample size n a trial can reach (P23_SIZES: nine
// sizes of Phase II, and those with 100 and 200 patients of Phase III added), u16, simulations
// contiguous.  Row r starts at at * 64, size column c of simulation k at (at + c * stride) * 64 + k.
constexpr int P23_NSIZE = 9, P23_SIZES = 3 * P23_NSIZE;
constexpr int64_t P23_TABLE_MAX = (int64_t)1 << 30;   // bytes (more: every trial draws its own words)
struct P23Row {
    uint32_t T;
    int32_t arm;
    uint32_t at;       // units of 64 entries
    uint32_t stride;   // chunks of 64 simulations of the row
};

// Phase II/III design, states already evaluated in the call and the open trials (k_p23_*): slots of
// 64-bit states and their outcomes, the states without a place in the table, the new states of a
// round by phase, the open trials' records (two uint4 each, rounds alternate; workgroup b's are
// range[b].y from range[b].x on) and counters: per round {new Phase II states, new Phase III states,
// states without a place}, then the trials.  Each counter has a cache line of its own.
constexpr int P23_WAVES = 2;                          // waves per SIMD of the posterior kernel
constexpr int64_t P23_GRID = 256 * P23_WAVES;          // and its workgroups
constexpr int P23_ROUNDS = 5;                          // looks after the first, and the end
constexpr int64_t P23_BLOCKS = 8192;                  // workgroups of k_p23_open and k_p23_step, at most
constexpr int P23_CTR = 32, P23_COUNTERS = 3 * P23_ROUNDS + 1;
constexpr int64_t P23_CAP_MAX = (int64_t)32 << 20;     // trials of a chunk
constexpr int64_t P23_CAP_MIN = 512, P23_SLOTS_MIN = 4096;   // an item's trials at least
struct P23Memo {
    unsigned long long *state;
    uint32_t *value;
    uint64_t *own;
    uint32_t *list[2];
    uint4 *trial[2];
    uint2 *range;
    uint32_t *ctr;
    uint32_t mask;
    uint32_t pad;
    __host__ __device__ uint32_t *count(int round, int j) const { return ctr + (3 * round + j) * P23_CTR; }
    __host__ __device__ uint32_t *trials() const { return ctr + 3 * P23_ROUNDS * P23_CTR; }
};

// Family of the data model for the bound (Example 1 / Section 4.2).
enum Family : int32_t { FAM_NORMAL = 1, FAM_BINOM = 2 };

struct Platten {
    cse_design design{};
    int d = 0;              // parameter dimension
    int p = 0;              // number of null hypotheses
    int32_t family = 0;
    int32_t n_per_arm = 0;
    int64_t n_boxes = 0, n_tiles = 0;
    int device = -1;

    // host copies
    std::vector<int64_t> tile_box;
    std::vector<int32_t> tile_cfg, tile_nv, tile_in_null, tile_N;
    std::vector<double> tile_theta;      // [n_tiles * d]
    std::vector<int32_t> vert_off;       // [n_tiles + 1]
    std::vector<double> verts;           // [total vertices * d] displacements from theta
    std::vector<double> tile_radii;      // [n_tiles * d]
    std::vector<int32_t> tile_is_box;    // [n_tiles]
    int32_t max_N = 0;
    int64_t total_sims = 0;              // sum of N over tiles
    int64_t block_sims = 0;              // sum over batches of their N
    int64_t group_sims = 0;              // sum over workgroup items of their simulation count

    // device copies (owned)
    double *d_theta = nullptr;
    int32_t *d_N = nullptr;
    int32_t *d_vert_off = nullptr;
    double *d_verts = nullptr;
    double *d_radii = nullptr;           // [n_tiles * d] half-widths of the tile's box
    int32_t *d_is_box = nullptr;         // [n_tiles] 1 when the tile is its whole box
    std::vector<int32_t> border;         // tiles in the order of the bound's search (empty: as they are)
    int32_t *d_border = nullptr;
    int32_t *d_in_null = nullptr;        // [n_tiles] 1 when the tile lies in the null space
    int64_t *d_key_off = nullptr;        // [n_tiles] each tile's first key in d_keys
    int64_t *d_key_stride = nullptr;     // [n_tiles] distance between its 64-simulation chunks
    int64_t n_keys = 0;                  // key slots (sum over blocks of 64 * n_sims)
    void *d_blocks = nullptr;
    int64_t n_blocks = 0;
    WorkItem *d_items = nullptr;
    int64_t n_items = 0;
    SquareItem *d_sqitems = nullptr;     // 2-arm design
    Grp2 *d_grp2 = nullptr;              // 2-arm design: threshold groups
    int32_t n_grp2 = 0;
    int64_t b2_units = 0;                // count table: 128-byte units
    int64_t b2_recs = 0;                 // calibration workspace: 8-byte entries
    uint4 *d_b2tab = nullptr;            // count table (one window of b2_win granules)
    int64_t b2_win = 0;                  // granules of a window (a multiple of 4)
    int64_t n_gitems = 0;
    // 4-arm designs: threshold groups, tile sets, wave items, count table (one window of b4_win
    // granules); calibration from candidates: per tile the upper bound of the k-th key and the
    // keys equal to it, the candidates kept per slice, the tile's place (set * 64 + lane) and the number of tiles the
    // last selection regenerated
    Grp4 *d_grp4 = nullptr;
    int32_t n_grp4 = 0;
    H4Set *d_h4set = nullptr;
    H4Item *d_h4item = nullptr;
    int64_t n_h4set = 0, n_h4item = 0;
    std::vector<H4Set> h4set;            // host copy (launch shapes)
    int64_t b4_units = 0, b4_win = 0;
    uint32_t *d_h4rows = nullptr;        // the sets' row lists
    int32_t h4_max_rows = 0;             // longest of them
    size_t table_bytes = 0;              // of d_b2tab or d_b4tab
    uint4 *d_b4tab = nullptr;
    float *d_h4u = nullptr;
    uint32_t *d_h4eq = nullptr;
    uint32_t *d_h4cnt = nullptr;
    int32_t *d_h4at = nullptr;
    uint32_t *d_h4fb = nullptr;
    bool h4_candidates = false;          // candidates at any size
    float h4_margin = 6.0f;              // pilot margin in standard deviations of the rank

    // design tables (device)
    float4 *d_h4tbl = nullptr;           // 4-arm: (1 - P_1, 1 - P_2, 1 - P_3, 0) per outcome
    std::vector<H4Run> h4run;            // runs of tiles along arm 3
    H4Run *d_h4run = nullptr;
    H4Item *d_h4runitem = nullptr;
    int64_t n_h4runitem = 0;
    int32_t h4_run_rows = 0;             // rows of the longest list of a set of runs
    uint64_t *d_h4bits = nullptr;        // rejecting y3 (bits) per (b, y0, y1, y2)
    float *d_h4plane = nullptr;          // 4-arm designs: S_b per outcome, one plane per configuration
    HierNode *d_hnodes = nullptr;        // per-node constants of the hierarchical posterior
    // Phase II/III design: per-tile thresholds / configurations, the work queue
    uint32_t *d_tileT = nullptr;
    int32_t *d_cfg = nullptr;
    uint32_t *d_queue = nullptr;
    double *d_gh = nullptr;              // Gauss-Hermite nodes and weights
    unsigned long long *d_p23stats = nullptr;   // [4] work counters of the last launch
    uint8_t *d_p23look1 = nullptr;       // first-look decisions (51^4)
    WorkItem *d_p23items = nullptr;
    P23Args p23{};
    int64_t p23_grid = 0;
    P23Memo p23memo{};
    int64_t p23_cap = 0;                 // trials the records hold
    void *d_p23mem = nullptr;            // all of p23memo's memory
    std::vector<WorkItem> p23_items;     // host copy of the items
    P23Row *d_p23row = nullptr;          // count table: rows (by arm), their place per tile, the table
    int32_t n_p23row = 0, p23_arm_row[5] = {0, 0, 0, 0, 0};
    int64_t p23_chunks = 0;              // chunks of 64 simulations of the longest row
    uint2 *d_p23tilerow = nullptr;
    uint16_t *d_p23counts = nullptr;
    int32_t p23_chunk = 256;             // simulations per queue item
    // launch shapes (cse_autotune): waves of the one-wave-per-block kernels, workgroups of the
    // group kernels
    int64_t tune_waves = 16384, tune_wgs = 16384;
    std::vector<int64_t> blk_sims;       // simulations of each block
    std::vector<int64_t> blk_row, blk_col;   // 2-arm: each block's row / column group of 8 thresholds
    std::vector<int32_t> blk_rg, blk_cg;     // 2-arm: their indices in d_grp2
    std::vector<int64_t> p23_item_off;   // [n_tiles + 1] first queue item of each tile
    int64_t h4_outcomes = 0;
    double table_ms = 0.0;               // time to build the design table at platten creation
    int32_t *d_cut_tbl = nullptr;        // 2-arm: c(y0) = min{y1 : z(y0, y1) > cut}, [n+1]
    double *d_S_tbl = nullptr;           // 2-arm: S = -z per outcome y0*(n+1)+y1
    int32_t *d_S_order = nullptr;        // 2-arm: outcomes sorted by S ascending
    int32_t *d_S_group = nullptr;        // 2-arm: index of first outcome with equal S in that order
    int32_t *d_S_pos = nullptr;          // 2-arm: position of each outcome in that order
    int32_t *d_gstart = nullptr;         // 2-arm: first position of each tie group of S, [n_groups + 1]
    uint8_t *d_gcut = nullptr;           // 2-arm: per tie group g and y0, #{y1 : S(y0, y1) >= S_g}, [n_groups + 1][n + 1]
    int32_t n_groups = 0;
    float b2_margin = 5.0f;              // 2-arm selection: bracket margin in standard deviations of the count
    int32_t n_outcomes = 0;
    // 2-arm calibration: per-tile bracket of S-order positions [lo, hi] expected to hold the
    // k-th smallest statistic, and the number of tiles the last selection took from the full histogram
    int2 *d_b2br = nullptr;
    uint32_t *d_b2fb = nullptr;
    // 2-arm calibration: per block, row group u and arm-0 count y0, the cut points on y1 of the
    // row's 8 tiles as bytes: x, y = clo (S < S(lo) iff y1 >= clo), z, w = chi (S <= S(hi) iff
    // y1 >= chi); [n_blocks][8][n + 1]
    uint4 *d_b2cut = nullptr;

    std::vector<uint32_t> tile_T;        // [n_tiles * d] Bernoulli thresholds (binomial designs)

    // launch-shape generation: advanced whenever the work-item arrays a captured plan refers to are
    // rebuilt (cse_autotune), and set to PLATTEN_GONE when the platten is destroyed.  Plans hold a
    // reference to this counter and refuse to replay once it differs from its value at capture.
    std::shared_ptr<std::atomic<uint64_t>> shape_gen = std::make_shared<std::atomic<uint64_t>>(0);

    // side stream (default priority) and fork/join events of the calibration step: the
    // validation bound runs beside the selection, and in a captured graph the inversion beside
    // the simulation
    hipStream_t side = nullptr;
    // device arenas holding the read-only per-tile arrays and design tables, each filled by one
    // host-to-device copy at creation (base, bytes); the arrays point into them
    std::vector<std::pair<void *, size_t>> arenas;
    hipEvent_t ev_sim = nullptr, ev_val = nullptr, ev_fork = nullptr, ev_inv = nullptr;

    // Clopper-Pearson table: one entry per (N class, R), R = 0..N (classes = distinct N)
    int32_t n_cls = 0;
    int64_t n_cp = 0;                    // sum over classes of N + 1
    int32_t *d_cls_N = nullptr;          // [n_cls]
    int64_t *d_cls_off = nullptr;        // [n_cls] first entry of each class
    int64_t *d_cp_base = nullptr;        // [n_tiles] first entry of the tile's class
    uint32_t *d_cp_mark = nullptr;       // [n_cp] R values present in this call
    double *d_cp_tbl = nullptr;          // [n_cp]
    int32_t max_cls_N = 0;
    int32_t max_nv = 1;   // most vertices of any tile (the bound kernel's per-tile LDS rows)

    // per-tile workspaces (allocated with the platten)
    uint32_t *d_Rw = nullptr;            // rejection counts
    unsigned long long *d_Tw = nullptr;  // score sums T (binomial) [n_tiles * d]
    unsigned long long *d_Zw = nullptr;  // score sums Z (z-test), fixed point 2^-32
    double *d_apw = nullptr;             // alpha'
    int32_t *d_kw = nullptr;             // k
    double *d_lamw = nullptr;            // lambda*_i
    double *d_lamg = nullptr;            // lambda* (1)
    double *d_minpart = nullptr;         // [2 * MIN_PARTS] partial minima of the reductions over tiles
                                         // (values; for pairs, their second components after them)

    // calibration keys (allocated on first calibration): n_keys entries of 2 (outcome
    // index) or 4 (float32 statistic) bytes
    void *d_keys = nullptr;
    size_t keys_bytes = 0;
};

// error reporting
void set_error(const std::string &msg);
const char *get_error();

int build_platten(const cse_design *design, int64_t n_boxes, const double *theta,
                  const double *radii, const int32_t *sims, int32_t flags, Platten *P);
void free_platten(Platten *P);
// hipMalloc on the current device; short of memory, the buffers that the library keeps for later plattens go first.
hipError_t dev_malloc(void **p, size_t bytes);
void release_cached_memory();
int plan_work_items(Platten *P, int64_t target_waves);
int plan_group_items(Platten *P, int64_t target_wgs);
int plan_h4_items(Platten *P, int64_t target_wgs);
int plan_queue_items(Platten *P, int32_t chunk, int64_t grid);

}  // namespace cse

#define CSE_HIP_TRY(expr)                                                                   \
    do {                                                                                    \
        hipError_t _e = (expr);                                                             \
        if (_e != hipSuccess) {                                                             \
            ::cse::set_error(std::string(#expr " failed: ") + hipGetErrorString(_e));       \
            return CSE_EHIP;                                                                \
        }                                                                                   \
    } while (0)
