// exact_topk: plans and launch entry points.
#pragma once

#include "atk_common.h"

namespace atk {

// exact_topk plan: rows that one workgroup holds in registers (atk_exact_row.hip) ...
constexpr int kRowMaxK = 16384;   // survivors that its selection orders in LDS
constexpr int kRowBinMax = 64;    // fullest bin whose elements it ranks by comparing them with one another
struct RowPlan {
    int T, nv;          // threads per workgroup, 16-byte vectors of the row per lane
    int lg_bins;        // log2 of the histogram's bins
    int filed_words;    // composites that the LDS holds
    int cap;            // elements at or above the first bound that pass through LDS (0: none do)
    int lds_bytes;
    int sub, rank;      // the first lower bound: the rank-th largest of the maxima of 64 * sub groups in every wavefront
    int ve;             // elements per vector
    int parts;          // > 0: workgroups to a row, each with part_vecs vectors of it, which pass on up to part_cap elements
    int part_vecs, part_cap;
    int rank_up;        // the rank of an upper bound, where LDS does not hold what a row's parts pass on
};
// false: the row does not fit.  pairs: the rows are lists of (value, index) pairs.  ptr16: x lies on a 16-byte boundary.
bool plan_exact_row(int64_t m, int64_t n, int64_t k, int dtype, bool pairs, bool ptr16, RowPlan *out);
hipError_t launch_exact_row(const RowPlan &pl, int64_t m, int64_t n, int64_t k, int64_t idx_n, int dtype, const void *x,
                            const int32_t *xi, void *out_vals, int32_t *out_idx, void *state, void *data, hipStream_t stream);
bool plan_exact_parts(int64_t m, int64_t n, int64_t k, int dtype, bool ptr16, RowPlan *out);
int64_t exact_parts_state_bytes(int64_t m);
int64_t exact_parts_data_bytes(const RowPlan &pl, int64_t m);
// A kernel that is about to be launched with more dynamic LDS than a launch may ask for by default is told so, once per
// device (told: that kernel's own flags).
hipError_t allow_whole_cu_lds(const void *kernel, bool (&told)[64]);

// ... short bf16 rows that a wavefront takes alone (atk_wave_exact.hip) ...
struct WaveExactPlan {
    int NV;   // 16-byte vectors per lane
    int R;    // rows sorted as a whole: words per lane that the sorted outputs take (0: not that)
    int H;    // else: blocks of 64 H words are sorted,
    int G;    // and the bound comes from 128 G groups of elements
};
bool plan_wave_exact(int64_t m, int64_t n, int64_t k, int dtype, bool ptr16, WaveExactPlan *out);
hipError_t launch_wave_exact(const WaveExactPlan &pl, int64_t m, int64_t n, int64_t k, const void *x, void *out_vals, int32_t *out_idx, hipStream_t stream);

// ... long rows with many winners (atk_exact_deal.hip) ...
struct DealRow {          // per row, on the device
    uint32_t k_min, k_max;   // range of the fine bins
    uint32_t tb;             // the threshold: the lowest fine bin that counts
    uint32_t cursor;         // candidates dealt
    uint32_t split;          // the bins are cut at elements of the sample, not at fine bins
};
struct DealPlan {
    int chunks, bins;        // per row
    int sample_rank;         // sampled elements above the threshold, at least
    int split_rank;          // the same where the bins are cut at sampled elements
    float expect;            // sampled elements among the k largest
    int rank;                // of the sample's lower bound, as in RowPlan
    int64_t pool_cap;        // candidates per row
    int64_t rows_off, table_off, totals_off, segs_off, pool_off, rest_off, bytes;  // byte offsets into the data pool
};
bool plan_exact_deal(int64_t m, int64_t n, int64_t k, int dtype, bool ptr16, DealPlan *out);
hipError_t launch_exact_deal(const DealPlan &pl, int64_t m, int64_t n, int64_t k, int64_t idx_n, int dtype, const void *x,
                             const int32_t *xi, void *out_vals, int32_t *out_idx, void *data, hipStream_t stream);
// The rows whose candidates number fewer than k or more than pool_cap: one workgroup per row.
// buf0, buf1: m * k composites each.
hipError_t launch_exact_rest_rows(int64_t m, int64_t n, int64_t k, int idx_bits, int dtype, const void *x, const int32_t *xi,
                                  const DealRow *rows, int64_t pool_cap, u64 *buf0, u64 *buf1, void *out_vals, int32_t *out_idx,
                                  hipStream_t stream);

// ... and the rest
struct ExactPlan {
    int dtype;
    int64_t m, n, k;
    int64_t idx_n;          // column indices are below this (n, unless the rows are lists of (value, index) pairs)
    bool single_wg;         // one workgroup per row, the row in its registers (`row`)
    bool parts;             // several, each with a part of it (`row`)
    bool wave;              // one wavefront per row (`wv`; single_wg is set, too: no scratch, no limit on the rows)
    WaveExactPlan wv;
    RowPlan row;
    bool dealt;             // dealt to bins (`deal`)
    DealPlan deal;
    int chunks;             // workgroups per row of the global path
    int chunk_elems;        // elements of a row that one of them sweeps
    bool filter;            // small k: rows may finish through the copy-out buffer
    int filter_cap;         // ... of this many elements per row
    bool sample;            // very small k on big inputs: the copy-out threshold is first guessed from a sample of the row
    int64_t scratch_bytes;  // data pool
    int64_t state_bytes;    // zeroed-state pool
};
int make_exact_plan(int64_t m, int64_t n, int64_t k, int dtype, bool pairs, bool ptr16, ExactPlan *plan, bool by_digits = false);
// xi: NULL, or (device, m x n int32) the column index each element of x stands for: the rows are then
// lists of (value, index) pairs with distinct indices below plan.idx_n, and the order among equal
// values and out_idx follow those indices (Stage 2 over more candidates than fit one workgroup).
hipError_t launch_exact(const ExactPlan &plan, const void *x, const int32_t *xi, void *out_vals, int32_t *out_idx,
                        void *state, void *data, hipStream_t stream);

// approx_topk: Stage 2 over candidates that the fused kernels could select from as a launch of its own (planner, estimate).
bool stage2_apart(int64_t m, int64_t n, int64_t k, int64_t b, int64_t k_b, int dtype);

}  // namespace atk
