// exact_topk of rows that one workgroup holds in registers (and Stage 2 over more candidates than the fused kernels
// select from): one launch, one workgroup per row, the row read once.
//
//   1. Every lane loads its share of the row, 16 bytes per load, all loads in flight together.
//   2. A lower bound on the k-th largest: every wavefront finds the rank-th largest of the maxima of its groups of elements (of
//      a lane's elements, or of parts of them), with wavefronts times rank just over k, and the smallest of these is
//      reached by at least k elements; among elements in no particular order, by not many more (k = 256 of 128256: 370; the
//      minimum over as many groups' maxima, which needs no selection in the wavefront, lets 1400 through and now and then 3000).
//   3. A histogram of the elements from there on, over bins linear in (value key, index) between the bound and the row's
//      maximum; a descending prefix sum turns counts into places.  A bin too full to be ranked by comparing its elements
//      with one another: again from the lower edge of the bin that holds the k-th, which is a range without what lies
//      below (values around zero stretch a range of keys over every exponent).
//   4. The elements of the bins down to the k-th's go to LDS, bin by bin; each finds its rank as its bin's start plus
//      the larger elements of its bin.  Lanes side by side take places side by side, so the row is written nearly in order.
// Rows whose bins stay crowded (long runs of one value) are selected digit by digit (RadixSelect, Appendix D.2) and ordered
// by order_write(); they re-read the row, which is in the caches by then.
// Longer rows, and long rows of small batches, are shared out between workgroups (ex_parts_kernel).
//
// What bounds it: with at most one row per CU, the rate at which one CU takes in a row (about 45 GB/s, measured: 256 KB in
// 5.8 us) and then the operations on every element; with many rows the latter, shared out over the workgroups of a CU.
// Measured against the launches this replaced (a histogram, a decision, a copy-out and a selection; one workgroup
// with the row in LDS for short rows): 2048 x 8192 bf16, k = 512: 79.9 -> 19.5 us; 64 x 128256 bf16, k = 256: 28.9 -> 12.0;
// 1024 x 65536 f32, k = 64: 106 -> 62; 128 x 65536 f32, k = 16384: 148 -> 57; one row of 65536 f32, k = 4096: 120 -> 32;
// 2048 x 2048 f32, k = 64: 43 -> 8.2; 128 lists of 8192 pairs, k = 4096 (Stage 2): 118 -> 12.4.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "atk_common.h"
#include "atk_exact.h"
#include "atk_exact_regs.h"
#include "atk_select.h"

namespace atk {

template <int ELT>
__device__ __forceinline__ u64 row_composite(const RowParams &p, int64_t r, int i) {
    const uint32_t bits = (ELT == ATK_F32) ? ((const uint32_t *)p.x)[r * p.n + i] : ((uint32_t)((const uint16_t *)p.x)[r * p.n + i]) << 16;
    return make_composite(bits, p.xi ? p.xi[r * p.n + i] : i);
}

// f(composite, whether it is one) for every element of row r, whole wavefronts together
template <int ELT, bool XI, typename F>
__device__ __forceinline__ void row_sweep(const RowParams &p, int64_t r, F f) {
    constexpr int ES = (ELT == ATK_F32) ? 4 : 2, VE = 16 / ES;
    if constexpr (!XI) {
        const int rot = (int)(((uintptr_t)p.x + (uintptr_t)(r * p.n) * ES) & 15) / ES;
        row_vec_sweep<ELT>(p, r, 0, (rot + p.n + VE - 1) / VE, rot, f);
        return;
    }
    const int T = blockDim.x, lane = threadIdx.x & (kWave - 1);
    for (int i0 = (int)threadIdx.x - lane; i0 < p.n; i0 += 4 * T) {
        u64 c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) c[u] = row_composite<ELT>(p, r, min(i0 + lane + u * T, p.n - 1));
#pragma unroll
        for (int u = 0; u < 4; ++u) f(c[u], i0 + lane + u * T < p.n);
    }
}

// The elements at or above thr (squeezed), of which there are k, are put in order and written.
template <int ELT, typename SWEEP>
__device__ __forceinline__ void row_order_from(const RowParams &p, int64_t r, SWEEP sweep, u64 thr, u64 *filed, uint32_t *cur, uint32_t *misc) {
    const int tid = threadIdx.x, T = blockDim.x;
    const RowSqueeze<ELT> sq{p.idx_bits + 1};
    if (tid == 0) misc[5] = 0u;
    for (int i = tid; i < kRankMax; i += T) cur[i] = 0u;
    __syncthreads();
    sweep([&](u64 c, bool on) {
        if (on && sq(c) >= thr) {
            const uint32_t at = atomicAdd(&misc[5], 1u);
            if (at < (uint32_t)p.k) filed[at] = c;
        }
    });
    __syncthreads();
    order_write<ELT>(filed, p.k, cur, p.out_vals, p.out_idx, r);
}
// Digit by digit over what sweep() goes through, as in row_threshold_by_digits().
template <int ELT, typename SWEEP>
__device__ __forceinline__ void row_by_digits(const RowParams &p, int64_t r, SWEEP sweep, uint32_t k_lo, uint32_t k_hi, u64 *filed,
                                              uint32_t *cur, uint32_t *misc) {
    const u64 thr = row_threshold_by_digits<ELT>(sweep, (uint32_t)p.k, k_lo, k_hi, p.idx_bits, p.lg_bins, cur, misc);
    row_order_from<ELT>(p, r, sweep, thr, filed, cur, misc);
}

// The filed elements (bin by bin, cur[b] the place behind bin b) find their ranks and are written.
template <int ELT>
__device__ __forceinline__ void row_rank_write(const RowParams &p, int64_t r, const RowBins &bins, const u64 *filed, int filed_n,
                                               const uint32_t *cur, int n_bins) {
    for (int i = threadIdx.x; i < filed_n; i += blockDim.x) {
        const u64 c = filed[i];
        const uint32_t b = bins.template bin<ELT>((uint32_t)(c >> 32), (uint32_t)c >> 1);
        const int s = b + 1u < (uint32_t)n_bins ? (int)cur[b + 1] : 0, e = (int)cur[b];
        u64 peer[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) peer[u] = filed[s + u < e ? s + u : i];  // (itself: not larger)
        int rank = s;
#pragma unroll
        for (int u = 0; u < 4; ++u) rank += peer[u] > c ? 1 : 0;
        for (int j = s + 4; j < e; ++j) rank += filed[j] > c ? 1 : 0;
        if (rank < p.k) write_composite<ELT>(c, p.out_vals, p.out_idx, r * p.k + rank);
    }
}

// Selects and writes the row's k largest from those of passed[0 .. n_passed) (value bits, column index) at or above k_min, k or
// more of them.  cur: zeroed bins.  False where a bin is too full to be ranked: nothing is written then, and k_min is raised to
// the lower edge of the k-th largest's bin.  Called by the whole workgroup after a barrier.
template <int ELT>
__device__ __forceinline__ bool row_select_passed(const RowParams &p, int64_t r, const int2 *passed, uint32_t n_passed, uint32_t &k_min,
                                                  uint32_t k_max, u64 *filed, uint32_t *cur, uint32_t *misc) {
    const int tid = threadIdx.x, T = blockDim.x, n_bins = 1 << p.lg_bins;
    RowBins bins;
    bins.template set<ELT>(k_min, k_max, p.idx_bits, n_bins);
    for (uint32_t i = tid; i < n_passed; i += T) {
        const int2 w = passed[i];
        const uint32_t key = ukey_of_bits((uint32_t)w.x);
        if (key >= bins.k_min) atomicAdd(&cur[bins.template bin<ELT>(key, 0x7fffffffu - (uint32_t)w.y)], 1u);
    }
    __syncthreads();
    row_scan(cur, misc, n_bins, (uint32_t)p.k);
    const uint32_t tb = misc[0];
    if (misc[4] != 0u) {
        const uint32_t lo = bins.template edge<ELT>(tb);
        if (lo > k_min) k_min = lo;
        __syncthreads();
        return false;
    }
    for (uint32_t i = tid; i < n_passed; i += T) {
        const int2 w = passed[i];
        const uint32_t key = ukey_of_bits((uint32_t)w.x), b = bins.template bin<ELT>(key, 0x7fffffffu - (uint32_t)w.y);
        if (key >= bins.k_min && b >= tb) filed[atomicAdd(&cur[b], 1u)] = make_composite((uint32_t)w.x, w.y);
    }
    __syncthreads();
    row_rank_write<ELT>(p, r, bins, filed, (int)cur[tb], cur, n_bins);
    return true;
}

template <int ELT, int NV, bool XI>
__global__ void __launch_bounds__(1024) ex_row_kernel(RowParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int ES = (ELT == ATK_F32) ? 4 : 2, VE = 16 / ES;
    const int tid = threadIdx.x, T = blockDim.x;
    const int64_t r = blockIdx.x;
    const int n_bins = 1 << p.lg_bins;
    u64 *filed = (u64 *)smem;
    uint32_t *cur = (uint32_t *)(filed + p.filed_words);  // [n_bins], then a zero: nothing lies above the last bin
    uint32_t *misc = cur + n_bins + 4;
    int2 *passed = (int2 *)(misc + kRowMisc);

    const int rot = (int)(((uintptr_t)p.x + (uintptr_t)(r * p.n) * ES) & 15) / ES, end = rot + p.n;
    const int n_vec = (end + VE - 1) / VE;
    RowRegs<ELT, NV> regs;
    regs.load(p, r, 0, n_vec, rot);
    int32_t xi[XI ? NV * VE : 1];
    if constexpr (XI) {
        // (the pairs' two arrays start on 16-byte boundaries, so a vector of values and its indices do together)
        const int4 *ir = (const int4 *)(p.xi + (r * p.n - rot));
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int v = tid + j * T;
#pragma unroll
            for (int h = 0; h < VE / 4; ++h) {
                const int64_t at = (int64_t)(v < n_vec ? v : 0) * (VE / 4) + h;
                // (four indices without one of the row's may lie past the array: the first four again)
                const int4 w = ir[at * 4 < end ? at : at - h];
                xi[j * VE + 4 * h] = w.x;
                xi[j * VE + 4 * h + 1] = w.y;
                xi[j * VE + 4 * h + 2] = w.z;
                xi[j * VE + 4 * h + 3] = w.w;
            }
        }
    }
    for (int i = tid; i < n_bins + 4; i += T) cur[i] = 0u;
    if (tid == 0) misc[5] = 0u;
    regs.mask_ends(p, 0, n_vec, rot);
    uint32_t k_min, k_max;
    regs.bound(p.sub, p.rank, misc, k_min, k_max);

    int attempt = 0;
    if (p.cap) {
        // few of the elements reach the bound: they go to LDS (value bits, index) side by side, and the histogram and the
        // filing, a dozen operations and an LDS atomic per element each, run over them instead of over all registers with
        // most lanes idle (2048 x 8192 bf16, k = 512: 29.7 -> 20.3 us; 2048 x 32768 bf16, k = 256: 68.9 -> 37.7)
        regs.list_from(__uint_as_float(bits_of_ukey(k_min)), passed, (uint32_t)p.cap, &misc[5]);
        const uint32_t n_passed = misc[5];
        if (n_passed >= (uint32_t)p.k && n_passed <= (uint32_t)p.cap) {
            for (uint32_t i = tid; i < n_passed; i += T) {  // (each lane's own entries: no barrier before the histogram reads them)
                const int at = passed[i].y;
                passed[i] = make_int2((int)row_bits<ELT>(p, r, at), XI ? p.xi[r * p.n + at] : at);
            }
            if (row_select_passed<ELT>(p, r, passed, n_passed, k_min, k_max, filed, cur, misc)) return;
            attempt = 1;
            for (int i = tid; i < n_bins; i += T) cur[i] = 0u;
            __syncthreads();
        }
    }
    RowBins bins;
    for (;; ++attempt) {
        bins.template set<ELT>(k_min, k_max, p.idx_bits, n_bins);
        const float v_lo = __uint_as_float(bits_of_ukey(k_min));
        regs.each([&](uint32_t bits, int at, int en) {
            if (__uint_as_float(bits) >= v_lo)
                atomicAdd(&cur[bins.template bin<ELT>(ukey_of_bits(bits), 0x7fffffffu - (uint32_t)(XI ? xi[en] : at))], 1u);
        });
        __syncthreads();
        row_scan(cur, misc, n_bins, (uint32_t)p.k);
        const bool few = misc[3] < (uint32_t)p.k, crowded = misc[4] != 0u;
        if (!few && !crowded) break;
        const uint32_t lo = few ? 0x007fffffu : bins.template edge<ELT>(misc[0]);  // (-inf's key)
        // (twice from a raised lower end at most, and once from -inf)
        if (attempt == 3 || (few ? k_min <= lo : lo <= k_min)) {
            __syncthreads();
            // (few: NaNs)
            row_by_digits<ELT>(p, r, [&](auto f) { row_sweep<ELT, XI>(p, r, f); }, few ? 0u : k_min, few ? 0xffffffffu : k_max, filed, cur, misc);
            return;
        }
        k_min = lo;
        __syncthreads();
        for (int i = tid; i < n_bins; i += T) cur[i] = 0u;
        __syncthreads();
    }
    // ---- the winners' bins, brought together; cur[b] ends as the place behind bin b, which is where bin b - 1 starts
    const uint32_t tb = misc[0];
    {
        const float v_lo = __uint_as_float(bits_of_ukey(bins.template edge<ELT>(tb)));
        regs.each([&](uint32_t bits, int at, int en) {
            if (__uint_as_float(bits) >= v_lo) {
                const int idx = XI ? xi[en] : at;
                const uint32_t b = bins.template bin<ELT>(ukey_of_bits(bits), 0x7fffffffu - (uint32_t)idx);
                if (b >= tb) filed[atomicAdd(&cur[b], 1u)] = make_composite(bits, idx);
            }
        });
    }
    __syncthreads();
    row_rank_write<ELT>(p, r, bins, filed, (int)cur[tb], cur, n_bins);
}

// A row shared out between workgroups (ex_parts_kernel).
template <int ELT>
struct PartsRow {
    static constexpr int VE = (ELT == ATK_F32) ? 4 : 8;
    int64_t r;
    int rot, n_vec, n_bins;
    u64 *filed;
    uint32_t *cur, *misc;
    int2 *passed;
    __device__ __forceinline__ PartsRow(const RowParams &p, int64_t row, unsigned char *smem) : r(row) {
        rot = (int)(((uintptr_t)p.x + (uintptr_t)(r * p.n) * (16 / VE)) & 15) / (16 / VE);
        n_vec = (rot + p.n + VE - 1) / VE;
        n_bins = 1 << p.lg_bins;
        filed = (u64 *)smem;
        cur = (uint32_t *)(filed + p.filed_words);
        misc = cur + n_bins + 4;
        passed = (int2 *)(misc + kRowMisc);
    }
    // (a part may be empty: the plan counts a vector more for rows off the 16-byte boundaries)
    __device__ __forceinline__ int first_vec(const RowParams &p, int part) const { return min(part * p.part_vecs, n_vec - 1); }
    __device__ __forceinline__ int end_vec(const RowParams &p, int part) const {
        return part * p.part_vecs < n_vec ? min(part * p.part_vecs + p.part_vecs, n_vec) : first_vec(p, part);
    }
    __device__ __forceinline__ uint32_t elements(const RowParams &p, int part) const {
        return (uint32_t)(min(end_vec(p, part) * VE, rot + p.n) - max(first_vec(p, part) * VE, rot));
    }
    __device__ __forceinline__ void clear_bins() const {
        for (int i = threadIdx.x; i < n_bins + 4; i += blockDim.x) cur[i] = 0u;
    }
    __device__ __forceinline__ void clear() const {  // the bins and the cursors; ends in a barrier
        clear_bins();
        if (threadIdx.x == 0) misc[5] = misc[7] = 0u;
        __syncthreads();
    }
    __device__ __forceinline__ void put_head(const RowParams &p, int part, uint32_t low, uint32_t front, uint32_t back, uint32_t k_up, uint32_t k_max) const {
        if (threadIdx.x != 0) return;
        u64 *head = p.heads + (r * p.parts + part) * 4;
        __hip_atomic_store(&head[0], ((u64)low << 32) | front, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&head[1], ((u64)k_max << 32) | back, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&head[2], (u64)k_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ u64 element(const RowParams &p, uint32_t i) const {  // of passed[], where it has a position only
        const int at = passed[i].y;
        return make_composite(row_bits<ELT>(p, r, at), at);
    }
};
__device__ __forceinline__ uint32_t key_of(u64 c) { return (uint32_t)(c >> 32); }

// Part `part` passes on the n_passed elements whose positions are in passed[] (none below `low` or above k_max, its k largest among them), or
// where that is more than it may pass on, those down to the bin of the k-th, or where that bin is too full exactly k.  k_up: the part's
// upper bound.
template <int ELT>
__device__ __forceinline__ void parts_hand_over(const RowParams &p, const PartsRow<ELT> &w, int part, uint32_t n_passed, uint32_t low, uint32_t k_up,
                                                uint32_t k_max) {
    const int tid = threadIdx.x, T = blockDim.x, lane = tid & (kWave - 1);
    __syncthreads();  // (the cursor has been read by all)
    if (tid == 0) w.misc[5] = w.misc[7] = 0u;
    __syncthreads();
    u64 *list = p.lists + (w.r * p.parts + part) * p.part_cap;
    auto put = [&](u64 c, bool on) {  // whole wavefronts together
        const bool up = on && key_of(c) >= k_up;
        const u64 m_up = __ballot(up), m_low = __ballot(on && !up);
        uint32_t to = 0;
        if (lane == 0 && m_up) to = atomicAdd(&w.misc[5], (uint32_t)__popcll(m_up));
        if (lane == 1 && m_low) to = atomicAdd(&w.misc[7], (uint32_t)__popcll(m_low));
        const uint32_t to_up = (uint32_t)__builtin_amdgcn_readlane((int)to, 0), to_low = (uint32_t)__builtin_amdgcn_readlane((int)to, 1);
        const u64 mine = up ? m_up : m_low;
        const uint32_t place = __builtin_amdgcn_mbcnt_hi((uint32_t)(mine >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mine, 0u));
        const uint32_t at = up ? to_up + place : (uint32_t)p.part_cap - 1u - to_low - place;
        if (on && at < (uint32_t)p.part_cap) __hip_atomic_store(&list[at], c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    if (n_passed <= (uint32_t)p.part_cap) {
        for (uint32_t i0 = tid - lane; i0 < n_passed; i0 += T) {
            const bool on = i0 + lane < n_passed;
            put(on ? w.element(p, i0 + lane) : 0ull, on);
        }
    } else {
        w.clear();
        RowBins bins;
        bins.template set<ELT>(low, k_max, p.idx_bits, w.n_bins);
        auto bin_of = [&](u64 c) { return bins.template bin<ELT>(key_of(c), (uint32_t)c >> 1); };
        // (each lane's own entries, which get their values first)
        for (uint32_t i = tid; i < n_passed; i += T) w.passed[i].x = (int)row_bits<ELT>(p, w.r, w.passed[i].y);
        auto listed = [&](auto f) {  // whole wavefronts together
            for (uint32_t i0 = tid - lane; i0 < n_passed; i0 += T) {
                const bool on = i0 + lane < n_passed;
                const int2 e = w.passed[on ? i0 + lane : 0u];
                f(make_composite((uint32_t)e.x, e.y), on);
            }
        };
        listed([&](u64 c, bool on) { row_count(w.cur, on ? bin_of(c) : 0u, on); });
        __syncthreads();
        row_scan(w.cur, w.misc, w.n_bins, (uint32_t)p.k);
        const uint32_t tb = w.misc[0];
        const bool fits = w.misc[1] + w.misc[2] <= (uint32_t)p.part_cap;
        __syncthreads();
        const RowSqueeze<ELT> sq{p.idx_bits + 1};
        const u64 thr = fits ? 0ull : row_threshold_by_digits<ELT>(listed, (uint32_t)p.k, low, k_max, p.idx_bits, p.lg_bins, w.cur, w.misc);
        uint32_t least = 0xffffffffu;
        listed([&](u64 c, bool on) {
            const bool goes = on && (fits ? bin_of(c) >= tb : sq(c) >= thr);
            least = goes ? min(least, key_of(c)) : least;
            put(c, goes);
        });
        least = wave_min_u32(least);
        if (lane == 0) w.misc[8 + (tid >> 6)] = least;
        __syncthreads();
        low = wave_min_u32(lane < (T >> 6) ? w.misc[8 + lane] : 0xffffffffu);
    }
    __syncthreads();
    w.put_head(p, part, low, w.misc[5], w.misc[7], k_up, k_max);
}

// A part whose elements at or above k_min are more than LDS lists: its k largest, from registers that are loaded again (kept from the first
// time, they would be spilled on the way that most parts take).
template <int ELT, int NV>
__device__ __forceinline__ void part_largest(const RowParams &p, const PartsRow<ELT> &w, int part, uint32_t k_min, uint32_t k_up, uint32_t k_max) {
    RowRegs<ELT, NV> regs;
    const int v0 = w.first_vec(p, part), v1 = w.end_vec(p, part);
    __syncthreads();
    regs.load(p, w.r, v0, v1, w.rot);
    if (threadIdx.x == 0) w.misc[5] = 0u;
    regs.mask_ends(p, v0, v1, w.rot);
    uint32_t n_passed;
    const uint32_t low = regs.list_largest((uint32_t)p.k, k_min, k_max, w.passed, (uint32_t)p.cap, n_passed, &w.misc[5], w.cur, w.misc);
    parts_hand_over<ELT>(p, w, part, n_passed, low, k_up, k_max);
}

// The lists of a row as its last workgroup sees them: lane i of every wavefront has the head of part i.
struct PartsHeads {
    uint32_t front = 0u, back = 0u;   // elements in the two pieces
    uint32_t k_min = 0u, k_max = 0u;  // of the row: its k largest lie between them
    uint32_t k_up = 0u;               // everything passed on from there on is in the first pieces
    __device__ __forceinline__ PartsHeads(const RowParams &p, int64_t r) {
        const int lane = threadIdx.x & (kWave - 1);
        if (lane < p.parts) {
            const u64 *head = p.heads + (r * p.parts + lane) * 4;
            const u64 h0 = __hip_atomic_load(&head[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const u64 h1 = __hip_atomic_load(&head[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            k_up = (uint32_t)__hip_atomic_load(&head[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            front = (uint32_t)h0;
            back = (uint32_t)h1;
            k_min = front + back >= (uint32_t)p.k ? (uint32_t)(h0 >> 32) : 0u;  // (k elements of this part reach it)
            k_max = (uint32_t)(h1 >> 32);
        }
        k_min = wave_max_u32(k_min);
        k_max = wave_max_u32(k_max);
        k_up = max(wave_max_u32(k_up), k_min);
    }
    // f(composite, whether there is one) for every element of the lists' first or second pieces: the wavefronts take 64 in turn, eight
    // loads in flight
    template <typename F>
    __device__ __forceinline__ void sweep(const RowParams &p, int64_t r, bool first_pieces, F f) const {
        constexpr int U = 8;
        const int lane = threadIdx.x & (kWave - 1);
        const uint32_t len = first_pieces ? front : back;
        const u64 *lists = p.lists + r * p.parts * p.part_cap;
        const uint32_t pieces = (len + kWave - 1) / kWave, pieces_end = wave_incl_scan_u32(pieces);
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)pieces_end, kWave - 1);
        const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), n_waves = blockDim.x >> 6;
        for (uint32_t c0 = wave; c0 < total; c0 += U * n_waves) {
            u64 c[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t id = c0 + u * n_waves;
                c[u] = 0ull;
                if (id < total) {  // uniform over the wavefront
                    const int of = __popcll(__ballot(pieces_end <= id));  // the part whose piece it is
                    const uint32_t n_of = (uint32_t)__builtin_amdgcn_readlane((int)len, of);
                    const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)(pieces_end - pieces), of);
                    const uint32_t i = (id - first) * kWave + (uint32_t)lane, at = min(i, n_of - 1u);
                    c[u] = __hip_atomic_load(&lists[(uint32_t)of * (uint32_t)p.part_cap + (first_pieces ? at : (uint32_t)p.part_cap - 1u - at)],
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (i >= n_of) c[u] = 0ull;
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) f(c[u], c[u] != 0ull);
        }
    }
};

// sweep()'s elements that take() says, side by side into passed[]; returns how many.  Called by the whole workgroup with the cursors cleared.
template <int ELT, typename SWEEP, typename TAKE>
__device__ __forceinline__ uint32_t parts_gather(const RowParams &p, const PartsRow<ELT> &w, SWEEP sweep, TAKE take) {
    const int lane = threadIdx.x & (kWave - 1);
    sweep([&](u64 c, bool on) {
        const bool mine = take(c, on);
        const u64 mask = __ballot(mine);
        if (mask) {  // uniform over the wavefront
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&w.misc[5], (uint32_t)__popcll(mask));
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) +
                 __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            if (mine && at < (uint32_t)p.cap) w.passed[at] = make_int2((int)composite_bits(c), composite_index(c));
        }
    });
    __syncthreads();
    return w.misc[5];
}

// The row's k largest of what has been gathered (n >= k elements, all at or above k_min, no more than LDS holds) are written.
template <int ELT>
__device__ __forceinline__ void parts_finish(const RowParams &p, const PartsRow<ELT> &w, uint32_t n, uint32_t k_min, uint32_t k_max) {
    const int lane = threadIdx.x & (kWave - 1);
    for (uint32_t from = k_min;;) {  // once more from a raised lower end
        const uint32_t was = from;
        if (row_select_passed<ELT>(p, w.r, w.passed, n, from, k_max, w.filed, w.cur, w.misc)) return;
        w.clear();
        if (from == was || was != k_min) break;
    }
    auto listed = [&](auto f) {  // whole wavefronts together
        for (uint32_t i0 = threadIdx.x - lane; i0 < n; i0 += blockDim.x) {
            const bool on = i0 + lane < n;
            const int2 e = w.passed[on ? i0 + lane : 0u];
            f(make_composite((uint32_t)e.x, e.y), on);
        }
    };
    row_by_digits<ELT>(p, w.r, listed, k_min, k_max, w.filed, w.cur, w.misc);
}

// Several workgroups to a row: each holds a part of it in registers, finds a lower bound that at least k of its elements reach, and
// passes on what lies at or above it, so that the k largest of the row are among what its parts pass on however unlike each other these
// are (masked stretches, rows with a trend, neighbours that go together).  A part where more reach the bound than it may pass on (long
// runs of ties) passes on its k largest.  The workgroup that draws the row's last ticket takes the largest of the bounds, which k elements of
// the row reach, and selects from what was passed on above it.  Where that is more than LDS holds (many parts, large k), the lists are cut
// at a second bound that fewer elements reach - k shared out over the parts, and a margin - and if k elements of the row
// reach the largest of these, the first pieces of the lists are enough; else all of them are binned.
// One sweep over memory, one launch.  us per call, of the launches this replaced (a sample or a histogram, a copy-out, a selection) and here:
//                                          N(0,1)   first half -inf   ascending   constant   three levels   lagged average
//   128 x 2^20 f32, k = 64                 135, 122       156, 157     832, 156  2205, 270      1130, 254         138, 145
//   128 x 2^18 f32, k = 64                  60, 34         69, 41      262, 39    512, 74        320, 72           64, 35
//   16 x 2^18 f32, k = 64                   31, 12         40, 13       41, 15     92, 16         75, 21           31, 15
//   64 x 128256 bf16, k = 256               29, 12.8       49, 13.7     53, 17.6  223, 18.6      147, 22.7         36, 17.5
//   one row of 2^20 f32, k = 1000           52, 19         55, 24       51, 63     84, 81         77, 80           51, 23
// (Parts that pass on little more than their share of k, and a row that starts over, in one workgroup, when their bounds leave fewer than
// k elements: 104, 30, 9.4, 10.2 and 13 us in the first column, and 220 to 45000 in the others.)
// The lists go through memory as in the fused kernels' hand-over: agent-scope stores, a wait for their acknowledgement, a ticket.
template <int ELT, int NV>
__global__ void __launch_bounds__(1024) ex_parts_kernel(RowParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    const int64_t r = blockIdx.x / (unsigned)p.parts;
    const int part = (int)(blockIdx.x - (unsigned)r * (unsigned)p.parts);
    const PartsRow<ELT> w(p, r, smem);
    uint32_t *misc = w.misc;
    uint32_t k_min, k_up, k_max, n_passed;
    {
        const int v0 = w.first_vec(p, part), v1 = w.end_vec(p, part);
        RowRegs<ELT, NV> regs;
        regs.load(p, r, v0, v1, w.rot);
        if (tid == 0) misc[5] = 0u;
        regs.mask_ends(p, v0, v1, w.rot);
        if constexpr (ELT == ATK_BF16) {
            regs.to_keys();
            regs.template bound<false, true, true>(p.sub, p.rank, misc, k_min, k_max, w.cur, p.rank_up, &k_up);
            regs.list_keys(k_min, w.passed, (uint32_t)p.cap, &misc[5]);
        } else {
            regs.template bound<false, true>(p.sub, p.rank, misc, k_min, k_max, w.cur, p.rank_up, &k_up);
            regs.list_from(__uint_as_float(bits_of_ukey(k_min)), w.passed, (uint32_t)p.cap, &misc[5]);
        }
        n_passed = misc[5];
    }
    bool over = n_passed > (uint32_t)p.part_cap;  // uniform, as is what follows from it
    if (over && k_min == k_max && n_passed == w.elements(p, part)) {  // one value throughout: the first k
        __syncthreads();
        for (int i = tid; i < p.k; i += (int)blockDim.x) w.passed[i].y = max(w.first_vec(p, part) * w.VE - w.rot, 0) + i;
        __syncthreads();
        n_passed = (uint32_t)p.k;
        over = false;
    }
    if (!over && !p.rank_up) {
        u64 *list = p.lists + (r * p.parts + part) * p.part_cap;
        for (uint32_t i = tid; i < n_passed; i += blockDim.x)
            __hip_atomic_store(&list[i], w.element(p, i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        w.put_head(p, part, k_min, n_passed, 0u, 0u, k_max);
    } else if (n_passed > (uint32_t)p.cap) {
        // (the same addresses as above, which the compiler must not keep until here)
        RowParams q = p;
        int same = __builtin_amdgcn_readfirstlane(part);
        asm volatile("" : "+s"(q.x), "+s"(same));
        part_largest<ELT, NV>(q, PartsRow<ELT>(q, r, smem), same, k_min, k_up, k_max);
    } else {
        parts_hand_over<ELT>(p, w, part, n_passed, k_min, k_up, k_max);
    }
    if (over || p.rank_up) __syncthreads();  // (they have worked in the bins; above, the lists end in a barrier)
    w.clear_bins();  // (by all of the workgroups, while the stores are under way, not by the last one when all wait for it: 64 x 128256 bf16, k = 64: 12.1 -> 11.8 us, k = 256 13.05 -> 12.75)
    // (a barrier alone does not wait for stores; the memory clobber keeps the compiler from moving the ticket above this)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
        uint32_t *ticket = p.tickets + r * kTicketStride;
        const bool last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)p.parts - 1u;
        misc[6] = last ? 1u : 0u;
        misc[5] = misc[7] = 0u;
        if (last) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // ready for the next call
    }
    __syncthreads();
    if (!misc[6]) return;
    // ---- the row's last workgroup
    const PartsHeads h(p, r);
    auto in = [&](u64 c, bool on) { return on && key_of(c) >= h.k_min; };
    uint32_t from = h.k_up;
    uint32_t n = parts_gather<ELT>(p, w, [&](auto f) { h.sweep(p, r, true, f); }, [&](u64 c, bool on) { return on && key_of(c) >= h.k_up; });
    if (n < (uint32_t)p.k || n > (uint32_t)p.cap) {  // down to the bin of the k-th
        auto sweep = [&](auto f) {
            h.sweep(p, r, true, f);
            h.sweep(p, r, false, f);
        };
        __syncthreads();
        w.clear();
        RowBins bins;
        bins.template set<ELT>(h.k_min, h.k_max, p.idx_bits, w.n_bins);
        auto bin_of = [&](u64 c) { return bins.template bin<ELT>(key_of(c), (uint32_t)c >> 1); };
        sweep([&](u64 c, bool on) { row_count(w.cur, in(c, on) ? bin_of(c) : 0u, in(c, on)); });
        __syncthreads();
        row_scan(w.cur, misc, w.n_bins, (uint32_t)p.k);
        const uint32_t tb = misc[0];
        n = misc[3] < (uint32_t)p.k ? 0u : misc[1] + misc[2];
        from = max(h.k_min, bins.template edge<ELT>(tb));
        __syncthreads();
        w.clear();
        if (n > (uint32_t)p.cap) {  // (ties)
            row_by_digits<ELT>(p, r, [&](auto f) { sweep([&](u64 c, bool on) { f(c, in(c, on)); }); }, from, h.k_max, w.filed, w.cur, misc);
            return;
        }
        if (n) parts_gather<ELT>(p, w, sweep, [&](u64 c, bool on) { return in(c, on) && bin_of(c) >= tb; });
    }
    if (n >= (uint32_t)p.k)
        parts_finish<ELT>(p, w, n, from, h.k_max);
    else  // (NaNs)
        row_by_digits<ELT>(p, r, [&](auto f) { row_vec_sweep<ELT>(p, r, 0, w.n_vec, w.rot, f); }, 0u, 0xffffffffu, w.filed, w.cur, misc);
}

// ------------------------------------------------------------------------------------ host
static int row_nv(int64_t want, bool pairs) {  // vectors per lane of the smallest instance that holds `want`, 0: none
    static const int have[] = {1, 2, 3, 4, 6, 8, 12, 16};
    for (int v : have)
        if (v >= want) return (pairs && v > 4) ? 0 : v;
    return 0;
}

// The bound that at least `want` elements reach: rank per wavefront, and the fewest groups per lane that keep the rank in
// the upper half of a wavefront's maxima (close to all of them the bound falls off: the smallest of the maxima).  Returns how
// many of the n_vec vectors' elements may be expected to reach it: among random elements the share above the
// rank-th of the g maxima of groups of e is 1 - (1 - rank/g)^(1/e), and the smallest over the wavefronts lies
// two or so deviations further down (`below`; half of one where the wavefronts' counts are summed).
static double row_bound_plan(RowPlan &p, int T, int64_t n_vec, double want, double below = 2.2) {
    const int ve = p.ve, waves = T / kWave;
    const int sm = p.nv * 4 < 8 ? 4 : 8;
    p.rank = (int)std::ceil(want / waves);
    p.sub = 1;
    while (p.sub < sm && p.rank > 32 * p.sub) p.sub *= 2;
    // Where much of the row is kept, finding the rank-th costs more than it drops: then the smallest of the maxima of G groups,
    // which about G ln G elements reach where the groups are small parts of the row, with half of that at k or more (checked
    // by the histogram; 128 lists of 8192 pairs, k = 4096: 26.6 us with the ranks, 23.2 so, 28.8 from the smallest element)
    const bool most = want > 0.4 * (double)(n_vec * ve);
    if (most) {
        p.rank = 0;
        for (p.sub = 1; p.sub < sm && 0.5 * T * p.sub * std::log((double)T * p.sub) < want;) p.sub *= 2;
        return (double)(n_vec * ve);
    }
    const double g = 64.0 * p.sub, per_wave = (double)n_vec * ve / waves, e = per_wave / g > 1.0 ? per_wave / g : 1.0;
    const double low = p.rank + below * std::sqrt((double)p.rank) + 1.0;
    const double share = low < g * 0.98 ? 1.0 - std::pow(1.0 - low / g, 1.0 / e) : 1.0;
    return share * per_wave * waves;
}

bool plan_exact_row(int64_t m, int64_t n, int64_t k, int dtype, bool pairs, bool ptr16, RowPlan *out) {
    const int ve = dtype == ATK_F32 ? 4 : 8;
    RowPlan p;
    memset(&p, 0, sizeof p);
    p.ve = ve;
    if (k > kRowMaxK || n > (int64_t)1024 * 16 * ve) return false;
    // vectors that hold an element of a row (rows off the 16-byte boundaries: with the worst alignment)
    const int64_t n_vec = ptr16 && n % ve == 0 ? n / ve : (n + 2 * ve - 2) / ve;
    // At most one row per CU: the biggest workgroup that still has a vector per lane.  More rows: several workgroups to a
    // CU, so that one reads while others select, each with 4 to 16 vectors per lane (2048 rows: 8192 f32, k = 64: 16.9 us with
    // 256 lanes, 39.3 with 1024; 2048 f32: 8.2 with 128, 14.6 with 512; 32768 bf16, k = 256: 37.7 with 256, 43.8 with 512), and
    // twice the lanes where a quarter of the row or more is kept, of which the tables in LDS leave room for a few workgroups
    // only (8192 f32, k = 2048: 82.3 with 256, 57.8 with 512).
    int T = kWave;
    if (m <= kNumCU) {
        while (T < 1024 && 2 * T <= n_vec) T <<= 1;
    } else {
        T = n_vec <= 512 ? 128 : (n_vec <= 4096 ? 256 : (n_vec <= 8192 ? 512 : 1024));
        if (4 * k >= n && T * 2 <= n_vec && T < 512) T *= 2;
        while (T > kWave && T > n_vec) T >>= 1;
    }
    if (plan_override().T) T = plan_override().T;
    p.nv = row_nv((n_vec + T - 1) / T, pairs);
    while (!p.nv && T < 1024) {
        T <<= 1;
        p.nv = row_nv((n_vec + T - 1) / T, pairs);
    }
    if (!p.nv) return false;
    const double expect = row_bound_plan(p, T, n_vec, (double)k);
    // Where few of the elements reach the bound they pass through LDS (a row that has more stays in the registers).
    const double cap = expect * 1.3 + 6.0 * std::sqrt(expect) + 128.0;
    p.cap = cap * 1.6 < (double)n && cap < 8192.0 ? ((int)cap + 1) & ~1 : 0;
    int lg = 8;
    while (lg < 13 && ((1 << lg) < 2 * k || (1 << lg) < T)) ++lg;
    int64_t kp = 1;
    while (kp < k) kp <<= 1;
    p.filed_words = (int)((kp > k + kRowBinMax ? kp : k + kRowBinMax) + 1) & ~1;
    auto lds = [&](int l) { return (int64_t)(p.filed_words + p.cap) * 8 + ((1 << l) + 4 + kRowMisc) * 4; };
    if (lds(lg) > kLdsBudgetWholeRow) p.cap = 0;
    while (lg > 10 && lds(lg) > kLdsBudgetWholeRow) --lg;
    if ((1 << lg) < T || lds(lg) > kLdsBudgetWholeRow) return false;
    p.lg_bins = lg;
    p.lds_bytes = (int)lds(lg);
    p.T = T;
    *out = p;
    return true;
}

// Several workgroups to a row.  false: the row is too long for that, or k too large.
bool plan_exact_parts(int64_t m, int64_t n, int64_t k, int dtype, bool ptr16, RowPlan *out) {
    const int ve = dtype == ATK_F32 ? 4 : 8;
    RowPlan p;
    memset(&p, 0, sizeof p);
    p.ve = ve;
    const int64_t n_vec = ptr16 && n % ve == 0 ? n / ve : (n + 2 * ve - 2) / ve;
    const PlanOverride &ov = plan_override();
    // Rows that one workgroup holds are shared out only where that gives CUs without a row something to do, down to 1024 vectors a part, from
    // 12288 vectors on (128 x 32768 f32, k = 64: 8.1 us in one workgroup, 10.5 in two).  Parts are the safer way, not the quicker one on every row: what
    // they pass on, and the row's last workgroup goes through alone, grows with k, but rows full of ties cost one workgroup its whole row again and
    // again.  65536 f32, in parts and in one workgroup: 128 rows, k = 1000: N(0,1) 16.5 and 11.8, averaged over neighbours 24.6 and 24.5, three levels
    // 24.2 and 27.4, constant 19.6 and 34.3, zeros but for one in 200 47.7 and 183; k = 3000 32.7 and 17.1, 33 and 32, 41 and 31, 35 and 32, 96 and
    // 197; 64 rows, k = 701: 16.0 and 10.7, 19.8 and 22.1, 22.8 and 26.9, 21.4 and 33.8, 47 and 181.
    // Longer rows take parts of up to 8192 vectors, two workgroups of 512 lanes to a CU.
    int64_t parts = std::min<int64_t>(std::min<int64_t>(kNumCU / m, 32), n_vec / 1024);
    if (parts < 1) parts = 1;
    if (n_vec <= 16 * 1024 && (2 * m > kNumCU || n_vec < 12288) && !ov.S) return false;
    if (ov.S) parts = ov.S;
    int64_t pv = (n_vec + parts - 1) / parts;
    int t_max = 1024;
    if (pv > 8192) {
        parts = (n_vec + 8191) / 8192;
        t_max = 512;
    }
    pv = (n_vec + parts - 1) / parts;
    parts = (n_vec + pv - 1) / pv;
    if (parts < 2 || parts > kWave || m * parts >= (1ll << 31)) return false;
    int T = kWave;  // (the last part may be some vectors shorter, and no wavefront should be without)
    while (T < t_max && 2 * T + kWave <= pv) T <<= 1;
    if (ov.T) T = ov.T;
    p.nv = row_nv((pv + T - 1) / T, false);
    if (!p.nv) return false;
    p.parts = (int)parts;
    p.part_vecs = (int)pv;
    // What a row's parts pass on is about half a MB at most, and no part passes on much of what it reads.
    if (parts * k > 65536 || (double)k > 0.2 * (double)((pv - parts) * ve)) return false;
    const double expect = row_bound_plan(p, T, pv, (double)k, 0.5);
    p.part_cap = (int)(expect * 1.25 + 8.0 * std::sqrt(expect) + 128.0);
    if (p.part_cap < k) p.part_cap = (int)k;
    p.cap = 4096;
    if ((double)parts * expect > 3500.0) {
        // (not on launches of more than two rounds of workgroups: what a row's last workgroup then does alone, where the row is unlike
        // itself along its length, is done by all of them in the sweeps of the digit-by-digit path: 128 x 2^20 f32, k = 1000, ascending
        // 580 us there, 950 here, first half -inf 430 and 510, without order 225 and 207)
        if (m * parts > 4 * kNumCU) return false;
        // The largest of the parts' upper bounds decides how many elements are left, so every part aims at k / parts and a margin
        const double want = 1.5 * (double)k / (double)parts + 3.0 * std::sqrt((double)k / (double)parts) + 3.0;
        p.rank_up = (int)std::ceil(want / (T / kWave));
        if (p.rank_up >= p.rank) p.rank_up = 0;
        const double up = p.rank_up ? (double)p.rank_up * (double)(T / kWave) * (expect / ((double)p.rank * (T / kWave))) : expect;
        p.cap = std::max(p.cap, ((int)(1.1 * (double)parts * up + 512.0) + 1) & ~1);
    }
    if (p.cap < p.part_cap) p.cap = (p.part_cap + 1) & ~1;
    if (p.cap > 16384 || exact_parts_data_bytes(p, m) > (1ll << 30)) return false;
    int lg = 8;
    while (lg < 13 && ((1 << lg) < 2 * k || (1 << lg) < T)) ++lg;
    int64_t kp = 1;
    while (kp < k) kp <<= 1;
    p.filed_words = (int)((kp > k + kRowBinMax ? kp : k + kRowBinMax) + 1) & ~1;
    p.lg_bins = lg;
    const int64_t lds = (int64_t)(p.filed_words + p.cap) * 8 + ((1 << lg) + 4 + kRowMisc) * 4;
    if (lds > kLdsBudgetWholeRow) return false;
    p.lds_bytes = (int)lds;
    p.T = T;
    *out = p;
    return true;
}
int64_t exact_parts_data_bytes(const RowPlan &p, int64_t m) { return m * p.parts * (32 + (int64_t)p.part_cap * 8); }
int64_t exact_parts_state_bytes(int64_t m) { return m * kTicketStride * 4; }

template <typename K>
static hipError_t launch_row(K kernel, const RowPlan &pl, const RowParams &prm, int64_t grid, bool (&told)[64], hipStream_t stream) {
    if (pl.lds_bytes > 64 * 1024) {
        const hipError_t e = allow_whole_cu_lds((const void *)kernel, told);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3((unsigned)pl.T), (size_t)pl.lds_bytes, stream, prm);
    return hipGetLastError();
}

template <int ELT>
static hipError_t launch_row_t(const RowPlan &pl, const RowParams &prm, int64_t m, hipStream_t stream) {
#define ATK_ROW(KERNEL, GRID)                                        \
    do {                                                             \
        static bool told[64] = {};                                   \
        return launch_row(KERNEL, pl, prm, GRID, told, stream);      \
    } while (0)
    if (prm.xi) {
        switch (pl.nv) {
            case 1: ATK_ROW((ex_row_kernel<ELT, 1, true>), m);
            case 2: ATK_ROW((ex_row_kernel<ELT, 2, true>), m);
            case 3: ATK_ROW((ex_row_kernel<ELT, 3, true>), m);
            case 4: ATK_ROW((ex_row_kernel<ELT, 4, true>), m);
        }
        return hipErrorInvalidValue;
    }
#define ATK_ROW_NV(NV)                                                       \
    case NV:                                                                 \
        if (pl.parts) ATK_ROW((ex_parts_kernel<ELT, NV>), m * pl.parts);     \
        ATK_ROW((ex_row_kernel<ELT, NV, false>), m);
    switch (pl.nv) {
        ATK_ROW_NV(1)
        ATK_ROW_NV(2)
        ATK_ROW_NV(3)
        ATK_ROW_NV(4)
        ATK_ROW_NV(6)
        ATK_ROW_NV(8)
        ATK_ROW_NV(12)
        ATK_ROW_NV(16)
    }
#undef ATK_ROW_NV
#undef ATK_ROW
    return hipErrorInvalidValue;
}

// state, data: of plans with several workgroups to a row, exact_parts_state_bytes() zeroed and exact_parts_data_bytes()
hipError_t launch_exact_row(const RowPlan &pl, int64_t m, int64_t n, int64_t k, int64_t idx_n, int dtype, const void *x,
                            const int32_t *xi, void *out_vals, int32_t *out_idx, void *state, void *data, hipStream_t stream) {
    RowParams prm;
    memset(&prm, 0, sizeof prm);
    prm.x = x;
    prm.xi = xi;
    prm.out_vals = out_vals;
    prm.out_idx = out_idx;
    prm.n = (int)n;
    prm.k = (int)k;
    prm.idx_bits = 1;
    while (((int64_t)1 << prm.idx_bits) < idx_n) ++prm.idx_bits;
    prm.lg_bins = pl.lg_bins;
    prm.filed_words = pl.filed_words;
    prm.cap = pl.cap;
    prm.sub = pl.sub;
    prm.rank = pl.rank;
    prm.parts = pl.parts;
    prm.part_vecs = pl.part_vecs;
    prm.part_cap = pl.part_cap;
    prm.rank_up = pl.rank_up;
    prm.heads = (u64 *)data;
    prm.lists = prm.heads + m * pl.parts * 4;
    prm.tickets = (uint32_t *)state;
    if (xi && (((uintptr_t)x | (uintptr_t)xi) & 15u)) return hipErrorInvalidValue;  // never: the pairs lie in the library's scratch
    if (pl.parts && (xi || !state || !data)) return hipErrorInvalidValue;
    // (a launch holds fewer than 2^32 lanes)
    const int64_t es = dtype == ATK_F32 ? 4 : 2, rows = pl.parts ? m : ((int64_t)1 << 31) / pl.T;
    for (int64_t r0 = 0; r0 < m; r0 += rows) {
        prm.x = (const unsigned char *)x + r0 * n * es;
        prm.xi = xi ? xi + r0 * n : nullptr;
        prm.out_vals = (unsigned char *)out_vals + r0 * k * es;
        prm.out_idx = out_idx + r0 * k;
        const int64_t now = std::min(rows, m - r0);
        const hipError_t e = dtype == ATK_F32 ? launch_row_t<ATK_F32>(pl, prm, now, stream) : launch_row_t<ATK_BF16>(pl, prm, now, stream);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace atk
