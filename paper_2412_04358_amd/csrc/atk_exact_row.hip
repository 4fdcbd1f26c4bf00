// exact_topk of rows that one workgroup holds in registers (and Stage 2 over more candidates than the fused kernels
// select from): one launch, one workgroup per row, the row read once.
//
//   1. Every lane loads its share of the row, 16 bytes per load, all loads in flight together.
//   2. A guess of a value that at least k elements reach: the smallest of the maxima of G groups of lanes (or of parts of a
//      lane's elements).  With the elements spread over the groups at random, about G ln G of them lie at or above it
//      (the coupon collector's count), so G is the smallest with half of that at k or more.  It is checked, not trusted.
//   3. A histogram of the elements from there on, over bins linear in (value key, index) between the guess and the row's
//      maximum; a descending prefix sum turns counts into places.  Fewer than k counted: again from -inf.  A bin too full
//      to be ranked by comparing its elements with one another: again from the lower edge of the bin that holds the
//      k-th, which is a range without what lies below (values around zero stretch a range of keys over every exponent).
//   4. The elements of the bins down to the k-th's go to LDS, bin by bin; each finds its rank as its bin's start plus
//      the larger elements of its bin.  Lanes side by side take places side by side, so the row is written nearly in order.
// Rows whose bins stay crowded (long runs of one value) are selected digit by digit (RadixSelect, Appendix D.2) and ordered
// by order_write(); they re-read the row, which is in the caches by then.
//
// What bounds it: with at most one row per CU, the rate at which one CU takes in a row (about 45 GB/s, measured: 256 KB in
// 5.8 us) and then the operations on every element; with many rows the latter, shared out over the workgroups of a CU.
// Measured against the launches this replaced (a histogram, a decision, a copy-out and a selection; one workgroup
// with the row in LDS for short rows): 2048 x 8192 bf16, k = 512: 79.7 -> 22.5 us; 64 x 128256 bf16, k = 256: 28.7 -> 19.1;
// 1024 x 65536 f32, k = 64: 106 -> 72; 128 x 65536 f32, k = 16384: 148 -> 57; one row of 65536 f32, k = 4096: 120 -> 31;
// 2048 x 2048 f32, k = 64: 43 -> 10.4; 128 lists of 8192 pairs, k = 4096 (Stage 2): 118 -> 12.4.
#include <cmath>
#include <cstring>

#include "atk_common.h"
#include "atk_exact.h"
#include "atk_select.h"

namespace atk {

struct RowParams {
    const void *x;
    const int32_t *xi;    // NULL, or the column index each element stands for
    void *out_vals;
    int32_t *out_idx;
    int n, k, idx_bits;
    int lg_bins, filed_words;
    int cap;              // elements at or above the guess that LDS holds in passing (0: they stay in the registers)
    int sub, gl;          // groups of the guess: sub > 1 parts of a lane's elements each, else gl lanes side by side
};

typedef uint32_t row_v4u __attribute__((ext_vector_type(4)));

// Bins linear in the order key (ties: in the index) between two keys.  d grows with the composite: the value key relative
// to the lower end without the low bits that bf16 leaves constant, then as many index bits as 32 bits have room for.
struct RowBins {
    uint32_t k_min, scale;
    int n_bins, s_idx, r_idx;
    uint32_t i_mask;
    float inv_scale;
    template <int ELT>
    __device__ __forceinline__ void set(uint32_t lo, uint32_t hi, int idx_bits, int bins) {
        constexpr int tz = (ELT == ATK_BF16) ? 16 : 0;
        k_min = lo;
        n_bins = bins;
        const uint32_t span = (hi - lo) >> tz;
        const int span_bits = span ? 32 - __builtin_clz(span) : 0;
        s_idx = 32 - span_bits < idx_bits ? 32 - span_bits : idx_bits;
        r_idx = idx_bits - s_idx;
        i_mask = idx_bits >= 31 ? 0x7fffffffu : ((1u << idx_bits) - 1u);
        const uint32_t d_max = (uint32_t)((((u64)span + 1ull) << s_idx) - 1ull);  // < 2^32: span < 2^span_bits, s_idx <= 32 - span_bits
        const float d1 = (float)d_max + 1.0f;
        // a little under bins * 2^32 / (d_max + 1): the conversion's rounding must not push the largest d past the last bin
        const float s = ((float)bins * 4294967296.0f / d1) * 0.999999f;
        scale = s >= 4294967040.0f ? 0xffffffffu : (uint32_t)s;
        inv_scale = 4294967296.0f / (float)scale;
    }
    // key >= k_min; inv_idx: 0x7fffffff - index
    template <int ELT>
    __device__ __forceinline__ uint32_t bin(uint32_t key, uint32_t inv_idx) const {
        constexpr int tz = (ELT == ATK_BF16) ? 16 : 0;
        uint32_t d = (key - k_min) >> tz;
        d = s_idx >= 32 ? 0u : (d << s_idx);
        d |= (inv_idx & i_mask) >> r_idx;
        const uint32_t b = __umulhi(d, scale);
        return b < (uint32_t)n_bins ? b : (uint32_t)n_bins - 1u;  // (only a NaN's key lies past the last bin)
    }
    // a key at or a little below the lowest of bin b
    template <int ELT>
    __device__ __forceinline__ uint32_t edge(uint32_t b) const {
        constexpr int tz = (ELT == ATK_BF16) ? 16 : 0;
        float d = (float)b * inv_scale;
        d = d - d * 4.0e-7f - 2.0f;
        if (!(d > 0.0f)) return k_min;
        const uint32_t di = d >= 4294967040.0f ? 0xffffff00u : (uint32_t)d;
        return k_min + ((s_idx >= 32 ? 0u : (di >> s_idx)) << tz);
    }
};

// LDS words behind the bins: [0] bin of the need-th largest, [1] elements in higher bins, [2] its elements, [3] all counted,
// [4] crowded, [5] cursor, [8..24) and [24..40) per-wavefront words
constexpr int kRowMisc = 40;

// Counts cur[0 .. n_bins) -> elements in higher bins, in place; finds the bin of the need-th largest.  n_bins is a power
// of two and at least the workgroup's size, which is one too.  Called by the whole workgroup after a barrier; ends in one.
__device__ __forceinline__ void row_scan(uint32_t *cur, uint32_t *misc, int n_bins, uint32_t need) {
    const int tid = threadIdx.x, T = blockDim.x, lane = tid & (kWave - 1), n_waves = T >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = n_bins / T, hi = n_bins - 1 - tid * q;  // this lane's bins: hi, hi - 1, ... hi - q + 1
    uint32_t s = 0;
    for (int j = 0; j < q; ++j) s += cur[hi - j];
    const uint32_t incl = wave_incl_scan_u32(s);
    if (lane == kWave - 1) misc[8 + wave] = incl;
    if (tid == 0) misc[4] = 0u;
    __syncthreads();
    const uint32_t tot = (lane < n_waves) ? misc[8 + lane] : 0u;
    const uint32_t tot_incl = wave_incl_scan_u32(tot);
    uint32_t run = incl - s;
    if (wave > 0) run += (uint32_t)__builtin_amdgcn_readlane((int)tot_incl, wave - 1);
    bool crowded = false;
    for (int j = 0; j < q; ++j) {
        const uint32_t v = cur[hi - j];
        cur[hi - j] = run;
        if (run < need) {
            crowded = crowded || v > (uint32_t)kRowBinMax;
            if (run + v >= need) {
                misc[0] = (uint32_t)(hi - j);
                misc[1] = run;
                misc[2] = v;
            }
        }
        run += v;
    }
    if (crowded) misc[4] = 1u;
    if (tid == T - 1) misc[3] = run;
    __syncthreads();
}

template <int ELT>
__device__ __forceinline__ u64 row_composite(const RowParams &p, int64_t r, int i) {
    const uint32_t bits = (ELT == ATK_F32) ? ((const uint32_t *)p.x)[r * p.n + i] : ((uint32_t)((const uint16_t *)p.x)[r * p.n + i]) << 16;
    return make_composite(bits, p.xi ? p.xi[r * p.n + i] : i);
}

// Digit by digit over the row, most significant first, on the composite without the bits that carry nothing (the low 16
// of a bf16 key, the index bits above idx_bits); the k survivors are then put in order.
template <int ELT>
__device__ __forceinline__ void row_by_digits(const RowParams &p, int64_t r, u64 *filed, uint32_t *cur, uint32_t *misc) {
    const int tid = threadIdx.x, T = blockDim.x, lane = tid & (kWave - 1);
    const int drop = ELT == ATK_BF16 ? 16 : 0, keep = p.idx_bits + 1;
    auto squeeze = [&](u64 c) { return ((c >> (32 + drop)) << keep) | (c & ((1ull << keep) - 1ull)); };
    const int n_bins = 1 << p.lg_bins;
    int top = 32 - drop + keep;  // bits still open
    u64 prefix = 0ull;
    uint32_t need = (uint32_t)p.k;
    for (;;) {
        const int w = top < p.lg_bins ? top : p.lg_bins;
        const int shift = top - w;
        const u64 hi_mask = top >= 64 ? 0ull : (~0ull << top);
        for (int i = tid; i < n_bins; i += T) cur[i] = 0u;
        __syncthreads();
        for (int i = tid; i < p.n; i += T) {
            const u64 q = squeeze(row_composite<ELT>(p, r, i));
            if ((q & hi_mask) == prefix) atomicAdd(&cur[(uint32_t)(q >> shift) & ((1u << w) - 1u)], 1u);
        }
        __syncthreads();
        row_scan(cur, misc, n_bins, need);
        prefix |= (u64)misc[0] << shift;
        need -= misc[1];
        const bool done = misc[2] == need || shift == 0;
        __syncthreads();  // misc and cur are written again
        if (done) break;
        top = shift;
    }
    if (tid == 0) misc[5] = 0u;
    for (int i = tid; i < kRankMax; i += T) cur[i] = 0u;
    __syncthreads();
    for (int i0 = 0; i0 < p.n; i0 += T) {
        const int i = i0 + tid;
        const u64 c = i < p.n ? row_composite<ELT>(p, r, i) : 0ull;
        const bool take = i < p.n && squeeze(c) >= prefix;
        const u64 mask = __ballot(take);
        if (mask) {  // uniform over the wavefront
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&misc[5], (uint32_t)__popcll(mask));
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) +
                 __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            if (take && at < (uint32_t)p.k) filed[at] = c;
        }
    }
    __syncthreads();
    order_write<ELT>(filed, p.k, cur, p.out_vals, p.out_idx, r);
}

template <int ELT, int NV, bool XI>
__global__ void __launch_bounds__(1024) ex_row_kernel(RowParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int ES = (ELT == ATK_F32) ? 4 : 2, VE = 16 / ES;
    const int tid = threadIdx.x, T = blockDim.x, lane = tid & (kWave - 1), n_waves = T >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t r = blockIdx.x;
    const int n_bins = 1 << p.lg_bins;
    u64 *filed = (u64 *)smem;
    uint32_t *cur = (uint32_t *)(filed + p.filed_words);  // [n_bins], then a zero: nothing lies above the last bin
    uint32_t *misc = cur + n_bins + 4;

    // ---- the row, from the 16-byte boundary at or before its first element to the one at or after its last (no vector
    // without an element of the row is read); elements of the neighbours become NaN, which no comparison below lets through
    const uintptr_t addr = (uintptr_t)p.x + (uintptr_t)(r * p.n) * ES;
    const int rot = (int)(addr & 15) / ES, end = rot + p.n;
    const int n_vec = (end + VE - 1) / VE;
    const row_v4u *row = (const row_v4u *)(addr & ~(uintptr_t)15);
    row_v4u q[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int v = tid + j * T;
        q[j] = __builtin_nontemporal_load(row + (v < n_vec ? v : 0));
    }
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
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int v = tid + j * T;
        if (v >= n_vec) {
            const row_v4u none = {0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu};
            q[j] = none;
        } else if (v == 0 || v == n_vec - 1) {
#pragma unroll
            for (int e = 0; e < VE; ++e) {
                const int at = v * VE + e;
                if (at < rot || at >= end) {
                    if (ELT == ATK_F32)
                        q[j][e] = 0xffffffffu;
                    else
                        q[j][e >> 1] |= (e & 1) ? 0xffff0000u : 0x0000ffffu;
                }
            }
        }
    }

    // ---- the guess: maxima of groups
    constexpr int SM = NV * 4 < 8 ? 4 : 8;
    float mx[SM];
#pragma unroll
    for (int i = 0; i < SM; ++i) mx[i] = __uint_as_float(0x7fc00000u);
#pragma unroll
    for (int w = 0; w < NV * 4; ++w) {
        const uint32_t a = q[w >> 2][w & 3];
        const float f = ELT == ATK_F32 ? __uint_as_float(a) : fmaxf(__uint_as_float(a << 16), __uint_as_float(a & 0xffff0000u));
        mx[w % SM] = fmaxf(mx[w % SM], f);  // (the number where one of the two is NaN)
    }
    auto key_of = [](float f) { return f == f ? ukey_of_bits(__float_as_uint(f)) : 0u; };
    uint32_t k_min = 0xffffffffu, k_max;
    {
        if (SM > 4 && p.sub <= 4) {
#pragma unroll
            for (int i = 0; i < SM / 2; ++i) mx[i] = fmaxf(mx[i], mx[i + SM / 2]);
        }
        if (p.sub <= 2) {
            mx[0] = fmaxf(mx[0], mx[2]);
            mx[1] = fmaxf(mx[1], mx[3]);
        }
        if (p.sub <= 1) mx[0] = fmaxf(mx[0], mx[1]);
        float m = mx[0];
        if (p.sub > 1) {
#pragma unroll
            for (int i = 0; i < SM; ++i)
                if (i < p.sub) {
                    const uint32_t key = key_of(mx[i]);
                    k_min = key && key < k_min ? key : k_min;
                    m = fmaxf(m, mx[i]);
                }
            k_max = key_of(m);
        } else {
            k_max = key_of(m);
            uint32_t g = k_max;
            if (p.gl >= 2) g = max(g, dpp_u32<0xB1>(g));
            if (p.gl >= 4) g = max(g, dpp_u32<0x4E>(g));
            if (p.gl >= 8) g = max(g, dpp_u32<0x141>(g));
            if (p.gl >= 16) g = max(g, dpp_u32<0x140>(g));
            if (p.gl >= 64) g = wave_max_u32(g);
            k_min = g ? g : 0xffffffffu;
        }
    }
    k_min = wave_min_u32(k_min);
    k_max = wave_max_u32(k_max);
    if (lane == 0) {
        misc[8 + wave] = k_min;
        misc[24 + wave] = k_max;
    }
    __syncthreads();
    k_min = wave_min_u32(lane < n_waves ? misc[8 + lane] : 0xffffffffu);
    k_max = wave_max_u32(lane < n_waves ? misc[24 + lane] : 0u);
    if (k_min > k_max) k_min = k_max;
    __syncthreads();  // (the words are used again by the scan)

    // f(value, column index) for every element of this lane.  The words pass through an empty asm statement: else what is
    // worked out from them (order keys, indices, comparisons) is kept in registers from one pass to the next, and spills.
    auto each = [&](auto f) {
        int i0 = tid * VE - rot;
        asm volatile("" : "+v"(i0));
#pragma unroll
        for (int j = 0; j < NV; ++j)
#pragma unroll
            for (int e = 0; e < VE; ++e) {
                if ((ELT == ATK_F32 || (e & 1) == 0)) asm volatile("" : "+v"(q[j][ELT == ATK_F32 ? e : (e >> 1)]));
                const uint32_t a = q[j][ELT == ATK_F32 ? e : (e >> 1)];
                const uint32_t bits = ELT == ATK_F32 ? a : ((e & 1) ? (a & 0xffff0000u) : (a << 16));
                f(bits, XI ? xi[j * VE + e] : i0 + j * T * VE + e);
            }
    };
    RowBins bins;
    float v_lo;
    uint32_t tb;  // bin of the k-th largest
    bool in_lds = false;
    int2 *passed = (int2 *)(misc + kRowMisc);
    uint32_t n_passed = 0;
    int attempt = 0;
    if (p.cap) {
        // few of the elements reach the guess: they go to LDS (value bits, index) side by side, and the histogram and the
        // filing, a dozen operations and an LDS atomic per element each, run over them instead of over all registers with
        // most lanes idle (2048 x 8192 bf16, k = 512: 29.7 -> 23.9 us; 2048 x 32768 bf16, k = 256: 68.9 -> 56.5)
        v_lo = __uint_as_float(bits_of_ukey(k_min));
        uint32_t cnt = 0;
        each([&](uint32_t bits, int) { cnt += __uint_as_float(bits) >= v_lo ? 1u : 0u; });
        const uint32_t incl = wave_incl_scan_u32(cnt);
        uint32_t at = 0;
        if (lane == kWave - 1) at = atomicAdd(&misc[5], incl);
        at = (uint32_t)__builtin_amdgcn_readlane((int)at, kWave - 1) + incl - cnt;
        each([&](uint32_t bits, int idx) {
            if (__uint_as_float(bits) >= v_lo) {
                if (at < (uint32_t)p.cap) passed[at] = make_int2((int)bits, idx);
                ++at;
            }
        });
        __syncthreads();
        n_passed = misc[5];
        if (n_passed >= (uint32_t)p.k && n_passed <= (uint32_t)p.cap) {
            bins.template set<ELT>(k_min, k_max, p.idx_bits, n_bins);
            for (uint32_t i = tid; i < n_passed; i += T) {
                const int2 w = passed[i];
                atomicAdd(&cur[bins.template bin<ELT>(ukey_of_bits((uint32_t)w.x), 0x7fffffffu - (uint32_t)w.y)], 1u);
            }
            __syncthreads();
            row_scan(cur, misc, n_bins, (uint32_t)p.k);
            in_lds = misc[4] == 0u;
            if (!in_lds) {
                const uint32_t lo = bins.template edge<ELT>(misc[0]);
                if (lo > k_min) k_min = lo;
                attempt = 1;
                __syncthreads();
                for (int i = tid; i < n_bins; i += T) cur[i] = 0u;
                __syncthreads();
            }
        }
    }
    for (; !in_lds; ++attempt) {
        bins.template set<ELT>(k_min, k_max, p.idx_bits, n_bins);
        v_lo = __uint_as_float(bits_of_ukey(k_min));
        each([&](uint32_t bits, int idx) {
            if (__uint_as_float(bits) >= v_lo) atomicAdd(&cur[bins.template bin<ELT>(ukey_of_bits(bits), 0x7fffffffu - (uint32_t)idx)], 1u);
        });
        __syncthreads();
        row_scan(cur, misc, n_bins, (uint32_t)p.k);
        const bool few = misc[3] < (uint32_t)p.k, crowded = misc[4] != 0u;
        if (!few && !crowded) break;
        const uint32_t lo = few ? 0x007fffffu : bins.template edge<ELT>(misc[0]);  // (-inf's key)
        // (twice from a raised lower end at most, and once from -inf)
        if (attempt == 3 || (few ? k_min <= lo : lo <= k_min)) {
            __syncthreads();
            row_by_digits<ELT>(p, r, filed, cur, misc);
            return;
        }
        k_min = lo;
        __syncthreads();
        for (int i = tid; i < n_bins; i += T) cur[i] = 0u;
        __syncthreads();
    }

    // ---- the winners' bins, brought together; cur[b] ends as the place behind bin b, which is where bin b - 1 starts
    tb = misc[0];
    if (in_lds) {
        for (uint32_t i = tid; i < n_passed; i += T) {
            const int2 w = passed[i];
            const uint32_t b = bins.template bin<ELT>(ukey_of_bits((uint32_t)w.x), 0x7fffffffu - (uint32_t)w.y);
            if (b >= tb) filed[atomicAdd(&cur[b], 1u)] = make_composite((uint32_t)w.x, w.y);
        }
    } else {
        v_lo = __uint_as_float(bits_of_ukey(bins.template edge<ELT>(tb)));
        each([&](uint32_t bits, int idx) {
            if (__uint_as_float(bits) >= v_lo) {
                const uint32_t b = bins.template bin<ELT>(ukey_of_bits(bits), 0x7fffffffu - (uint32_t)idx);
                if (b >= tb) filed[atomicAdd(&cur[b], 1u)] = make_composite(bits, idx);
            }
        });
    }
    __syncthreads();
    const int filed_n = (int)cur[tb];
    for (int i = tid; i < filed_n; i += T) {
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

// ------------------------------------------------------------------------------------ host
static int row_nv(int64_t want, bool pairs) {  // vectors per lane of the smallest instance that holds `want`, 0: none
    static const int have[] = {1, 2, 3, 4, 6, 8, 12, 16};
    for (int v : have)
        if (v >= want) return (pairs && v > 4) ? 0 : v;
    return 0;
}

bool plan_exact_row(int64_t m, int64_t n, int64_t k, int dtype, bool pairs, bool ptr16, RowPlan *out) {
    const int ve = dtype == ATK_F32 ? 4 : 8;
    RowPlan p;
    memset(&p, 0, sizeof p);
    if (k > kRowMaxK || n > (int64_t)1024 * 16 * ve) return false;
    // vectors that hold an element of a row (rows off the 16-byte boundaries: with the worst alignment)
    const int64_t n_vec = ptr16 && n % ve == 0 ? n / ve : (n + 2 * ve - 2) / ve;
    // At most one row per CU: the biggest workgroup that still has a vector per lane.  More rows: several workgroups to a
    // CU, so that one reads while others select, each with 4 to 8 vectors per lane (2048 rows: 8192 f32, k = 64: 21.1 us with
    // 256 lanes, 40.3 with 1024; 2048 f32: 10.4 with 128, 14.4 with 512; 32768 bf16, k = 256: 53.9 with 512, 69.0 with 1024), and
    // twice the lanes where a quarter of the row or more is kept, which the tables in LDS leave room for no more than a few
    // of at a time (8192 f32, k = 2048: 78.5 with 256, 63.0 with 512), or where only some CUs get a second row
    // (300 rows of 4096 f32: 7.4 with 256, 6.8 with 512).
    int T = kWave;
    if (m <= kNumCU) {
        while (T < 1024 && T < n_vec) T <<= 1;
    } else {
        T = n_vec <= 512 ? 128 : (n_vec <= 2048 ? 256 : (n_vec <= 8192 ? 512 : 1024));
        if ((4 * k >= n || m <= 2 * kNumCU) && T * 2 <= n_vec && T < 512) T *= 2;
        while (T > kWave && T / 2 >= n_vec) T >>= 1;
    }
    if (plan_override().T) T = plan_override().T;
    p.nv = row_nv((n_vec + T - 1) / T, pairs);
    while (!p.nv && T < 1024) {
        T <<= 1;
        p.nv = row_nv((n_vec + T - 1) / T, pairs);
    }
    if (!p.nv) return false;
    // groups of the guess: the fewest G with G ln G / 2 >= k
    p.sub = 1;
    p.gl = 1;
    auto enough = [&](double g) { return g > 1.0 && 0.5 * g * std::log(g) >= (double)k; };
    const int lanes = (int)(n_vec < T ? n_vec : T);
    static const int gls[] = {64, 16, 8, 4, 2, 1};
    double groups = 0.0;
    for (int g : gls)
        if (enough((double)(lanes / g))) {
            p.gl = g;
            groups = lanes / g;
            break;
        }
    if (groups == 0.0) {
        const int sm = p.nv * 4 < 8 ? 4 : 8;
        for (p.sub = 2; p.sub < sm && !enough((double)lanes * p.sub);) p.sub *= 2;
        groups = (double)lanes * p.sub;
    }
    // How many elements reach the guess: G (ln G + 0.58) on average, more than G (ln G + c) on one row in e^c (which then
    // stays in the registers, at twice the time: rarer still where a launch is one round of rows and waits for its slowest).
    // Where that is a small part of the row they pass through LDS.
    const double expect = groups * (std::log(groups) + (m <= kNumCU ? 9.0 : 7.0));
    p.cap = expect * 2.0 < (double)n && expect < 8192.0 ? ((int)expect + 1) & ~1 : 0;
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

template <int ELT, int NV, bool XI>
static hipError_t launch_row(const RowPlan &pl, const RowParams &prm, int64_t m, hipStream_t stream) {
    if (pl.lds_bytes > 64 * 1024) {
        static bool told[64] = {};
        const hipError_t e = allow_whole_cu_lds((const void *)ex_row_kernel<ELT, NV, XI>, told);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((ex_row_kernel<ELT, NV, XI>), dim3((unsigned)m), dim3((unsigned)pl.T), (size_t)pl.lds_bytes, stream, prm);
    return hipGetLastError();
}

template <int ELT>
static hipError_t launch_row_t(const RowPlan &pl, const RowParams &prm, int64_t m, hipStream_t stream) {
    if (prm.xi) {
        switch (pl.nv) {
            case 1: return launch_row<ELT, 1, true>(pl, prm, m, stream);
            case 2: return launch_row<ELT, 2, true>(pl, prm, m, stream);
            case 3: return launch_row<ELT, 3, true>(pl, prm, m, stream);
            case 4: return launch_row<ELT, 4, true>(pl, prm, m, stream);
        }
        return hipErrorInvalidValue;
    }
    switch (pl.nv) {
        case 1: return launch_row<ELT, 1, false>(pl, prm, m, stream);
        case 2: return launch_row<ELT, 2, false>(pl, prm, m, stream);
        case 3: return launch_row<ELT, 3, false>(pl, prm, m, stream);
        case 4: return launch_row<ELT, 4, false>(pl, prm, m, stream);
        case 6: return launch_row<ELT, 6, false>(pl, prm, m, stream);
        case 8: return launch_row<ELT, 8, false>(pl, prm, m, stream);
        case 12: return launch_row<ELT, 12, false>(pl, prm, m, stream);
        case 16: return launch_row<ELT, 16, false>(pl, prm, m, stream);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_exact_row(const RowPlan &pl, int64_t m, int64_t n, int64_t k, int64_t idx_n, int dtype, const void *x,
                            const int32_t *xi, void *out_vals, int32_t *out_idx, hipStream_t stream) {
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
    prm.gl = pl.gl;
    if (xi && (((uintptr_t)x | (uintptr_t)xi) & 15u)) return hipErrorInvalidValue;  // never: the pairs lie in the library's scratch
    return dtype == ATK_F32 ? launch_row_t<ATK_F32>(pl, prm, m, stream) : launch_row_t<ATK_BF16>(pl, prm, m, stream);
}

}  // namespace atk
