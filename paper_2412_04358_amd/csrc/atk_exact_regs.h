// Device code that exact_topk's row kernels share: a row or a part of one in a workgroup's registers, bins linear in the order of
// the elements, and the prefix sum that turns their counts into places.  What it is for: atk_exact_row.hip.
#pragma once

#include <type_traits>

#include "atk_common.h"
#include "atk_exact.h"
#include "atk_row_bins.h"
#include "atk_select.h"

namespace atk {

struct RowParams {
    const void *x;
    const int32_t *xi;    // NULL, or the column index each element stands for
    void *out_vals;
    int32_t *out_idx;
    int n, k, idx_bits;
    int lg_bins, filed_words;
    int cap;              // elements at or above the bound that LDS holds in passing (0: they stay in the registers)
    int sub, rank;        // the bound: the rank-th largest of 64 * sub maxima in every wavefront
    // several workgroups to a row
    int parts, part_vecs;   // workgroups per row, 16-byte vectors of the row that each reads
    int part_cap;           // elements that each passes on
    u64 *lists;             // [row][part][part_cap] composites
    u64 *heads;             // [row][part][2]: (bound << 32 | elements passed on), the part's largest key
    uint32_t *tickets;      // one per row, kTicketStride apart, zero between calls
};

typedef uint32_t row_v4u __attribute__((ext_vector_type(4)));

// LDS words behind the bins: [0] bin of the need-th largest, [1] elements in higher bins, [2] its elements, [3] all counted,
// [4] crowded, [5] cursor, [8..24) and [24..40) per-wavefront words
constexpr int kRowMisc = 40;

// Counts cur[0 .. n_bins) -> elements in higher bins, in place; finds the bin of the need-th largest.  n_bins is a power
// of two and at least the workgroup's size, which is one too; cur lies on a 16-byte boundary.  Called by the whole workgroup after a barrier; ends in one.
__device__ __forceinline__ void row_scan(uint32_t *cur, uint32_t *misc, int n_bins, uint32_t need) {
    const int tid = threadIdx.x, T = blockDim.x, lane = tid & (kWave - 1), n_waves = T >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = n_bins / T, hi = n_bins - 1 - tid * q;  // this lane's bins: hi, hi - 1, ... hi - q + 1
    uint32_t s = 0;
    if (q >= 4) {  // (four bins per read: lanes four and more words apart share their banks' turns)
        for (int j = 0; j < q; j += 4) {
            const uint4 v = *(const uint4 *)&cur[hi - j - 3];
            s += v.x + v.y + v.z + v.w;
        }
    } else {
        for (int j = 0; j < q; ++j) s += cur[hi - j];
    }
    const uint32_t incl = wave_incl_scan_u32(s);
    if (lane == kWave - 1) misc[8 + wave] = incl;
    if (tid == 0) misc[4] = 0u;
    __syncthreads();
    const uint32_t tot = (lane < n_waves) ? misc[8 + lane] : 0u;
    const uint32_t tot_incl = wave_incl_scan_u32(tot);
    uint32_t run = incl - s;
    if (wave > 0) run += (uint32_t)__builtin_amdgcn_readlane((int)tot_incl, wave - 1);
    bool crowded = false;
    auto step = [&](int b, uint32_t v) {  // returns the elements above bin b
        const uint32_t above = run;
        if (run < need) {
            crowded = crowded || v > (uint32_t)kRowBinMax;
            if (run + v >= need) {
                misc[0] = (uint32_t)b;
                misc[1] = run;
                misc[2] = v;
            }
        }
        run += v;
        return above;
    };
    if (q >= 4) {
        for (int j = 0; j < q; j += 4) {
            uint4 v = *(const uint4 *)&cur[hi - j - 3];
            v.w = step(hi - j, v.w);
            v.z = step(hi - j - 1, v.z);
            v.y = step(hi - j - 2, v.y);
            v.x = step(hi - j - 3, v.x);
            *(uint4 *)&cur[hi - j - 3] = v;
        }
    } else {
        for (int j = 0; j < q; ++j) cur[hi - j] = step(hi - j, cur[hi - j]);
    }
    if (crowded) misc[4] = 1u;
    if (tid == T - 1) misc[3] = run;
    __syncthreads();
}

// ---- a row, or a part of one, in the registers of a workgroup: lane t holds the vectors v0 + t, v0 + t + T, ... below v1
template <int ELT, int NV>
struct RowRegs {
    static constexpr int ES = (ELT == ATK_F32) ? 4 : 2, VE = 16 / ES, E = NV * VE;
    row_v4u q[NV];
    int i0;  // row position of the lane's first element

    // The row from the 16-byte boundary at or before its first element to the one at or after its last (no vector without an
    // element of the row is read); elements of the neighbours become NaN, which no comparison below lets through.
    __device__ __forceinline__ void load(const RowParams &p, int64_t r, int v0, int v1, int rot) {
        const int tid = threadIdx.x, T = blockDim.x;
        const uintptr_t addr = (uintptr_t)p.x + (uintptr_t)(r * p.n) * ES;
        const row_v4u *row = (const row_v4u *)(addr & ~(uintptr_t)15);
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int v = v0 + tid + j * T;
            q[j] = row[v < v1 ? v : v0];
        }
        i0 = (v0 + tid) * VE - rot;
    }
    __device__ __forceinline__ void mask_ends(const RowParams &p, int v0, int v1, int rot) {
        const int tid = threadIdx.x, T = blockDim.x;
        const int end = rot + p.n, last = (end - 1) / VE;
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int v = v0 + tid + j * T;
            if (v >= v1) {
                const row_v4u none = {0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu};
                q[j] = none;
            } else if (v == 0 || v == last) {
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
    }

    // f(value bits, position in the row, element number) for every element of this lane.  The words pass through an empty
    // asm statement: else what is worked out from them (order keys, positions, comparisons) is kept in registers from one
    // pass over the elements to the next, and spills.
    template <typename F>
    __device__ __forceinline__ void each(F f) {
        const int T = blockDim.x;
        int at = i0;
        asm volatile("" : "+v"(at));
#pragma unroll
        for (int j = 0; j < NV; ++j)
#pragma unroll
            for (int e = 0; e < VE; ++e) {
                if (ELT == ATK_F32 || (e & 1) == 0) asm volatile("" : "+v"(q[j][ELT == ATK_F32 ? e : (e >> 1)]));
                const uint32_t a = q[j][ELT == ATK_F32 ? e : (e >> 1)];
                f(ELT == ATK_F32 ? a : ((e & 1) ? (a & 0xffff0000u) : (a << 16)), at + j * T * VE + e, j * VE + e);
            }
    }

    // A lower bound: every wavefront's `rank`-th largest of the maxima of its groups - the smallest of these over the wavefronts is
    // reached by rank elements in each of them (and the largest element).  sub (1, 2, 4 or 8) groups per lane.  Where a wavefront has
    // fewer elements than that the bound is the lowest key there is.  rank 0: the smallest of the maxima.  Called by the whole workgroup; two barriers.
    // FIRST: the groups are the lane's first eight elements, one each (the largest element then is theirs, too).
    template <bool FIRST = false>
    __device__ __forceinline__ void bound(int sub, int rank, uint32_t *misc, uint32_t &k_min, uint32_t &k_max) {
        const int tid = threadIdx.x, lane = tid & (kWave - 1), n_waves = blockDim.x >> 6;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        constexpr int SM = NV * 4 < 8 ? 4 : 8;
        float mx[SM];
#pragma unroll
        for (int i = 0; i < SM; ++i) mx[i] = __uint_as_float(0x7fc00000u);
#pragma unroll
        for (int w = 0; w < NV * 4; ++w) {
            if (FIRST) break;
            const uint32_t a = q[w >> 2][w & 3];
            const float f = ELT == ATK_F32 ? __uint_as_float(a) : fmaxf(__uint_as_float(a << 16), __uint_as_float(a & 0xffff0000u));
            mx[w % SM] = fmaxf(mx[w % SM], f);  // (the number where one of the two is NaN)
        }
        if constexpr (FIRST) {
            static_assert(!FIRST || (SM == 8 && E >= 8), "eight elements");
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t a = ELT == ATK_F32 ? q[i >> 2][i & 3] : q[0][i >> 1];
                mx[i] = __uint_as_float(ELT == ATK_F32 ? a : ((i & 1) ? (a & 0xffff0000u) : (a << 16)));
            }
        }
        auto key_of = [](float f) { return f == f ? ukey_of_bits(__float_as_uint(f)) : 0u; };
        // The rank-th largest of the S * 64 keys of a wavefront, to its highest 16 bits (the bits below stay zero, which
        // can only lower the bound, by under one part in 128): bit by bit from the top, counting the keys that agree so far.
        auto nth = [&](auto s_tag) {
            constexpr int S = decltype(s_tag)::value;
            uint32_t key[S];
            uint32_t top = 0u;
#pragma unroll
            for (int i = 0; i < S; ++i) {
                float m = mx[i];
#pragma unroll
                for (int j = i + S; j < SM; j += S) m = fmaxf(m, mx[j]);
                key[i] = key_of(m);
                top = max(top, key[i]);
            }
            k_max = top;
            if (rank == 0) {
                k_min = 0xffffffffu;
#pragma unroll
                for (int i = 0; i < S; ++i) k_min = key[i] && key[i] < k_min ? key[i] : k_min;
                k_min = wave_min_u32(k_min);
                return;
            }
            uint32_t have = 0u;
#pragma unroll
            for (int bit = 31; bit >= 16; --bit) {
                const uint32_t want = have | (1u << bit);
                int cnt = 0;
#pragma unroll
                for (int i = 0; i < S; ++i) cnt += __popcll(__ballot(key[i] >= want));
                if (cnt >= rank) have = want;
            }
            k_min = have;
        };
        if (sub == 1)
            nth(std::integral_constant<int, 1>());
        else if (sub == 2)
            nth(std::integral_constant<int, 2>());
        else if (sub == 4 || SM == 4)
            nth(std::integral_constant<int, 4>());
        else
            nth(std::integral_constant<int, SM>());
        k_max = wave_max_u32(k_max);
        if (lane == 0) {
            misc[8 + wave] = k_min;
            misc[24 + wave] = k_max;
        }
        __syncthreads();
        k_min = wave_min_u32(lane < n_waves ? misc[8 + lane] : 0xffffffffu);
        k_max = wave_max_u32(lane < n_waves ? misc[24 + lane] : 0u);
        if (k_min < 0x007fffffu) k_min = 0x007fffffu;  // (-inf's)
        if (k_min > k_max) k_min = k_max;
        __syncthreads();  // (the words are used again)
    }

    // Positions of the elements at or above v_lo to list[0 .. ] (at most cap of them); the cursor *count starts from zero and
    // ends as their number.  Two operations per element set a bit each - a comparison and an addition of the mask
    // to itself with the comparison as carry -, the few that are set are then taken one by one: storing an element under
    // its own condition costs every element the six or so operations of a branch that few of the lanes take
    // (64 x 128256 bf16, k = 256: 8.2 us of the kernel's 18).  Called by the whole workgroup; ends in a barrier.
    __device__ __forceinline__ void list_from(float v_lo, int2 *list, uint32_t cap, uint32_t *count) {
        const int lane = threadIdx.x & (kWave - 1), T = blockDim.x;
        constexpr int M = (E + 31) / 32;  // masks of 32 elements, the last perhaps of fewer
        uint32_t mk[M];
#pragma unroll
        for (int w = 0; w < M; ++w) mk[w] = 0u;
        each([&](uint32_t bits, int, int en) {
            asm volatile("v_cmp_le_f32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(mk[en / 32]) : "v"(v_lo), "v"(bits) : "vcc");
        });
        uint32_t cnt = 0;
#pragma unroll
        for (int w = 0; w < M; ++w) cnt += (uint32_t)__popc(mk[w]);
        const uint32_t incl = wave_incl_scan_u32(cnt);
        uint32_t at = 0;
        if (lane == kWave - 1) at = atomicAdd(count, incl);
        at = (uint32_t)__builtin_amdgcn_readlane((int)at, kWave - 1) + incl - cnt;
#pragma unroll
        for (int w = 0; w < M; ++w) {
            uint32_t b = mk[w] << (32 - (E - 32 * w < 32 ? E - 32 * w : 32));  // the first element's bit is bit 31
            while (b) {
                const int t = __clz((int)b), en = w * 32 + t;
                b &= ~(0x80000000u >> t);
                if (at < cap) list[at].y = i0 + (en / VE) * T * VE + en % VE;
                ++at;
            }
        }
        __syncthreads();
    }
};

// value bits of element `at` of row r
template <int ELT>
__device__ __forceinline__ uint32_t row_bits(const RowParams &p, int64_t r, int at) {
    return (ELT == ATK_F32) ? ((const uint32_t *)p.x)[r * p.n + at] : ((uint32_t)((const uint16_t *)p.x)[r * p.n + at]) << 16;
}

}  // namespace atk
