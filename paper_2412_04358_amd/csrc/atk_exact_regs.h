// Device code that exact_topk's row kernels share: a row or a part of one in a workgroup's registers, bins linear in the order of
// the elements, and the prefix sum that turns their counts into places.  What it is for: atk_exact_row.hip.
#pragma once

#include <type_traits>

#include "atk_common.h"
#include "atk_exact.h"
#include "atk_packed.h"
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
    int rank_up;            // the upper bound (0: there is none)
    u64 *lists;             // [row][part][part_cap] composites: those at or above the upper bound from the front, the rest from the back
    u64 *heads;             // [row][part][4]: (a key that none of the list lies below << 32 | elements in front), (the part's largest
                            // key << 32 | elements at the back), the upper bound, unused
    uint32_t *tickets;      // one per row, kTicketStride apart, zero between calls
};

typedef uint32_t row_v4u __attribute__((ext_vector_type(4)));

// The order key of the float that a packed bf16 key (a two's complement number of 16 bits, -0 as +0) stands for, and the least packed key whose float has the order key
// u or a higher one, for u of the kind that bounds are: bits below the sixteenth clear, or a bf16's.
__device__ __forceinline__ uint32_t ukey_of_pk(int s) { return (((uint32_t)s << 16) ^ 0x80000000u) + (uint32_t)(s >> 31); }
__device__ __forceinline__ int pk_of_ukey(uint32_t u) { return (int)(u >> 16) - (u & 0x80000000u ? 0x8000 : 0x7fff); }

// The 16-byte boundary at or before row r's first element.  It is reached from x by an offset: an address that has been a number may
// lie in any memory as far as the compiler knows, and its (flat) loads are waited for together with those of LDS.  Global loads are not:
// 2048 x 8192 bf16, k = 512: 18.86 -> 18.63 us; 128 x 2^20 f32, k = 2^18, and rows in parts the same.
__device__ __forceinline__ const row_v4u *row_vectors(const void *x, int64_t first_byte) {
    const int64_t off = (int64_t)((((uintptr_t)x + (uintptr_t)first_byte) & ~(uintptr_t)15) - (uintptr_t)x);
    return (const row_v4u *)((const unsigned char *)x + off);
}

// LDS words behind the bins: [0] bin of the need-th largest, [1] elements in higher bins, [2] its elements, [3] all counted,
// [4] crowded, [5] and [7] cursors, [8..24), [24..40) and [40..56) per-wavefront words
constexpr int kRowMisc = 56;

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
        const row_v4u *row = row_vectors(p.x, r * p.n * ES);
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
    // FIRST: the groups are the lane's first eight elements, one each (k_max is still the largest of all).
    // SUM: not the smallest of the wavefronts' candidates but the largest that, all wavefronts together, rank maxima per wavefront reach:
    // wavefronts may be unlike each other then (masked in part, sorted).  words: 32 words of LDS.  k_up: the same with rank_up (0: none).
    // KEYS: the words hold keys (to_keys()).
    template <bool FIRST = false, bool SUM = false, bool KEYS = false>
    __device__ __forceinline__ void bound(int sub, int rank, uint32_t *misc, uint32_t &k_min, uint32_t &k_max, uint32_t *words = nullptr,
                                          int rank_up = 0, uint32_t *k_up = nullptr) {
        const int tid = threadIdx.x, lane = tid & (kWave - 1), n_waves = blockDim.x >> 6;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        constexpr int SM = NV * 4 < 8 ? 4 : 8;
        float mx[SM];
#pragma unroll
        for (int i = 0; i < SM; ++i) mx[i] = __uint_as_float(0x7fc00000u);
#pragma unroll
        for (int w = 0; w < NV * 4; ++w) {
            if (FIRST || KEYS) break;
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
        if constexpr (KEYS) {  // (a group's maximum in the upper half of its word, as a number; the lower one is the maximum of the other half of its elements)
            uint32_t pm[SM];
#pragma unroll
            for (int w = 0; w < NV * 4; ++w) {
                const uint32_t a = q[w >> 2][w & 3];
                pm[w % SM] = w < SM ? a : __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(pk2, pm[w % SM]), __builtin_bit_cast(pk2, a)));
            }
#pragma unroll
            for (int i = 0; i < SM; ++i) mx[i] = __int_as_float(max((int)pm[i], (int)(pm[i] << 16)) >> 16);
        }
        // (of two groups' maxima as they stand: the larger)
        auto top_of = [](float a, float b) { return KEYS ? __int_as_float(max(__float_as_int(a), __float_as_int(b))) : fmaxf(a, b); };
        auto key_of = [](float f) {
            if constexpr (KEYS) return ukey_of_pk(__float_as_int(f));
            return f == f ? ukey_of_bits(__float_as_uint(f)) : 0u;
        };
        if (SUM && tid < 32) words[tid] = 0u;
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
                for (int j = i + S; j < SM; j += S) m = top_of(m, mx[j]);
                key[i] = key_of(m);
                top = max(top, key[i]);
            }
            k_max = top;
            auto count = [&](uint32_t from) {
                int cnt = 0;
#pragma unroll
                for (int i = 0; i < S; ++i) cnt += __popcll(__ballot(key[i] >= from));
                return cnt;
            };
            auto nth_key = [&](int of) {
                uint32_t have = 0u;
#pragma unroll
                for (int bit = 31; bit >= 16; --bit) {
                    const uint32_t want = have | (1u << bit);
                    if (count(want) >= of) have = want;
                }
                return have;
            };
            if (rank == 0) {
                k_min = 0xffffffffu;
#pragma unroll
                for (int i = 0; i < S; ++i) k_min = key[i] && key[i] < k_min ? key[i] : k_min;
                k_min = wave_min_u32(k_min);
            } else {
                k_min = nth_key(rank);
            }
            if constexpr (SUM) {
                const uint32_t top_of_wave = wave_max_u32(k_max), up = rank_up ? nth_key(rank_up) : 0u;
                if (lane == 0) {
                    misc[8 + wave] = k_min;
                    misc[24 + wave] = top_of_wave;
                    misc[40 + wave] = up;
                }
                __syncthreads();
                const bool is = lane < n_waves;
                auto reached = [&](uint32_t theirs, uint32_t *sums) {  // lane j: the j-th wavefront's candidate
                    int mine = 0;  // maxima of this wavefront that reach it
                    if (S == 1 && n_waves > 4) {
                        // (all counts at once: one after the other each waits for its own comparison; 64 x 128256 bf16, k = 256: 13.03 -> 12.75 us)
                        int cnt[16];
#pragma unroll
                        for (int j = 0; j < 16; ++j) cnt[j] = __popcll(__ballot(key[0] >= (uint32_t)__builtin_amdgcn_readlane((int)theirs, j)));
#pragma unroll
                        for (int j = 0; j < 16; ++j) mine = lane == j ? cnt[j] : mine;
                    } else {
                        for (int j = 0; j < n_waves; ++j) {
                            const int cnt = count((uint32_t)__builtin_amdgcn_readlane((int)theirs, j));
                            if (lane == j) mine = cnt;
                        }
                    }
                    if (is && mine) atomicAdd(&sums[lane], (uint32_t)mine);
                };
                const uint32_t theirs = is ? misc[8 + lane] : 0u, theirs_up = is ? misc[40 + lane] : 0u;
                reached(theirs, words);
                if (rank_up) reached(theirs_up, words + 16);
                __syncthreads();
                k_min = wave_max_u32(is && words[lane] >= (uint32_t)(rank * n_waves) ? theirs : 0u);
                if (rank_up) *k_up = wave_max_u32(is && words[16 + lane] >= (uint32_t)(rank_up * n_waves) ? theirs_up : 0u);
            }
        };
        if (sub == 1)
            nth(std::integral_constant<int, 1>());
        else if (sub == 2)
            nth(std::integral_constant<int, 2>());
        else if (sub == 4 || SM == 4)
            nth(std::integral_constant<int, 4>());
        else
            nth(std::integral_constant<int, SM>());
        if constexpr (FIRST) {
            float most = __uint_as_float(0x7fc00000u);
            each([&](uint32_t bits, int, int) { most = fmaxf(most, __uint_as_float(bits)); });
            k_max = key_of(most);
        }
        if constexpr (!SUM) {
            k_max = wave_max_u32(k_max);
            if (lane == 0) {
                misc[8 + wave] = k_min;
                misc[24 + wave] = k_max;
            }
            __syncthreads();
            k_min = wave_min_u32(lane < n_waves ? misc[8 + lane] : 0xffffffffu);
        }
        k_max = wave_max_u32(lane < n_waves ? misc[24 + lane] : 0u);
        if (k_min < 0x007fffffu) k_min = 0x007fffffu;  // (-inf's)
        if (k_min > k_max) k_min = k_max;
        if constexpr (SUM) *k_up = rank_up ? min(*k_up, k_max) : 0u;
        __syncthreads();  // (the words are used again)
    }

    // ---- bf16: the words as keys, two signed 16-bit numbers each in the order of the values (elements that are none, as NaNs, below all): a comparison is then
    // a subtraction for two elements at once (rows in parts; 64 x 128256, k = 256: 13.25 -> 12.75 us, k = 64 12.2 -> 11.8)
    __device__ __forceinline__ void to_keys() {
        static_assert(ELT == ATK_BF16, "");
#pragma unroll
        for (int j = 0; j < NV; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) q[j][i] = pack_keys(q[j][i]);
    }
    // list_from() of keys: positions of the elements whose (order) keys are k_lo and above
    __device__ __forceinline__ void list_keys(uint32_t k_lo, int2 *list, uint32_t cap, uint32_t *count) {
        static_assert(ELT == ATK_BF16, "");
        constexpr int W = NV * 4, MW = (W + 15) / 16;
        const int lane = threadIdx.x & (kWave - 1), T = blockDim.x;
        const int from = pk_of_ukey(k_lo);
        const pk2 below = {(int16_t)(from - 1), (int16_t)(from - 1)};
        uint32_t mk[MW], cnt = 0;  // bit 16 h + i of mask w: element h of word 16 w + i (a last mask of n words: from bit 16 - n on)
#pragma unroll
        for (int w = 0; w < MW; ++w) {
            mk[w] = 0u;
#pragma unroll
            for (int i = 16 * w; i < 16 * w + 16 && i < W; ++i)
                mk[w] = (mk[w] >> 1) | (__builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(below, __builtin_bit_cast(pk2, (uint32_t)q[i >> 2][i & 3]))) & 0x80008000u);
            cnt += (uint32_t)__popc(mk[w]);
        }
        const uint32_t incl = wave_incl_scan_u32(cnt);
        uint32_t at = 0;
        if (lane == kWave - 1) at = atomicAdd(count, incl);
        at = (uint32_t)__builtin_amdgcn_readlane((int)at, kWave - 1) + incl - cnt;
#pragma unroll
        for (int w = 0; w < MW; ++w) {
            const int n_w = W - 16 * w < 16 ? W - 16 * w : 16;
            uint32_t b = mk[w];
            while (b && at < cap) {  // (once the list is full, the number alone matters)
                const int bit = __builtin_ctz(b), word = (bit & 15) - (16 - n_w) + 16 * w;
                b &= b - 1u;
                list[at++].y = i0 + (word >> 2) * T * VE + (word & 3) * 2 + (bit >> 4);
            }
        }
        __syncthreads();
    }

    static constexpr int M = (E + 31) / 32;  // masks of 32 elements, the last perhaps of fewer: element en has bit 31 - en % 32 of word en / 32

    // Which elements reach v_lo.  Two operations per element: a comparison, and an addition of the mask to itself with the
    // comparison as carry.
    __device__ __forceinline__ void masks_from(float v_lo, uint32_t (&mk)[M]) {
#pragma unroll
        for (int w = 0; w < M; ++w) mk[w] = 0u;
        each([&](uint32_t bits, int, int en) {
            asm volatile("v_cmp_le_f32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(mk[en / 32]) : "v"(v_lo), "v"(bits) : "vcc");
        });
#pragma unroll
        for (int w = 0; w < M; ++w) mk[w] <<= 32 - (E - 32 * w < 32 ? E - 32 * w : 32);
    }
    // Positions of the elements whose bits are set to list[0 .. ] (at most cap of them); the cursor *count starts from zero and
    // ends as their number.  The few that are set are taken one by one: storing an element under its own condition costs every
    // element the six or so operations of a branch that few of the lanes take (64 x 128256 bf16, k = 256: 8.2 us of the
    // kernel's 18).  Called by the whole workgroup; ends in a barrier.
    __device__ __forceinline__ void list_masks(const uint32_t (&mk)[M], int2 *list, uint32_t cap, uint32_t *count) {
        const int lane = threadIdx.x & (kWave - 1), T = blockDim.x;
        uint32_t cnt = 0;
#pragma unroll
        for (int w = 0; w < M; ++w) cnt += (uint32_t)__popc(mk[w]);
        const uint32_t incl = wave_incl_scan_u32(cnt);
        uint32_t at = 0;
        if (lane == kWave - 1) at = atomicAdd(count, incl);
        at = (uint32_t)__builtin_amdgcn_readlane((int)at, kWave - 1) + incl - cnt;
#pragma unroll
        for (int w = 0; w < M; ++w) {
            uint32_t b = mk[w];
            while (b && at < cap) {  // (once the list is full, the number alone matters)
                const int t = __clz((int)b), en = w * 32 + t;
                b &= ~(0x80000000u >> t);
                list[at++].y = i0 + (en / VE) * T * VE + en % VE;
            }
        }
        __syncthreads();
    }
    __device__ __forceinline__ void list_from(float v_lo, int2 *list, uint32_t cap, uint32_t *count) {
        uint32_t mk[M];
        masks_from(v_lo, mk);
        list_masks(mk, list, cap, count);
    }

    // Positions of the k largest elements (ties: the first ones) to list[], or of some more if that is the quicker way: of those above a
    // run of ties at the lower end, if there are k and no more than cap of them.  n: how many.  Returns a key that none of them
    // lies below (bf16: without the low bits).  More than k elements reach lo, none is above hi.  Where ties at the lower
    // end do not decide it, the key is searched by halving, a comparison and two scalar operations per element and step; then the
    // ties are counted by rows of vectors (lanes side by side hold vectors side by side).  words: NV words of LDS.  Called by
    // the whole workgroup; ends in a barrier.
    __device__ __forceinline__ uint32_t list_largest(uint32_t k, uint32_t lo, uint32_t hi, int2 *list, uint32_t cap, uint32_t &n, uint32_t *count,
                                                     uint32_t *words, uint32_t *misc) {
        constexpr int drop = (ELT == ATK_BF16) ? 16 : 0;
        const int tid = threadIdx.x, lane = tid & (kWave - 1), n_waves = blockDim.x >> 6;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        auto value = [](uint32_t t) { return __uint_as_float(bits_of_ukey(max(t << drop, 0x007fffffu))); };  // (no lower than -inf: NaNs lie there)
        int step = 0;
        auto reach = [&](uint32_t t) {  // how many elements do; one barrier
            const float v = value(t);
            int cnt = 0;
            each([&](uint32_t bits, int, int) { cnt += __popcll(__ballot(__uint_as_float(bits) >= v)); });
            uint32_t *sums = misc + 8 + 16 * (step++ & 1);
            if (lane == 0) sums[wave] = (uint32_t)cnt;
            __syncthreads();
            return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan_u32(lane < n_waves ? sums[lane] : 0u), kWave - 1);
        };
        // the least of those that reach lo
        {
            const float v = value(lo >> drop);
            float least = __uint_as_float(0x7f800000u);
            each([&](uint32_t bits, int, int) {
                const float f = __uint_as_float(bits);
                least = f >= v && f < least ? f : least;
            });
            uint32_t key = wave_min_u32(ukey_of_bits(__float_as_uint(least)));
            if (lane == 0) misc[24 + wave] = key;
            __syncthreads();
            lo = wave_min_u32(lane < n_waves ? misc[24 + lane] : 0xffffffffu);
        }
        uint32_t l = lo >> drop, h = (hi >> drop) + 1u;  // k and more reach l, fewer than k reach h
        const uint32_t higher = reach(l + 1u);
        if (higher < k) {
            h = l + 1u;
        } else if (higher <= cap) {
            n = higher;
            list_from(value(l + 1u), list, cap, count);
            return l << drop;
        } else {
            ++l;
        }
        while (h - l > 1u) {
            const uint32_t mid = l + (h - l) / 2u;
            if (reach(mid) >= k)
                l = mid;
            else
                h = mid;
        }
        n = k;
        uint32_t above[M], ties[M], mine = 0;
        masks_from(value(l), ties);
        masks_from(value(l + 1u), above);
#pragma unroll
        for (int w = 0; w < M; ++w) {
            ties[w] &= ~above[w];
            mine += (uint32_t)__popc(above[w]);
        }
        __syncthreads();  // (the sums have been read)
        if (tid < NV) words[tid] = 0u;
        if (tid == 0) misc[8] = 0u;
        __syncthreads();
        auto field = [&](int j) { return (ties[j * VE / 32] >> (32 - VE - j * VE % 32)) & ((1u << VE) - 1u); };
        mine = wave_incl_scan_u32(mine);
        if (lane == kWave - 1) atomicAdd(&misc[8], mine);
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const uint32_t sum = wave_incl_scan_u32((uint32_t)__popc(field(j)));
            if (lane == kWave - 1 && sum) atomicAdd(&words[j], sum);
        }
        __syncthreads();
        uint32_t left = k - misc[8];  // ties to take
        int row = 0;                  // all of the vectors' rows before this one, and the first of this one
        while (row < NV - 1 && words[row] <= left) left -= words[row++];
        uint32_t here = 0;
#pragma unroll
        for (int j = 0; j < NV; ++j)
            if (j == row) here = field(j);
        const uint32_t n_here = (uint32_t)__popc(here), incl = wave_incl_scan_u32(n_here);
        if (lane == kWave - 1) misc[24 + wave] = incl;
        __syncthreads();
        const uint32_t waves = wave_incl_scan_u32(lane < n_waves ? misc[24 + lane] : 0u);
        uint32_t before = incl - n_here;
        if (wave > 0) before += (uint32_t)__builtin_amdgcn_readlane((int)waves, wave - 1);
        uint32_t drop_n = before + n_here > left ? (before >= left ? n_here : before + n_here - left) : 0u;
        for (; drop_n; --drop_n) here &= here - 1u;  // (the last ones)
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const uint32_t f = j < row ? field(j) : (j == row ? here : 0u);
            above[j * VE / 32] |= f << (32 - VE - j * VE % 32);
        }
        list_masks(above, list, k, count);
        return l << drop;
    }
};

// ---- the digit descent in a workgroup (RadixSelect, Appendix D.2), most significant digit first, on the composite without the bits
// that carry nothing (the low 16 of a bf16 key, the index bits above idx_bits)
template <int ELT>
struct RowSqueeze {
    static constexpr int drop = ELT == ATK_BF16 ? 16 : 0;
    int keep;
    __device__ __forceinline__ u64 operator()(u64 c) const { return ((c >> (32 + drop)) << keep) | (c & ((1ull << keep) - 1ull)); }
    // the key that t's key bits stand for, without the bits that were dropped
    __device__ __forceinline__ uint32_t key(u64 t) const { return (uint32_t)(t >> keep) << drop; }
};

// cur[bin] += 1 for every lane with `on`.  Many lanes with one bin (ties) would queue up on one word of LDS: the first bin that
// comes up in the wavefront is counted by ballot.
__device__ __forceinline__ void row_count(uint32_t *cur, uint32_t bin, bool on) {
    const int lane = threadIdx.x & (kWave - 1);
    u64 todo = __ballot(on);
#pragma unroll
    for (int t = 0; t < 1; ++t) {
        if (!todo) return;  // uniform over the wavefront
        const int first = __builtin_ctzll(todo);
        const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)bin, first);
        const u64 same = __ballot(on && bin == b);
        if (lane == first) atomicAdd(&cur[b], (uint32_t)__popcll(same));
        on = on && bin != b;
        todo &= ~same;
    }
    if (on) atomicAdd(&cur[bin], 1u);
}

// The threshold (squeezed) that exactly `need` of the elements reach: sweep(f) calls f(composite, whether it counts) for every element,
// the same ones each time, with whole wavefronts together.  k_lo, k_hi: keys between which the need-th largest lies, none above
// k_hi.  cur: room for 2^lg_bins words, no fewer than the workgroup's lanes.  Called by the whole workgroup; ends in a barrier.
template <int ELT, typename SWEEP>
__device__ __forceinline__ u64 row_threshold_by_digits(SWEEP sweep, uint32_t need, uint32_t k_lo, uint32_t k_hi, int idx_bits, int lg_bins,
                                                       uint32_t *cur, uint32_t *misc) {
    const int tid = threadIdx.x, T = blockDim.x, n_bins = 1 << lg_bins;
    const RowSqueeze<ELT> sq{idx_bits + 1};
    const uint32_t differ = (k_lo ^ k_hi) >> sq.drop;
    int top = sq.keep + (differ ? 32 - __builtin_clz(differ) : 0);  // bits still open
    u64 prefix = (((u64)(k_lo >> sq.drop)) << sq.keep) & (top >= 64 ? 0ull : (~0ull << top));
    for (;;) {
        const int w = top < lg_bins ? top : lg_bins;
        const int shift = top - w;
        const u64 hi_mask = top >= 64 ? 0ull : (~0ull << top);
        for (int i = tid; i < n_bins; i += T) cur[i] = 0u;
        __syncthreads();
        sweep([&](u64 c, bool on) {
            const u64 q = sq(c);
            row_count(cur, (uint32_t)(q >> shift) & ((1u << w) - 1u), on && (q & hi_mask) == prefix);
        });
        __syncthreads();
        row_scan(cur, misc, n_bins, need);
        prefix |= (u64)misc[0] << shift;
        need -= misc[1];
        const bool done = misc[2] == need || shift == 0;
        __syncthreads();  // misc and cur are written again
        if (done) break;
        top = shift;
    }
    return prefix;
}

// f(composite, whether it is one) for every element of the vectors v0 .. v1 of row r, read from memory, whole wavefronts
// together: the ways that few rows take go through the elements like this and not through the registers that hold them, because a
// loop is small and what RowRegs::each() unrolls is not.
template <int ELT, typename F>
__device__ __forceinline__ void row_vec_sweep(const RowParams &p, int64_t r, int v0, int v1, int rot, F f) {
    constexpr int ES = (ELT == ATK_F32) ? 4 : 2, VE = 16 / ES, U = 8 / VE;
    const int T = blockDim.x, lane = threadIdx.x & (kWave - 1), end = rot + p.n;
    const row_v4u *row = row_vectors(p.x, r * p.n * ES);
    for (int w0 = v0 + (int)threadIdx.x - lane; w0 < v1; w0 += U * T) {  // uniform over the wavefront
        row_v4u q[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int v = w0 + lane + u * T;
            q[u] = row[v < v1 ? v : v1 - 1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int v = w0 + lane + u * T;
#pragma unroll
            for (int e = 0; e < VE; ++e) {
                const int at = v * VE + e;
                const uint32_t a = q[u][ELT == ATK_F32 ? e : (e >> 1)];
                const bool ok = v < v1 && at >= rot && at < end;
                f(make_composite(ELT == ATK_F32 ? a : ((e & 1) ? (a & 0xffff0000u) : (a << 16)), at - rot), ok);
            }
        }
    }
}

// value bits of element `at` of row r
template <int ELT>
__device__ __forceinline__ uint32_t row_bits(const RowParams &p, int64_t r, int at) {
    return (ELT == ATK_F32) ? ((const uint32_t *)p.x)[r * p.n + at] : ((uint32_t)((const uint16_t *)p.x)[r * p.n + at]) << 16;
}

}  // namespace atk
