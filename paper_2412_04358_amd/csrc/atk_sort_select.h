// Stage 2 by sorting networks: four wavefronts sort a quarter of the candidates each in their registers, cut to the k largest, and one joins their lists.
#pragma once

#include "atk_common.h"
#include "atk_packed.h"
#include "atk_select.h"
#include "atk_wave_sort.h"

namespace atk {

#ifdef __HIPCC__

constexpr int kSortWaves = 4;
constexpr int kSortIdxBits = 17;  // column indices that fit a word beside a positive bf16 without its sign

// The 64 * R largest of the workgroup's first NWV (4 or 8) wavefronts' 64 * W words each, largest first, in the first wavefront: its lane's top[i] is number
// R * place + i.  lists: LDS, NWV * 64 * R words.  Called by the whole workgroup; one barrier.
template <int NWV, int W, int R, typename T>
__device__ __forceinline__ void sort_waves(T (&w)[W], T (&top)[R], T *lists, const LanePlace &at) {
    constexpr int N = 64 * R, LN = log2_c(R) + 6, H = NWV / 2;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (wave < NWV) {  // (uniform over the wavefront)
        wave_largest<W, R, 1>(w, top, at);
        if (wave > 0) {
            // (every second list the other way round: of two lists the larger word of each place is then among the N largest)
#pragma unroll
            for (int i = 0; i < R; ++i) lists[wave * N + ((wave & 1) ? N - 1 - (R * at.place + i) : R * at.place + i)] = top[i];
        }
    }
    __syncthreads();
    if (wave > 0) return;
    T both[H * R];
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int o = R * at.place + i;
            both[h * R + i] = larger(h ? lists[2 * h * N + o] : top[i], lists[(2 * h + 1) * N + o]);
        }
    wave_sort_steps<H * R, R, LN, LN - 1>(both, at);
    wave_join_blocks<H * R, R>(both, top, at);
}

// Exact top-k of the `count` distinct composites at cand[0 .. count) (LDS, on a 16-byte boundary, 4112 bytes of free LDS behind them), written largest first to
// row row_out; false, and nothing is written, where fewer than k of them are positive.  bf16, indices of up to 17 bits: a positive value's 15 bits and the
// index are one word.  Called by the whole workgroup after a barrier that made cand visible.
//
// What it replaces (select_write) is a chain of six barriers: key range, histogram, prefix sum, filing, ranks.  64 x 128256, k = 256, b = 512,
// k_b = 2: 3.15 us from the last candidate to the last output there.  Rows with fewer positive candidates than that - logarithms of probabilities, say - go
// back to it, so these are counted first, which costs a barrier, 0.08 us (64 x 128256 as above: N(0,1) 11.7 us without networks, 9.57 counted after
// the sort, 9.65 before it; logarithms of probabilities 13.1, 13.6, 12.5; 2169 x 17628, k = 256, b = 226, k_b = 2, these: 27.9, 32.5, 28.3).
template <int ELT>
__device__ __forceinline__ bool sort_select_fits(int count, int k, int idx_bits) {
    return ELT == ATK_BF16 && count <= 1024 && k <= 256 && idx_bits <= kSortIdxBits && (int)blockDim.x >= kSortWaves * kWave;
}
template <int W, int R>
__device__ __forceinline__ bool sort_select_words(const u64 *cand, int count, int k, void *out_vals, int32_t *out_idx, int64_t row_out) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const LanePlace at;
    int32_t *n_pos = (int32_t *)(cand + ((count + 1) & ~1)), *lists = n_pos + 4;
    const uint32_t none = 0x80000000u;  // (the words are in the order of signed numbers)
    int32_t w[W], top[R];
    if (wave < kSortWaves) {
        int positive = 0;
#pragma unroll
        for (int i = 0; i < W; ++i) {
            const int c = tid * W + i;
            const u64 v = c < count ? cand[c] : 0ull;
            const uint32_t bits = (uint32_t)(v >> 48) & 0x7fffu;
            const bool on = (v >> 63) != 0ull && bits != 0u;
            const uint32_t inv = ((uint32_t)v >> 1) & ((1u << kSortIdxBits) - 1u);  // (0x7fffffff - index: the low bits of 0x1ffff - index)
            w[i] = (int32_t)((on ? bits << kSortIdxBits | inv : 0u) ^ none);
            positive += __popcll(__ballot(on));
        }
        if (lane == 0) n_pos[wave] = positive;
    }
    __syncthreads();
    const int4 positive = *(const int4 *)n_pos;
    if (__builtin_amdgcn_readfirstlane(positive.x + positive.y + positive.z + positive.w) < k) return false;
    sort_waves<kSortWaves, W, R>(w, top, lists, at);
    if (wave > 0) return true;
    uint16_t *vals = (uint16_t *)out_vals + row_out * k;
    int32_t *idx = out_idx + row_out * k;
    const int o = R * at.place;
    uint32_t b[R], x[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const uint32_t u = (uint32_t)top[i] ^ none;
        b[i] = u >> kSortIdxBits;
        x[i] = ((1u << kSortIdxBits) - 1u) - (u & ((1u << kSortIdxBits) - 1u));
    }
    if constexpr (R == 4) {
        if (k % 4 == 0 && (((uintptr_t)out_vals | (uintptr_t)out_idx) & 15u) == 0) {
            if (o < k) {
                *(uint2 *)(vals + o) = make_uint2(b[0] | b[1] << 16, b[2] | b[3] << 16);
                *(uint4 *)(idx + o) = make_uint4(x[0], x[1], x[2], x[3]);
            }
            return true;
        }
    }
#pragma unroll
    for (int i = 0; i < R; ++i)
        if (o + i < k) {
            vals[o + i] = (uint16_t)b[i];
            idx[o + i] = (int32_t)x[i];
        }
    return true;
}
__device__ __forceinline__ bool sort_select(const u64 *cand, int count, int k, void *out_vals, int32_t *out_idx, int64_t row_out) {
    if (k > 64) return sort_select_words<4, 4>(cand, count, k, out_vals, out_idx, row_out);
    if (count > 256) return sort_select_words<4, 1>(cand, count, k, out_vals, out_idx, row_out);
    return sort_select_words<1, 1>(cand, count, k, out_vals, out_idx, row_out);
}

// The k <= 64 largest of the `count` composites at cand[0 .. count) (LDS, in any order, 0 for none; count <= 64 * W * NWV), written largest first to row row_out.
// 512 * NWV bytes of free LDS behind them, on a 16-byte boundary.  Called by the whole workgroup, of NWV wavefronts at least, after a barrier that made
// cand visible.
template <int ELT, int NWV, int W>
__device__ __forceinline__ void sort_select_few(const u64 *cand, int count, int k, void *out_vals, int32_t *out_idx, int64_t row_out) {
    const LanePlace at;
    u64 w[W], top[1];
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const int c = (int)threadIdx.x + i * NWV * kWave;
        w[i] = c < count ? cand[c] : 0ull;
    }
    sort_waves<NWV, W, 1>(w, top, (u64 *)cand + ((count + 1) & ~1), at);
    if ((int)threadIdx.x < kWave && at.place < k) write_composite<ELT>(top[0], out_vals, out_idx, row_out * k + at.place);
}

#endif  // __HIPCC__

}  // namespace atk
