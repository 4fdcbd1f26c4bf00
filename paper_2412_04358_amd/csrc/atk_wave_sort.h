// A wavefront's 64 * W words, sorted or cut to their largest in its registers.
#pragma once

#include "atk_common.h"
#include "atk_packed.h"

namespace atk {

#ifdef __HIPCC__

// Bitonic networks (Batcher 1968) over words that lie in the lanes' registers: no LDS, no barrier, and the same time whatever the words are.
// A block is 64 * R words in R registers.  The low bits of a word's place in its block are the register's number - the low bits are
// compared most often, and there a comparison is a minimum and a maximum - and the next six the lane's: four by DPP (a move and a median
// for either word), two by v_permlane16_swap / v_permlane32_swap, which bring the words of two registers together and back.  A median with the
// largest or the smallest word in place of a third one is the maximum or the minimum, as a lane's place in the network wants it.
// place bits of a lane: x0 x1 x2 x3 with lane = x0 * 1 ^ x1 * 2 ^ x2 * 7 ^ x3 * 8 (what quad_perm, half_mirror and row_ror:8 reach), then bits 4 and 5
struct LanePlace {
    int32_t most[6];  // INT_MAX where the bit is clear: there a block's larger words go; else INT_MIN
    int place;
    __device__ __forceinline__ LanePlace() {
        const int lane = threadIdx.x & (kWave - 1);
        place = lane ^ ((lane & 4) ? 3 : 0);
#pragma unroll
        for (int i = 0; i < 6; ++i) most[i] = ((place >> i) & 1) ? (int32_t)0x80000000 : 0x7fffffff;
    }
};

// ---- words of 32 bits, in the order of signed numbers
__device__ __forceinline__ int32_t larger(int32_t a, int32_t b) { return max(a, b); }
__device__ __forceinline__ int32_t smaller(int32_t a, int32_t b) { return min(a, b); }
__device__ __forceinline__ int32_t pick(int32_t a, int32_t b, int32_t m) { return med3_i32(a, b, m); }  // the larger one where m is INT_MAX, the smaller one where it is INT_MIN
template <int CTRL>
__device__ __forceinline__ int32_t from_lane(int32_t v) {
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);  // (every lane has a source: no old value to keep, so no copy before the move)
}
template <int Q>
__device__ __forceinline__ void swap_halves(int32_t &a, int32_t &b) {
    const auto s = Q == 4 ? __builtin_amdgcn_permlane16_swap((uint32_t)a, (uint32_t)b, false, false)
                          : __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false);
    a = (int32_t)s[0];
    b = (int32_t)s[1];
}
// ---- composites.  (As doubles, which a maximum and a minimum order, they would take an instruction more between lanes, and there the steps are.)
__device__ __forceinline__ u64 larger(u64 a, u64 b) { return a > b ? a : b; }
__device__ __forceinline__ u64 smaller(u64 a, u64 b) { return a > b ? b : a; }
__device__ __forceinline__ u64 pick(u64 a, u64 b, int32_t m) { return (a > b) != (m < 0) ? a : b; }
template <int CTRL>
__device__ __forceinline__ u64 from_lane(u64 v) {
    return (u64)(uint32_t)from_lane<CTRL>((int32_t)(v >> 32)) << 32 | (uint32_t)from_lane<CTRL>((int32_t)v);
}
template <int Q>
__device__ __forceinline__ void swap_halves(u64 &a, u64 &b) {
    int32_t ah = (int32_t)(a >> 32), al = (int32_t)a, bh = (int32_t)(b >> 32), bl = (int32_t)b;
    swap_halves<Q>(ah, bh);
    swap_halves<Q>(al, bl);
    a = (u64)(uint32_t)ah << 32 | (uint32_t)al;
    b = (u64)(uint32_t)bh << 32 | (uint32_t)bl;
}

constexpr int log2_c(int v) { return v <= 1 ? 0 : 1 + log2_c(v >> 1); }

// One step: the words whose places differ in bit J alone, in the direction that bit P of the place says (P = log2(64 R): odd blocks smallest
// first, of three the last one too; P = 31: every block largest first).
template <int W, int R, int P, int J, typename T>
__device__ __forceinline__ void wave_sort_step(T (&w)[W], const LanePlace &at) {
    constexpr int LR = log2_c(R), LN = LR + 6;
    // direction: known at compile time (the register's number decides), or one of the lane's bits
    constexpr bool by_lane = P >= LR && P < LN;
    auto up = [](int i) { return P == 31 ? false : (P == LN ? (W == 3 * R ? i / R != 0 : ((i / R) & 1) != 0) : ((i >> P) & 1) != 0); };  // smallest first
    if constexpr (J < LR) {
#pragma unroll
        for (int i = 0; i < W; ++i)
            if ((i & (1 << J)) == 0) {
                const T a = w[i], b = w[i | (1 << J)];
                if constexpr (by_lane) {
                    const int32_t m = at.most[P - LR];
                    w[i] = pick(a, b, m);
                    w[i | (1 << J)] = pick(a, b, ~m);
                } else {
                    w[i] = up(i) ? smaller(a, b) : larger(a, b);
                    w[i | (1 << J)] = up(i) ? larger(a, b) : smaller(a, b);
                }
            }
    } else {
        constexpr int Q = J - LR;
        constexpr int32_t kMost = 0x7fffffff;
        if constexpr (Q < 4) {
            constexpr int ctrl = Q == 0 ? 0xB1 : (Q == 1 ? 0x4E : (Q == 2 ? 0x141 : 0x128));
            const int32_t m = by_lane ? (at.most[Q] ^ at.most[by_lane ? P - LR : 0] ^ kMost) : at.most[Q];
            T other[W];
#pragma unroll
            for (int i = 0; i < W; ++i) other[i] = from_lane<ctrl>(w[i]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < W; ++i) w[i] = pick(w[i], other[i], !by_lane && up(i) ? ~m : m);
        } else {
            const int32_t m = by_lane ? at.most[by_lane ? P - LR : 0] : kMost;
            if constexpr (R >= 2) {
#pragma unroll
                for (int i = 0; i < W; i += 2) swap_halves<Q>(w[i], w[i + 1]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < W; i += 2) {
                    const T a = w[i], b = w[i + 1];
                    if constexpr (by_lane) {
                        w[i] = pick(a, b, m);
                        w[i + 1] = pick(a, b, ~m);
                    } else {
                        w[i] = up(i) ? smaller(a, b) : larger(a, b);
                        w[i + 1] = up(i) ? larger(a, b) : smaller(a, b);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < W; i += 2) swap_halves<Q>(w[i], w[i + 1]);
            } else {
#pragma unroll
                for (int i = 0; i < W; ++i) {
                    T a = w[i], b = w[i];
                    swap_halves<Q>(a, b);
                    const int32_t mine = by_lane ? (at.most[Q] ^ m ^ kMost) : (up(i) ? ~at.most[Q] : at.most[Q]);
                    w[i] = pick(a, b, mine);
                }
            }
        }
    }
}

template <int W, int R, int P, int J, typename T>
__device__ __forceinline__ void wave_sort_steps(T (&w)[W], const LanePlace &at) {  // bits J, J - 1, ... 0
    wave_sort_step<W, R, P, J, T>(w, at);
    // (step by step through all the words: word by word through the steps, as the compiler would go, every DPP move waits for the word it reads)
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (J > 0) wave_sort_steps<W, R, P, J - 1, T>(w, at);
}
template <int W, int R, int P, typename T>
__device__ __forceinline__ void wave_sort_blocks(T (&w)[W], const LanePlace &at) {  // from runs of 2^(P - 1) words in alternating order
    constexpr int LN = log2_c(R) + 6;
    if constexpr (P < LN) {
        wave_sort_steps<W, R, P, P - 1>(w, at);
        wave_sort_blocks<W, R, P + 1>(w, at);
    } else {
        wave_sort_steps<W, R, W == R ? 31 : P, P - 1>(w, at);
    }
}
// Blocks sorted largest first and smallest first in turn -> the largest block of all of them, largest first.  Of two such blocks the
// larger word of each place is among the larger half, and these lie in bitonic order again.
template <int W, int R, typename T>
__device__ __forceinline__ void wave_join_blocks(const T (&w)[W], T (&top)[R], const LanePlace &at) {
    if constexpr (W == R) {
#pragma unroll
        for (int i = 0; i < R; ++i) top[i] = w[i];
    } else {
        constexpr int H = W / 2, LN = log2_c(R) + 6;
        T h[H];
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const int block = i / R, in = i % R;
            h[i] = larger(w[2 * block * R + in], w[(2 * block + 1) * R + in]);
        }
        wave_sort_steps<H, R, H == R ? 31 : LN, LN - 1>(h, at);
        wave_join_blocks<H, R>(h, top, at);
    }
}
// The 64 * R largest of the wavefront's 64 * W words, largest first: lane l's top[i] is number R * at.place + i.  sorted: the words already lie in
// runs of that many (a power of two below R), in registers side by side, largest first where the run's number is even, smallest first where odd.
template <int W, int R, int SORTED, typename T>
__device__ __forceinline__ void wave_largest(T (&w)[W], T (&top)[R], const LanePlace &at) {
    static_assert(SORTED == 1 || SORTED < R, "runs inside a lane's registers of a block");
    wave_sort_blocks<W, R, log2_c(SORTED) + 1>(w, at);
    wave_join_blocks<W, R>(w, top, at);
}
// The 128 * R largest of 192 * R words, largest first: lane l's top[i] is number R * at.place + i, its top[R + i] number 64 * R + that.  A list of
// that size, with a margin of half: three blocks cost 0.8 of sorting four (words to 512 of 1024: 1050 and 1270 instructions).
template <int R>
__device__ __forceinline__ void wave_largest_two_of_three(int32_t (&w)[3 * R], int32_t (&top)[2 * R], const LanePlace &at) {
    constexpr int LN = log2_c(R) + 6;
    wave_sort_blocks<3 * R, R, 1>(w, at);
    // of the first two blocks the larger half and the smaller one, each largest first
    auto halves = [&]() {
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int32_t a = top[i], b = top[R + i];
            top[i] = max(a, b);
            top[R + i] = min(a, b);
        }
        wave_sort_steps<2 * R, R, 31, LN - 1>(top, at);
    };
#pragma unroll
    for (int i = 0; i < 2 * R; ++i) top[i] = w[i];
    halves();
    // the third block, smallest first, against the smaller half: what wins is, behind the larger half, in bitonic order again
#pragma unroll
    for (int i = 0; i < R; ++i) top[R + i] = max(top[R + i], w[2 * R + i]);
    halves();
}

#endif  // __HIPCC__

}  // namespace atk
