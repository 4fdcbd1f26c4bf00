// Candidates of bf16 rows as one 32-bit word each - [31:16] the value as a two's complement number (-0 is +0), [15:0] 0xffff - column index - and a
// wavefront's sorted ones as outputs.
#pragma once

#include "atk_common.h"
#include "atk_packed.h"

namespace atk {

#ifdef __HIPCC__

typedef uint32_t wave_v4u __attribute__((ext_vector_type(4)));
typedef uint32_t wave_v2u __attribute__((ext_vector_type(2)));

// The values' bits (bf16, two to a word) of two candidate words
__device__ __forceinline__ uint32_t wave_pair_bits(int32_t even, int32_t odd) {
    const uint32_t keys = ((uint32_t)even >> 16) | ((uint32_t)odd & 0xffff0000u);
    const pk2 v = __builtin_bit_cast(pk2, keys), sgn = v >> 15;
    const pk2 mag = __builtin_bit_cast(pk2, keys ^ __builtin_bit_cast(uint32_t, sgn)) - sgn;
    return __builtin_bit_cast(uint32_t, mag) | (__builtin_bit_cast(uint32_t, sgn) & 0x80008000u);
}
__device__ __forceinline__ int32_t wave_index(int32_t c) { return (int32_t)(0xffffu - ((uint32_t)c & 0xffffu)); }

// top[0 .. R): outputs first, first + 1, ... of a row with k of them.  row: its elements.  vec: vals and idx lie on boundaries of min(R, 8) outputs, and k
// is a multiple of that.
template <int R>
__device__ __forceinline__ void wave_write(const uint16_t *row, uint16_t *vals, int32_t *idx, int k, bool vec, int first, const int32_t (&top)[R]) {
    constexpr int H = R < 2 ? 1 : R / 2;
    uint32_t bits[H];
    bool zero = false;
#pragma unroll
    for (int i = 0; i < H; ++i) bits[i] = wave_pair_bits(top[2 * i], R < 2 ? 0 : top[2 * i + 1]);
#pragma unroll
    for (int i = 0; i < R; ++i) zero = zero || ((uint32_t)top[i] >> 16) == 0u;
    if (__ballot(zero) != 0ull) {  // +0 or -0: the element itself says
        uint32_t own[R];
#pragma unroll
        for (int i = 0; i < R; ++i) own[i] = row[((uint32_t)top[i] >> 16) == 0u ? wave_index(top[i]) : 0];
#pragma unroll
        for (int i = 0; i < R; ++i)
            if (((uint32_t)top[i] >> 16) == 0u) bits[i / 2] |= (i & 1) ? own[i] << 16 : own[i];
    }
    if (vec) {
        constexpr int C = R < 8 ? R : 8;
#pragma unroll
        for (int c = 0; c < R; c += C) {
            const int o = first + c;
            if (o >= k) break;
            if constexpr (C == 8) {
                *(wave_v4u *)(vals + o) = wave_v4u{bits[c / 2], bits[c / 2 + 1], bits[c / 2 + 2], bits[c / 2 + 3]};
            } else if constexpr (C == 4) {
                *(wave_v2u *)(vals + o) = wave_v2u{bits[0], bits[1]};
            } else if constexpr (C == 2) {
                *(uint32_t *)(vals + o) = bits[0];
            } else {
                vals[o] = (uint16_t)bits[0];
            }
            if constexpr (C >= 4) {
#pragma unroll
                for (int i = 0; i < C; i += 4)
                    *(wave_v4u *)(idx + o + i) = wave_v4u{(uint32_t)wave_index(top[c + i]), (uint32_t)wave_index(top[c + i + 1]),
                                                          (uint32_t)wave_index(top[c + i + 2]), (uint32_t)wave_index(top[c + i + 3])};
            } else {
#pragma unroll
                for (int i = 0; i < C; ++i) idx[o + i] = wave_index(top[c + i]);
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < R; ++i)
        if (first + i < k) {
            vals[first + i] = (uint16_t)((i & 1) ? bits[i / 2] >> 16 : bits[i / 2]);
            idx[first + i] = wave_index(top[i]);
        }
}

#endif  // __HIPCC__

}  // namespace atk
