// Register queues of packed 32-bit words for bf16.
#pragma once

#include "atk_common.h"
#include "atk_stream.h"

namespace atk {

#ifdef __HIPCC__

__device__ __forceinline__ int32_t med3_i32(int32_t a, int32_t b, int32_t c) { return max(min(a, b), min(max(a, b), c)); }  // v_med3_i32

// ---- packed queues for bf16 with k_b >= 2 -------------------------------------------------------
// A bf16 element and its matrix row fit one signed 32-bit word: [31:16] the value's sign and magnitude as a two's complement
// number (so -0 is +0), [15:0] 0xffff - (row - first row of this lane's split).  Larger word <=> larger value, or
// equal value and earlier row, so inserting into a descending list is one median-of-three per slot instead of compares and
// selects on two arrays.  Two elements are converted together, by three packed 16-bit operations, and one more each puts the row
// beside it.  Which zeros were -0 is looked up in the row at the end, if any is left in a queue.  INT_MIN = empty (no
// magnitude is 0x8000).  (A wavefront that ends with a zero loads all its survivors' elements again: nothing measurable where they
// are the rows' first ones, 2 us where they lie all over the rows: 2048 x 8192, half of it -0, b = 512, 20.1 -> 22.3 us, as many loads in flight as
// there are survivors or a column's: the fetch itself is what takes it.)  Unpacked queues of two slots take 10.4 instructions per element, which the SIMDs issued in 79 % of their
// cycles on 128 x 2653751; these take 5 and leave such rows to memory: 136 -> 126 us (5.4 TB/s; k_b = 1: 112), 1024 x 131072,
// b = 512: 56 -> 48.  (A conversion element by element that carried "was -0" in the word took 6 more per element: no gain at two slots.)
constexpr int32_t kEmptyPk = (int32_t)0x80000000u;
typedef int16_t pk2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_keys(uint32_t w) {  // two elements
    const pk2 v = __builtin_bit_cast(pk2, w);
    const pk2 sgn = v >> 15;
    const uint32_t m = (w & 0x7fff7fffu) ^ __builtin_bit_cast(uint32_t, sgn);
    return __builtin_bit_cast(uint32_t, (pk2)(__builtin_bit_cast(pk2, m) - sgn));
}
__device__ __forceinline__ int32_t pack_bf16(uint32_t xb, uint32_t code) {  // xb: the bf16 in the high half
    return (int32_t)((pack_keys(xb) & 0xffff0000u) | code);
}
__device__ __forceinline__ void unpack_bf16(int32_t c, int t_first, float &v, int &t) {
    const uint32_t key = (uint32_t)c & 0xffff0000u;
    const uint32_t bits = c < 0 ? ((0u - key) | 0x80000000u) : key;
    v = __uint_as_float(c == kEmptyPk ? 0x7fc00000u : bits);
    t = c == kEmptyPk ? kEmptyT : t_first + 0xffff - (int)((uint32_t)c & 0xffffu);
}
template <int KB>
__device__ __forceinline__ void insert_pk(int32_t (&q)[KB], int32_t c) {
#pragma unroll
    for (int j = KB - 1; j >= 1; --j) q[j] = med3_i32(q[j - 1], q[j], c);  // q[j-1] >= q[j]: c clamped between them
    q[0] = max(q[0], c);
}
// mine <- the N largest of (mine U theirs); both sorted descending, result sorted descending.
template <int N>
__device__ __forceinline__ void merge_pk(int32_t (&mine)[N], const int32_t (&theirs)[N]) {
#pragma unroll
    for (int j = 0; j < N; ++j) mine[j] = max(mine[j], theirs[N - 1 - j]);
#pragma unroll
    for (int stride = N / 2; stride >= 1; stride >>= 1)
#pragma unroll
        for (int i = 0; i < N; ++i)
            if ((i & stride) == 0) {
                const int32_t a = mine[i], c = mine[i + stride];
                mine[i] = max(a, c);
                mine[i + stride] = min(a, c);
            }
}
template <int ELT, int V, int KB>
__device__ __forceinline__ void scan_vec_pk(int32_t (&q)[V][KB], const RowVec<ELT, V> &v, int t_local) {
    const uint32_t code = (uint32_t)(0xffff - t_local);
    int32_t c[V];
    if constexpr (V == 1) {
        c[0] = pack_bf16(v.w[0] << 16, code);
    } else {
#pragma unroll
        for (int w = 0; w < V / 2; ++w) {
            const uint32_t keys = pack_keys(v.w[w]);
            c[2 * w] = (int32_t)((keys << 16) | code);
            c[2 * w + 1] = (int32_t)((keys & 0xffff0000u) | code);
        }
    }
    if (KB >= 8) {  // the insertion is cheap: only long queues are worth a wavefront-uniform skip
        bool any = false;
#pragma unroll
        for (int e = 0; e < V; ++e) any = any || c[e] > q[e][KB - 1];
        if (__ballot(any) == 0ull) return;
    }
#pragma unroll
    for (int e = 0; e < V; ++e) insert_pk<KB>(q[e], c[e]);
}

#endif  // __HIPCC__

}  // namespace atk
