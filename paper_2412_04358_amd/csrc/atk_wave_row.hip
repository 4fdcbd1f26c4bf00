// approx_topk of bf16 rows that one wavefront takes from the first load to the last output: batches that give the chip's SIMDs a row
// or two each, where Stage 2 over lists in LDS (or in scratch, by a launch of its own) is a chain of short steps with a barrier
// after each.
//
//   1. A lane owns V adjacent columns of the row seen as a matrix (NG times that, 64 V columns apart) and walks down all matrix rows,
//      as in atk_stage1.hip, with queues of packed words.
//   2. The queues' words exchange the matrix row for the column index, which 16 bits hold, and are the candidates as they stand: larger word,
//      larger value or equal value and lower index.
//   3. The wavefront sorts them in its registers (atk_wave_sort.h), cut to the k largest on the way, and lane l has the l-th stretch of the output.
// No LDS, no barrier, no scratch, no second launch, and the same time for rows without order, sorted ones and ties.
//
// What bounds it: on 2048 rows, two to a SIMD, the sort of the rows that are in last, after the memory's 7 us (1270 vector instructions a row where 512 of
// 1024 words are wanted, one in four cycles: 2.1 us); with more rows memory (3.6 us per 1024 rows of 8192).  2048 x 8192, k = 512, b = 512,
// k_b = 2: 20.0 -> 12.1 us a call (Stage 1 and the selection from its pairs before, two launches), values on a grid of halves 55 -> 13.5;
// 4 x 4096, k = 256, b = 512: 12.6 -> 4.7.  (Against the other plans as they are by now, one launch on preallocated outputs: 19.4 -> 11.4 and
// 5.6 -> 3.6.)
#include <cstring>

#include "atk_common.h"
#include "atk_packed.h"
#include "atk_stream.h"
#include "atk_wave_out.h"
#include "atk_wave_sort.h"

namespace atk {

struct WaveParams {
    const void *x;
    void *out_vals;
    int32_t *out_idx;
    int64_t n;
    int b, L, rem;    // columns, full matrix rows, columns of the ragged last one
    int k, k_b;
    int whole;        // every lane has columns, every slot a survivor
    int vec_store;    // outputs in pieces of min(R, 8) words start on boundaries of as many
};

template <int V, int NG, int KB, int R>
__global__ void __launch_bounds__(64, 2) wave_row_kernel(WaveParams p) {
    constexpr int W = V * NG * KB, VW = NG * (V < 2 ? 1 : V / 2), U = VW > 4 ? 64 / VW : 16;  // U matrix rows' loads to a batch, VW registers each
    constexpr int RUN = KB < R ? KB : 1;
    typedef RowVec<ATK_BF16, V> Vec;
    const int lane = threadIdx.x;
    const uint32_t row_bytes = (uint32_t)p.b * 2u;
    const LanePlace at;
    int col0[NG];
    uint32_t off[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        col0[g] = (g * kWave + lane) * V;
        off[g] = col0[g] < p.b ? (uint32_t)col0[g] * 2u : 0u;  // (a lane without columns reads the first ones)
    }
    const int64_t r = blockIdx.x;
    const unsigned char *row = (const unsigned char *)p.x + r * p.n * 2;
    int32_t q[NG * V][KB];
#pragma unroll
    for (int c = 0; c < NG * V; ++c)
#pragma unroll
        for (int j = 0; j < KB; ++j) q[c][j] = kEmptyPk;
    auto feed = [&](const Vec &vec, int g, int t) {
        int32_t part[V][KB];
#pragma unroll
        for (int e = 0; e < V; ++e)
#pragma unroll
            for (int j = 0; j < KB; ++j) part[e][j] = q[g * V + e][j];
        scan_vec_pk<ATK_BF16, V, KB>(part, vec, t);
#pragma unroll
        for (int e = 0; e < V; ++e)
#pragma unroll
            for (int j = 0; j < KB; ++j) q[g * V + e][j] = part[e][j];
    };
    // ---- Stage 1.  The next batch is asked for before this one is worked on.
    {
        Vec v[U][NG], ahead[U][NG];
        auto load = [&](Vec (&to)[U][NG], int t) {  // matrix rows t, t + 1, ...; past the last one that again
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const unsigned char *from = row + (uint32_t)min(t + u, p.L - 1) * row_bytes;
#pragma unroll
                for (int g = 0; g < NG; ++g) to[u][g] = load_vec<ATK_BF16, V>(from + off[g]);
            }
        };
        load(v, 0);
        for (int t = 0; t < p.L; t += U) {
            if (t + U < p.L) load(ahead, t + U);
            __builtin_amdgcn_sched_barrier(0);
            if (t + U <= p.L) {
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int g = 0; g < NG; ++g) feed(v[u][g], g, t + u);
            } else {
#pragma unroll
                for (int u = 0; u < U - 1; ++u)
                    if (t + u < p.L) {  // uniform
#pragma unroll
                        for (int g = 0; g < NG; ++g) feed(v[u][g], g, t + u);
                    }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int g = 0; g < NG; ++g) v[u][g] = ahead[u][g];
        }
        if (p.rem > 0) {  // the ragged last matrix row: its first p.rem columns, which end where the row does
            const unsigned char *last = row + (uint32_t)p.L * row_bytes;
#pragma unroll
            for (int g = 0; g < NG; ++g)
                if (col0[g] + V <= p.rem) {  // (rem is a multiple of V, as n and b are)
                    const Vec one = load_vec<ATK_BF16, V>(last + off[g]);
                    feed(one, g, p.L);
                }
        }
    }
    // ---- candidates: [31:16] the value, [15:0] 0xffff - index
    int32_t w[W];
#pragma unroll
    for (int c = 0; c < NG * V; ++c) {
        const uint16_t first = (uint16_t)(0xffffu - 0xffffu * (uint32_t)p.b - (uint32_t)(col0[c / V] + c % V));
        const bool flip = RUN > 1 && (c & 1);
#pragma unroll
        for (int j = 0; j < KB; ++j) {
            const uint16_t low = (uint16_t)((uint16_t)q[c][j] * (uint16_t)p.b + first);
            w[c * KB + (flip ? KB - 1 - j : j)] = (int32_t)(((uint32_t)q[c][j] & 0xffff0000u) | low);
        }
    }
    if (!p.whole) {
#pragma unroll
        for (int c = 0; c < NG * V; ++c)
#pragma unroll
            for (int j = 0; j < KB; ++j) {
                int32_t &word = w[c * KB + (RUN > 1 && (c & 1) ? KB - 1 - j : j)];
                word = col0[c / V] < p.b && j < p.k_b ? word : kEmptyPk;
            }
    }
    // ---- Stage 2
    int32_t top[R];
    wave_largest<W, R, RUN>(w, top, at);
    wave_write<R>((const uint16_t *)p.x + r * p.n, (uint16_t *)p.out_vals + r * p.k, p.out_idx + r * p.k, p.k, p.vec_store, R * at.place, top);
}

// ------------------------------------------------------------------------------------ host
// Instances: X(columns per lane V, column groups NG, slots KB); each with R = W, W/2, W/4 and W/8 of its W = V * NG * KB words per lane
#define ATK_WAVE_INSTANCES(X)                                                                                                                              \
    X(8, 1, 1) X(8, 1, 2) X(8, 1, 4) X(8, 2, 1) X(8, 2, 2) X(4, 1, 1) X(4, 1, 2) X(4, 1, 4) X(4, 1, 8) X(2, 1, 2) X(2, 1, 4) X(2, 1, 8)                    \
    X(2, 2, 1) X(2, 2, 2) X(2, 2, 4) X(2, 4, 1) X(2, 4, 2) X(2, 8, 1) X(2, 8, 2)                                                                           \
    X(1, 2, 2) X(1, 2, 4) X(1, 2, 8) X(1, 4, 1) X(1, 4, 2) X(1, 4, 4) X(1, 8, 1) X(1, 8, 2) X(1, 16, 1) X(1, 16, 2)

bool plan_wave_row(int64_t m, int64_t n, int64_t k, int64_t b, int64_t k_b, int dtype, bool ptr16, WavePlan *out) {
    if (dtype != ATK_BF16 || !ptr16 || n > 65536 || b * k_b <= k) return false;
    WavePlan p;
    memset(&p, 0, sizeof p);
    p.KB = 1;
    while (p.KB < k_b) p.KB *= 2;
#define ATK_X(VV, GG, KK)                                                                                                       \
    if (!p.V && p.KB == KK && b <= 64 * VV * GG && b > 32 * VV * GG && b % VV == 0 && n % VV == 0 && (GG == 1 || b > 64 * VV)) { \
        p.V = VV;                                                                                                               \
        p.NG = GG;                                                                                                              \
    }
    ATK_WAVE_INSTANCES(ATK_X)
#undef ATK_X
    if (!p.V) return false;
    // Bucket counts or row lengths that leave loads of one or two elements, in more groups: short rows, batches that give a SIMD a second row to issue
    // from, or so many winners that the selection replaced is the longer part.  Against the plans replaced, 649 calls (4 to 4000 rows of 2047 to 12288
    // elements, 99 to 1023 buckets): 0.08 to 1.04 times as long where this says so, half of them below 0.49 (4 x 3816, k = 402, b = 201, k_b = 4:
    // 39.8 -> 7.3 us, 7.4 -> 6.9 since a workgroup's ranks no longer go through their bins one lane at a time; 256 x 8190, k = b = 1023, k_b = 2:
    // 37.3 -> 12.4, both then and now; 2048 x 12288 0.16 to 1.04, but 1500 rows of them 1.27); elsewhere up to 1.8.
    if (p.V < 4 && p.NG > 1 && plan_override().wv <= 0 &&
        !(n <= 2048 || (n <= 4096 && m >= 1024) || (n <= 8192 && (m >= 2048 || (k > 256 && k > 96 * p.KB)))))
        return false;
    const int W = p.V * p.NG * p.KB;
    p.R = W;
    while (p.R > 1 && p.R > W / 8 && 64ll * (p.R / 2) >= k) p.R /= 2;
    if (64ll * p.R < k) return false;
    *out = p;
    return true;
}

template <int V, int NG, int KB, int R>
static hipError_t launch_wave(const WaveParams &prm, int64_t m, hipStream_t stream) {
    constexpr int64_t rows = (1ll << 31) / kWave;  // (a launch holds fewer than 2^32 lanes)
    WaveParams now = prm;
    for (int64_t r0 = 0; r0 < m; r0 += rows) {
        now.x = (const uint16_t *)prm.x + r0 * prm.n;
        now.out_vals = (uint16_t *)prm.out_vals + r0 * prm.k;
        now.out_idx = prm.out_idx + r0 * prm.k;
        hipLaunchKernelGGL((wave_row_kernel<V, NG, KB, R>), dim3((unsigned)(m - r0 < rows ? m - r0 : rows)), dim3(kWave), 0, stream, now);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_wave_row(const WavePlan &pl, int64_t m, int64_t n, int64_t k, int64_t b, int64_t k_b, const void *x, void *out_vals,
                           int32_t *out_idx, hipStream_t stream) {
    WaveParams prm;
    memset(&prm, 0, sizeof prm);
    prm.x = x;
    prm.out_vals = out_vals;
    prm.out_idx = out_idx;
    prm.n = n;
    prm.b = (int)b;
    prm.L = (int)(n / b);
    prm.rem = (int)(n % b);
    prm.k = (int)k;
    prm.k_b = (int)k_b;
    prm.whole = b == 64ll * pl.V * pl.NG && k_b == pl.KB;
    const int piece = pl.R < 8 ? pl.R : 8;
    prm.vec_store = k % piece == 0 && (((uintptr_t)out_vals | (uintptr_t)out_idx) & 15u) == 0;
#define ATK_X(VV, GG, KK)                                                            \
    if (pl.V == VV && pl.NG == GG && pl.KB == KK) {                                  \
        constexpr int W = VV * GG * KK;                                              \
        if (pl.R == W) return launch_wave<VV, GG, KK, W>(prm, m, stream);            \
        if (pl.R == W / 2) return launch_wave<VV, GG, KK, W / 2>(prm, m, stream);    \
        if (pl.R == W / 4) return launch_wave<VV, GG, KK, W / 4>(prm, m, stream);    \
        if (W >= 8 && pl.R == W / 8) return launch_wave<VV, GG, KK, W >= 8 ? W / 8 : W>(prm, m, stream); \
    }
    ATK_WAVE_INSTANCES(ATK_X)
#undef ATK_X
    return hipErrorInvalidValue;
}

}  // namespace atk
