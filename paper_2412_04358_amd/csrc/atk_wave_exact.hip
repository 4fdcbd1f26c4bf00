// exact_topk of short bf16 rows, a wavefront each: the row in its registers, a bound that k elements reach, the few elements that do in a list in
// LDS, and these sorted in registers (atk_wave_sort.h).
//
//   1. A lane holds up to 16 vectors of 16 bytes.  A lower bound on the k-th largest: of 1024 or 2048 groups of elements (16 or 32 to a lane) the
//      k-th largest maximum, or one a little below, by interpolation and halving; two elements to an instruction, as signed 16-bit numbers.  Where the
//      bound is above zero that is right for bf16 as it stands (what is negative is below it, whatever its order); else the row is
//      converted to two's complement first (2048 x 8192, k = 512, logarithms of probabilities: 15.9 us, 13.5 for N(0,1)).
//   2. The elements that reach the bound are marked, three instructions to two of them, and listed in LDS one mark at a time; every lane then takes an
//      equal share of the list, with the values from a copy of the row in LDS (registers have no index).
//   3. Where more reach it than the list holds (rows unlike their groups: masked in part; ties), the value of the k-th is searched
//      among all elements, and of ties at it the first are marked, until there are k.  (Element by element in all the row's vectors: 7 x 7000 of
//      three values, k = 36, 13.2 us; whole vectors but for the one where they end, and none behind it: 7.1, ex_row_kernel 8.2.)
//   4. The list is sorted, cut to the k largest.
// Rows of up to 1024 elements are sorted as a whole.
//
// What bounds it: vector instructions, with two rows to a SIMD about 2400 for each of 8192 elements and k = 512, of which the sort takes 1050, the bound 660, the list
// and its values 500.  2048 x 8192, k = 512: 19.4 us (ex_row_kernel, 29 instructions an element) -> 15.7; k = 64: 12.7 -> 10.9; on a grid of halves,
// k = 512: 112 -> 32; 2048 x 4096, k = 256: 12.3 -> 10.4; 512 x 1024, k = 512: 0.17 times as long; 2048 x 8192 of one value, k = 512: 34.4 -> 15.5.
#include <cmath>
#include <cstring>
#include <utility>

#include "atk_common.h"
#include "atk_exact.h"
#include "atk_packed.h"
#include "atk_select.h"
#include "atk_stream.h"
#include "atk_wave_out.h"
#include "atk_wave_sort.h"

namespace atk {

struct WaveExactParams {
    const void *x;
    void *out_vals;
    int32_t *out_idx;
    int64_t n;
    int k;
    int vec_store;
};

constexpr uint32_t kNoKeys = 0x80008000u;  // two elements that are none: below every key
__device__ __forceinline__ pk2 as_pk(uint32_t w) { return __builtin_bit_cast(pk2, w); }
__device__ __forceinline__ uint32_t of_pk(pk2 v) { return __builtin_bit_cast(uint32_t, v); }

template <int NV>
__device__ __forceinline__ void wave_load_row(uint32_t (&q)[NV * 4], const uint16_t *row, int n_vec) {
    const int lane = threadIdx.x;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int v = j * kWave + lane;
        const RowVec<ATK_BF16, 8> one = load_vec<ATK_BF16, 8>((const unsigned char *)row + (v < n_vec ? v : 0) * 16);
#pragma unroll
        for (int i = 0; i < 4; ++i) q[4 * j + i] = one.w[i];
    }
}
template <int NV>
__device__ __forceinline__ void wave_mask_row(uint32_t (&q)[NV * 4], int n_vec) {
    if (n_vec >= NV * kWave) return;
#pragma unroll
    for (int j = 0; j < NV; ++j)
        if ((j + 1) * kWave > n_vec) {  // (uniform: the row's last vectors alone)
#pragma unroll
            for (int i = 0; i < 4; ++i) q[4 * j + i] = j * kWave + (int)threadIdx.x < n_vec ? q[4 * j + i] : kNoKeys;
        }
}

// How many of the wavefront's 128 * N numbers reach `from` (above -32768), three operations to two of them.  (Ballots and scalar counts of them, two to
// a number, wait for one another: 2048 x 8192, k = 1, 12.4 us with them in the search of the bound.)
template <int N>
__device__ __forceinline__ int reached(const uint32_t (&q)[N], int from) {
    const pk2 below = {(int16_t)(from - 1), (int16_t)(from - 1)};
    pk2 sum = {0, 0};
#pragma unroll
    for (int i = 0; i < N; ++i) sum -= __builtin_elementwise_sub_sat(below, as_pk(q[i])) >> 15;
    const uint32_t all = wave_incl_scan_u32((uint32_t)((int)sum.x + (int)sum.y));
    return __builtin_amdgcn_readlane((int)all, kWave - 1);
}
__host__ __device__ constexpr int wave_slack(int k) { return k / 16 > 8 ? k / 16 : 8; }  // maxima above the bound that the k-th is let go for

// Rows of up to 512 * NV elements, sorted as a whole
template <int NV, int R>
__global__ void __launch_bounds__(64, 2) wave_all_kernel(WaveExactParams p) {
    constexpr int W = 8 * NV;
    const int lane = threadIdx.x;
    const int64_t r = blockIdx.x;
    const uint16_t *row = (const uint16_t *)p.x + r * p.n;
    uint32_t q[NV * 4];
    wave_load_row<NV>(q, row, (int)p.n / 8);
    int32_t w[W], top[R];
#pragma unroll
    for (int i = 0; i < W / 2; ++i) {
        const uint32_t keys = pack_keys(q[i]), code = 0xffffu - (uint32_t)((i / 4) * kWave * 8 + lane * 8 + (i % 4) * 2);
        w[2 * i] = (int32_t)((keys << 16) | code);
        w[2 * i + 1] = (int32_t)((keys & 0xffff0000u) | (code - 1u));
    }
    if ((int)p.n < NV * kWave * 8) {
#pragma unroll
        for (int i = 0; i < W; ++i) w[i] = (i / 8) * kWave + lane < (int)p.n / 8 ? w[i] : kEmptyPk;
    }
    const LanePlace at;
    wave_largest<W, R, 1>(w, top, at);
    wave_write<R>(row, (uint16_t *)p.out_vals + r * p.k, p.out_idx + r * p.k, p.k, p.vec_store, R * at.place, top);
}

// Longer ones: k <= 128 * H, and a list of up to 192 * H elements.  G: words of groups' maxima per lane, two groups each - the same word of a
// half (8) or a quarter (16) of the lane's vectors side by side, so that rows masked from the middle on keep half of their groups, and in rows in
// order the largest elements are maxima of their own.
template <int NV, int H, int G>
__global__ void __launch_bounds__(64, 2) wave_exact_kernel(WaveExactParams p) {
    constexpr int Q = NV * 4, M = NV / 4;  // words of the row, masks
    constexpr int S = NV / (G / 4);        // vectors side by side that a group is of
    constexpr uint32_t cap = 192 * H;
    static_assert(NV % 4 == 0, "whole masks");
    __shared__ __align__(16) uint32_t keys[NV * kWave * 4];
    __shared__ uint16_t list[cap + kWave];
    const int lane = threadIdx.x, k = p.k, n_vec = (int)p.n / 8;
    const int64_t r = blockIdx.x;
    const uint16_t *row = (const uint16_t *)p.x + r * p.n;
    uint32_t q[Q];
    wave_load_row<NV>(q, row, n_vec);
    wave_mask_row<NV>(q, n_vec);
    // ---- the bound t: k elements reach it; most: the largest element
    int t, most;
    for (bool keyed = false;; keyed = true) {
        uint32_t mx[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            pk2 m = as_pk(q[(g >> 2) * 4 * S + (g & 3)]);
#pragma unroll
            for (int j = 1; j < S; ++j) m = __builtin_elementwise_max(m, as_pk(q[(g >> 2) * 4 * S + 4 * j + (g & 3)]));
            mx[g] = of_pk(m);
        }
        pk2 hi = as_pk(mx[0]);
#pragma unroll
        for (int g = 1; g < G; ++g) hi = __builtin_elementwise_max(hi, as_pk(mx[g]));
        // (as an unsigned number, for the wavefront's maximum)
        most = (int)wave_max_u32((uint32_t)(max((int)hi.x, (int)hi.y) + 32768)) - 32768;
        const int least = keyed ? -32767 : 1;
        auto reach = [&](int from) { return reached<G>(mx, from); };  // maxima that do
        // from the largest element down by two binades, eight, ..., then between what k maxima reach and what they do not, by
        // interpolation on the numbers that do: about four counts (halving the range of all positive numbers took fourteen)
        int h = most + 1, n_h = 0, n_t = 0;  // n_h < k reach h, n_t reach t
        for (int d = 256;; d *= 4) {
            t = max(most - d, least);
            n_t = most < least ? 0 : reach(t);
            if (n_t >= k || t == least) break;
            h = t;
            n_h = n_t;
        }
        if (n_t < k) {  // (uniform, as all of this is)
            if (keyed) break;  // rows shorter than their groups: all elements reach it
#pragma unroll
            for (int i = 0; i < Q; ++i) q[i] = pack_keys(q[i]);
            wave_mask_row<NV>(q, n_vec);
            continue;
        }
        const bool steep = 6 * k < 128 * G;  // far from the middle they fall off as an exponential does
        auto level = [&](int cnt) { return steep ? __builtin_amdgcn_logf((float)cnt + 0.5f) : (float)cnt; };
        for (int step = 1; h - t > 1 && n_t > k + wave_slack(k); ++step) {
            int mid = t + (h - t) / 2;
            if (step % 3) {
                const float low = level(n_h), part = (level(k + wave_slack(k) / 2) - low) * __builtin_amdgcn_rcpf(level(n_t) - low);
                mid = min(max(h - (int)((float)(h - t) * part), t + 1), h - 1);
            }
            const int cnt = reach(mid);
            if (cnt < k) {
                h = mid;
                n_h = cnt;
            } else {
                t = mid;
                n_t = cnt;
            }
        }
        break;
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) ((uint4 *)keys)[j * kWave + lane] = make_uint4(q[4 * j], q[4 * j + 1], q[4 * j + 2], q[4 * j + 3]);
    // ---- marks: bit 16 h + 4 (j % 4) + i of mask j / 4: element h of word i of vector j
    uint32_t mk[M];
    auto mark = [&](uint32_t (&to)[M], int from) {
        const pk2 below = {(int16_t)(from - 1), (int16_t)(from - 1)};
#pragma unroll
        for (int w = 0; w < M; ++w) {
            uint32_t m = 0u;
#pragma unroll
            for (int i = 0; i < 16; ++i) m = (m >> 1) | (of_pk(__builtin_elementwise_sub_sat(below, as_pk(q[16 * w + i]))) & 0x80008000u);
            to[w] = m;
        }
    };
    auto count = [&](const uint32_t (&of)[M]) {  // this lane's
        uint32_t c = 0;
#pragma unroll
        for (int w = 0; w < M; ++w) c += (uint32_t)__popc(of[w]);
        return c;
    };
    mark(mk, t);
    uint32_t mine = count(mk), incl = wave_incl_scan_u32(mine);
    uint32_t n_list = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
    if (n_list > cap) {
        // a bound that no more than the list holds reach, or the k-th largest value
        int h = most + 1;  // fewer than k reach it
        while (h - t > 1) {
            const int mid = t + (h - t) / 2, cnt = reached<Q>(q, mid);
            if (cnt < k) {
                h = mid;
            } else {
                t = mid;
                if (cnt <= (int)cap) break;
            }
        }
        mark(mk, t);
        mine = count(mk);
        incl = wave_incl_scan_u32(mine);
        n_list = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
        if (n_list > cap) {  // ties at it: the first ones.  They are counted by rows of vectors: lanes side by side hold vectors side by side
            uint32_t above[M];
            mark(above, t + 1);
            const uint32_t higher = wave_incl_scan_u32(count(above));
            int left = k - __builtin_amdgcn_readlane((int)higher, kWave - 1);
#pragma unroll
            for (int w = 0; w < M; ++w) {
                uint32_t ties = mk[w] & ~above[w], kept = 0u;
#pragma clang loop unroll(disable)
                for (int j = 0; j < 4 && left > 0; ++j) {
                    const uint32_t here = ties & (0x000f000fu << (4 * j)), n_here = (uint32_t)__popc(here), to_here = wave_incl_scan_u32(n_here);
                    int room = left - (int)(to_here - n_here);
                    if ((int)n_here <= room) {
                        kept |= here;
                    } else if (room > 0) {  // (one lane of the row)
#pragma clang loop unroll(disable)
                        for (int e = 0; e < 8 && room > 0; ++e) {  // in the order of the row
                            const uint32_t bit = 1u << ((e & 1) * 16 + 4 * j + (e >> 1));
                            if (here & bit) {
                                kept |= bit;
                                --room;
                            }
                        }
                    }
                    left -= __builtin_amdgcn_readlane((int)to_here, kWave - 1);
                }
                mk[w] = above[w] | kept;
            }
            mine = count(mk);
            incl = wave_incl_scan_u32(mine);
            n_list = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
        }
    }
    // ---- the list
    {
        // (a mark of every mask at a time: the lanes that have none left write past the list)
        uint32_t to = incl - mine, any = 0u;
#pragma unroll
        for (int w = 0; w < M; ++w) any |= mk[w];
        while (__ballot(any != 0u) != 0ull) {
            any = 0u;
#pragma unroll
            for (int w = 0; w < M; ++w) {
                const bool on = mk[w] != 0u;
                list[on ? to : cap + lane] = (uint16_t)((uint32_t)(w << 11 | lane << 5) | (uint32_t)(__ffs((int)mk[w]) - 1));
                to += on ? 1u : 0u;
                mk[w] &= mk[w] - 1u;
                any |= mk[w];
            }
        }
    }
    __syncthreads();  // (one wavefront: the LDS writes are waited for)
    int32_t w[3 * H], top[2 * H];
    {
        uint32_t entry[3 * H];
#pragma unroll
        for (int i = 0; i < 3 * H; ++i) entry[i] = list[i * kWave + lane];  // (past the list's end: anything, within the row)
        int pos[3 * H];
#pragma unroll
        for (int i = 0; i < 3 * H; ++i) {
            const uint32_t b = entry[i] & 31u;
            pos[i] = (int)(((entry[i] & 0x1800u) | ((b & 12u) << 7)) | ((entry[i] >> 2) & 0x1f8u) | ((b & 3u) << 1) | (b >> 4));
            if (M < 4) pos[i] = min(pos[i], NV * kWave * 8 - 1);
        }
        uint32_t key[3 * H];
#pragma unroll
        for (int i = 0; i < 3 * H; ++i) key[i] = ((const uint16_t *)keys)[pos[i]];
#pragma unroll
        for (int i = 0; i < 3 * H; ++i)
            w[i] = (uint32_t)(i * kWave + lane) < n_list ? (int32_t)((key[i] << 16) | (0xffffu - (uint32_t)pos[i])) : kEmptyPk;
    }
    // ---- sorted
    const LanePlace at;
    wave_largest_two_of_three<H>(w, top, at);
    uint16_t *vals = (uint16_t *)p.out_vals + r * k;
    int32_t *idx = p.out_idx + r * k;
    int32_t part[H];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
#pragma unroll
        for (int i = 0; i < H; ++i) part[i] = top[c * H + i];
        wave_write<H>(row, vals, idx, k, p.vec_store, c * kWave * H + H * at.place, part);
    }
}

// ------------------------------------------------------------------------------------ host
bool plan_wave_exact(int64_t m, int64_t n, int64_t k, int dtype, bool ptr16, WaveExactPlan *out) {
    if (dtype != ATK_BF16 || !ptr16 || n % 8 || n > 8192) return false;
    WaveExactPlan p;
    memset(&p, 0, sizeof p);
    // Against ex_row_kernel over 1 to 8192 rows of 520 to 8192 elements, 19 values of k, whole rows 0.13 to 0.99 times as long (2048 x 512, k = 256: 0.22)
    // but for few winners in large batches, which need no sort of all elements (8192 x 1024, k = 1: 1.17); with a bound and a list 0.27 to 1.05 on N(0,1)
    // and 0.54 to 1.16 on logarithms of probabilities, which are converted first, where it is taken.  A few rows leave a wavefront's steps nobody's to hide behind, and
    // four wavefronts have them in less time (256 x 8192, k = 512: 1.28): then only rows of up to 2048 elements (0.26 to 0.98, logarithms to 1.1) and short
    // lists (0.72 to 1.04, logarithms to 1.12).  The list's sort is as long as the next power of two of k needs: where k is little above one, and the
    // row short against it or the sort the longer part, ex_row_kernel has the row sooner -
    //   k > 512 on 1537 to 2304 elements        0.49 to 1.32, logarithms 0.81 to 1.55, one value 0.8 to 1.75
    //   k up to 575 on more than 4096           0.87 to 1.12, logarithms 0.96 to 1.30
    //   k from 257 to 384 on more than 6144, from 2049 rows on   1.00 to 1.07, logarithms 1.07 to 1.21 (up to 2048 rows 0.81 to 1.01 and 0.92 to 1.14)
    const bool forced = plan_override().wv > 0;
    if (!forced && n <= 1024 && ((n > 512 && m > 1024 && k < 128) || (m > 4096 && k < 32))) return false;
    if (!forced && n > 2048 && m < 1024 && k > 64) return false;
    if (!forced && ((k > 512 && n > 1536 && n <= 2304) || (k > 512 && k < 576 && n > 4096) || (k > 256 && k <= 384 && n > 6144 && m > 2048))) return false;
    if (n <= 1024) {
        p.NV = n <= 512 ? 1 : 2;
        p.R = 8 * p.NV;
        while (p.R > p.NV && 64ll * (p.R / 2) >= k) p.R /= 2;
        *out = p;
        return true;
    }
    for (int nv : {4, 8, 12, 16})
        if (!p.NV && n <= 512 * nv) p.NV = nv;
    for (const auto &hg : {std::pair<int, int>(1, 8), std::pair<int, int>(1, 16), std::pair<int, int>(2, 16), std::pair<int, int>(4, 16), std::pair<int, int>(8, 16)}) {
        const int h = hg.first, g = p.NV == 4 ? 8 : hg.second;
        if (k > 128 * h) continue;
        // elements expected to reach the bound: among random ones the share above the k-th (and the slack) of the maxima of so many groups
        const double groups = 128.0 * g, rank = (double)(k + wave_slack((int)k)), e = (double)n / groups;
        if (rank > 0.9 * groups) continue;
        const double expect = (double)n * (1.0 - std::pow(1.0 - rank / groups, 1.0 / e));
        if (expect + 4.0 * std::sqrt(expect) > 192.0 * h) continue;
        p.H = h;
        p.G = g;
        *out = p;
        return true;
    }
    return false;
}

template <typename K>
static hipError_t launch_rows(K kernel, const WaveExactParams &prm, int64_t m, hipStream_t stream) {
    constexpr int64_t rows = (1ll << 31) / kWave;  // (a launch holds fewer than 2^32 lanes)
    WaveExactParams now = prm;
    for (int64_t r0 = 0; r0 < m; r0 += rows) {
        now.x = (const uint16_t *)prm.x + r0 * prm.n;
        now.out_vals = (uint16_t *)prm.out_vals + r0 * prm.k;
        now.out_idx = prm.out_idx + r0 * prm.k;
        hipLaunchKernelGGL(kernel, dim3((unsigned)(m - r0 < rows ? m - r0 : rows)), dim3(kWave), 0, stream, now);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_wave_exact(const WaveExactPlan &pl, int64_t m, int64_t n, int64_t k, const void *x, void *out_vals, int32_t *out_idx, hipStream_t stream) {
    WaveExactParams prm;
    memset(&prm, 0, sizeof prm);
    prm.x = x;
    prm.out_vals = out_vals;
    prm.out_idx = out_idx;
    prm.n = n;
    prm.k = (int)k;
    const int words = pl.R ? pl.R : pl.H, piece = words < 8 ? words : 8;
    prm.vec_store = k % piece == 0 && (((uintptr_t)out_vals | (uintptr_t)out_idx) & 15u) == 0;
#define ATK_ALL(NV_, R_) \
    if (pl.NV == NV_ && pl.R == R_) return launch_rows(wave_all_kernel<NV_, R_>, prm, m, stream);
    ATK_ALL(1, 1) ATK_ALL(1, 2) ATK_ALL(1, 4) ATK_ALL(1, 8) ATK_ALL(2, 2) ATK_ALL(2, 4) ATK_ALL(2, 8) ATK_ALL(2, 16)
#undef ATK_ALL
#define ATK_EX(NV_, H_, G_) \
    if (!pl.R && pl.NV == NV_ && pl.H == H_ && pl.G == G_) return launch_rows(wave_exact_kernel<NV_, H_, G_>, prm, m, stream);
    ATK_EX(4, 1, 8) ATK_EX(4, 2, 8) ATK_EX(4, 4, 8) ATK_EX(4, 8, 8)
    ATK_EX(8, 1, 8) ATK_EX(8, 1, 16) ATK_EX(8, 2, 16) ATK_EX(8, 4, 16) ATK_EX(8, 8, 16)
    ATK_EX(12, 1, 8) ATK_EX(12, 1, 16) ATK_EX(12, 2, 16) ATK_EX(12, 4, 16) ATK_EX(12, 8, 16)
    ATK_EX(16, 1, 8) ATK_EX(16, 1, 16) ATK_EX(16, 2, 16) ATK_EX(16, 4, 16) ATK_EX(16, 8, 16)
#undef ATK_EX
    return hipErrorInvalidValue;
}

}  // namespace atk
