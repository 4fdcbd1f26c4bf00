// exact_topk of long rows with many winners: the elements are dealt to value-ordered bins in one sweep over the row, and
// every bin is ordered by a workgroup of its own.
//
//   ex_sample_kernel  one workgroup per row: a sample of 32768 elements (runs of 64 bytes, one at a random place in
//                     every piece of the row) gives a threshold that a little more than k elements of the row reach, and cuts
//                     what lies above it into bins of about 1000 elements: unions of fine bins that are linear in (value
//                     key, index), so a bin's number is one multiplication and one look into a table.  Rows with long runs of ties
//                     are cut between elements of the sample instead, which is sorted for that.
//   ex_deal_kernel    a workgroup per 16384 elements: what reaches the threshold is brought into the order of the
//                     bins in LDS and written to the row's pool in one piece, with a table of where each bin starts.  (No bin has
//                     space set aside for it: however unevenly the sample cut the row, the pool is as full as the threshold lets
//                     through.)
//   ex_bins_kernel    a workgroup per bin: its pieces from all the chunks, ordered in LDS by a second set of bins and exact
//                     ranks, written to their places in the output.
//   ex_rest_rows_kernel (atk_exact.hip): rows that a sample misjudged (fewer than k candidates, or more than the pool
//                     holds) go digit by digit, one workgroup per row: slow, and rare, as the threshold has a margin of six
//                     deviations as the sample itself shows them.
//
// Every element is read once and every candidate written and read once more; memory is what bounds it: 128 x 2^20 f32,
// k = 2^18 reads 537 MB, writes and reads back 8 bytes for each of 1.06 k candidates and writes 268 MB of output.
// Measured there: 25 us to sample, 160 to deal (5 TB/s), 188 to order (2.9 TB/s; a chain of short steps per bin that seven
// workgroups of 256 lanes to a CU overlap - five with more tables in LDS took 262, two of 512 lanes 466), 4 for the last
// launch that finds nothing to do (under the tracer; the call takes 368), against 1113 by digit passes, a collecting sweep
// and a partition sort in 18 launches.  64 x 2^21 bf16, k = 2^19: 1690 -> 418.  us per call, by digit passes and here:
//                                      N(0,1)    first quarter -inf  ascending   constant    three levels  lagged average
//   128 x 2^20 f32, k = 2^18        1113, 368        1306, 410       1457, 904  2487, 1121    1484, 784      1101, 431
//   32 x 2^18 f32, k = 2^14           112, 42          119, 42        138, 105   176, 156      133, 53        112, 44
//   8 x 2^21 bf16, k = 2^19           327, 91         334, 112        480, 758   254, 237      222, 143       332, 113
//   one row of 2^20 f32, k = 2^18     107, 35           82, 44         99, 67     91, 120       96, 155       106, 44
#include <algorithm>
#include <cmath>
#include <cstring>

#include "atk_common.h"
#include "atk_exact.h"
#include "atk_exact_regs.h"
#include "atk_select.h"

namespace atk {

constexpr int kDealT = 1024;            // threads of the sampling and dealing workgroups
constexpr int kDealChunk = 16384;       // elements that a dealing workgroup takes
constexpr int kDealSample = 32768;      // sampled elements of a row
constexpr int kDealFine = 4096;         // fine bins
constexpr int kDealStage = 6144;        // candidates of a chunk that LDS holds (more: written where they belong one by one)
constexpr int kDealBinsMax = 1024;
constexpr int kDealBinMean = 1024;      // candidates per bin aimed at
constexpr int kBinT = 256;              // threads that order a bin
constexpr int kBinCap = 2048;           // candidates of a bin that LDS holds
constexpr int kBinSub = 1024;           // bins inside a bin
constexpr int kBinPeers = 4;            // places of a sub-bin that are looked at together
constexpr int kDealChunksMax = 512;     // chunks of a row
constexpr int kSplitLane = 7;           // sampled elements of a lane that are sorted where bins are cut at elements
constexpr int kSplitSample = kSplitLane * kDealT;

// What the rows of the sampling cost and save: the threshold lets through about 7 % more than k of a row's elements where k is a
// quarter of it, twice k where 64 sampled elements lie among the k largest (the least that is taken; with fewer the copy-out path of
// atk_exact.hip is there).
struct DealParams : RowParams {
    DealRow *rows;
    uint16_t *table;      // [row][kDealFine]: bin of each fine bin (0: the largest values); or [row][n_deal] composites: the lowest of each bin
    uint32_t *totals;     // [row][n_deal]: candidates per bin
    uint32_t *segs;       // [row][chunk][n_deal + 1]: where the chunk's piece of each bin starts in the row's pool
    u64 *pool;            // [row][pool_cap] candidates
    int64_t pool_cap;
    int n_deal, chunks;
    int sample_rank;      // elements of the sample above the threshold, at least
    int split_rank;
    float expect;         // elements of the sample among the k largest
};

// Sorts buf[0 .. n), largest first: a bitonic network in which the places past the end up to a power of two count as empty - every
// comparison puts the larger one first (the first step of a size pairs places mirrored in their block, the others places `stride`
// apart), so nothing is ever moved there.  Words up to 64 apart are compared by one wavefront, which then needs no barrier between
// steps.  Called by the whole workgroup after a barrier; ends in one.
__device__ __forceinline__ void sort_words(u64 *buf, int n) {
    int kp = 1;
    while (kp < n) kp <<= 1;
    for (int size = 2; size <= kp; size <<= 1)
        for (int stride = size >> 1; stride >= 1; stride >>= 1) {
            for (int i = threadIdx.x; i < (kp >> 1); i += blockDim.x) {
                const int lo = ((i & ~(stride - 1)) << 1) | (i & (stride - 1));
                const int hi = stride == (size >> 1) ? (lo | (size - 1)) - (lo & (size - 1)) : lo + stride;
                if (hi < n) {
                    const u64 x = buf[lo], y = buf[hi];
                    if (y > x) {
                        buf[lo] = y;
                        buf[hi] = x;
                    }
                }
            }
            if (stride > kWave || (stride == 1 ? size : stride >> 1) > kWave) {
                __syncthreads();
            } else {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
        }
    __syncthreads();
}

template <int ELT>
__global__ void __launch_bounds__(kDealT) ex_sample_kernel(DealParams p) {
    constexpr int VE = ELT == ATK_F32 ? 4 : 8, NV = kDealSample / kDealT / VE;
    __shared__ __align__(16) u64 words[kSplitSample];
    __shared__ uint32_t misc[kRowMisc];
    static_assert(sizeof(words) >= (kDealFine + 4) * 4, "the fine bins lie there, too");
    uint32_t *cur = (uint32_t *)words;
    const int tid = threadIdx.x, T = kDealT, lane = tid & (kWave - 1);
    const int64_t r = blockIdx.x;
    const uintptr_t addr = (uintptr_t)p.x + (uintptr_t)(r * p.n) * (16 / VE);
    const int rot = (int)(addr & 15) / (16 / VE);
    const int n_vec = (rot + p.n + VE - 1) / VE - 2;  // whole vectors of the row: not the first and the last
    const row_v4u *row = row_vectors(p.x, r * p.n * (16 / VE)) + 1;
    // runs of four vectors, each at a place of its own inside its piece of the row; the pieces are dealt out so that every wavefront's
    // runs, and every lane's first ones, lie all over the row (masked and rising rows)
    constexpr int runs = NV * kDealT / 4, waves = kDealT / kWave;
    const int len = n_vec / runs;  // vectors of a piece: at least 4
    RowRegs<ELT, NV> regs;
    int at[NV];  // row position of each vector's first element
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int run = (((lane >> 2) * NV + j) * waves) + (tid >> 6);
        const uint32_t hash = (((uint32_t)run * 2654435761u) ^ ((uint32_t)r * 2246822519u)) * 3266489917u;
        const int v = (int)((int64_t)run * n_vec / runs) + (int)__umulhi(hash, (uint32_t)(len - 3)) + (lane & 3);
        at[j] = (v + 1) * VE - rot;
        regs.q[j] = row[v];
    }
    regs.i0 = 0;
    for (int i = tid; i < kDealFine + 4; i += T) cur[i] = 0u;
    for (int i = tid; i < p.n_deal; i += T) p.totals[r * p.n_deal + i] = 0u;
    auto index_at = [&](int en) {
        int pos = at[en / VE];
        asm volatile("" : "+v"(pos));  // (worked out again on each pass, not kept)
        pos += en % VE;
        return p.xi ? p.xi[r * p.n + pos] : pos;
    };
    // a lower bound from a part of the sample (eight elements per lane), with a margin: counted, not trusted
    uint32_t k_min, k_max;
    regs.template bound<true>(8, p.rank, misc, k_min, k_max);
    RowBins bins;
    // (a range that starts at -inf is taken again from the lower edge of the threshold's bin: a range without what lies far below; one with
    // too few elements in it, from -inf first)
    bool raised = k_min > 0x007fffffu, measured = false, cut = false, split = false;
    uint32_t rank = (uint32_t)p.sample_rank, total, tb;
    for (int pass = 0;; ++pass) {
        bins.template set<ELT>(k_min, k_max, p.idx_bits, kDealFine);
        float v_lo = __uint_as_float(bits_of_ukey(k_min));
        regs.each([&](uint32_t bits, int, int en) {
            if (__uint_as_float(bits) >= v_lo)
                atomicAdd(&cur[bins.template bin<ELT, true>(ukey_of_bits(bits), 0x7fffffffu - (uint32_t)index_at(en))], 1u);
        });
        if (tid == 0) misc[0] = misc[5] = misc[7] = 0u;
        __syncthreads();
        row_scan(cur, misc, kDealFine, rank);
        total = misc[3];
        bool few = total < rank, decide = false;
        if (pass < 5 && (few ? raised : !raised)) {
            raised = !few;
            k_min = few ? 0x007fffffu : bins.template edge<ELT>(misc[0]);
        } else if (measured) {
            decide = true;
        } else {
            // How far the sample may be off: sixteen elements of a run are as good as one where neighbours go together, so the deviation
            // is that of the runs' counts above the threshold, not that of single elements.
            measured = true;
            v_lo = __uint_as_float(bits_of_ukey(bins.template edge<ELT>(misc[0])));
            uint32_t n_in[NV], sum = 0, squares = 0;
#pragma unroll
            for (int j = 0; j < NV; ++j) n_in[j] = 0u;
            regs.each([&](uint32_t bits, int, int en) { n_in[en / VE] += __uint_as_float(bits) >= v_lo ? 1u : 0u; });
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                uint32_t c = n_in[j];
                c += (uint32_t)__shfl_xor((int)c, 1);
                c += (uint32_t)__shfl_xor((int)c, 2);
                sum += c;
                squares += c * c;
            }
            sum = wave_incl_scan_u32((lane & 3) ? 0u : sum);
            squares = wave_incl_scan_u32((lane & 3) ? 0u : squares);
            if (lane == kWave - 1) {
                atomicAdd(&misc[5], sum);
                atomicAdd(&misc[7], squares);
            }
            __syncthreads();
            const float n_above = (float)misc[5], var = (float)misc[7] - n_above * n_above / (float)runs;
            rank = max(rank, (uint32_t)(p.expect + 6.0f * sqrtf(fmaxf(var, 0.0f)) + 6.0f));
            few = total < rank;
            decide = !few || k_min <= 0x007fffffu;
            if (!decide) {  // counted further down
                raised = false;
                k_min = 0x007fffffu;
            }
        }
        if (decide) {
            // (a sample in which too few reach the bound - NaNs - leaves fewer than k candidates, or it does not: that is counted)
            rank = min(rank, max(total, (uint32_t)p.sample_rank));
            // the threshold's bin, and whether the bins from there on are fine enough to cut the row at
            if (tid == 0) misc[40] = misc[41] = 0u;
            __syncthreads();
            const uint32_t crowd = 2u * rank / (uint32_t)p.n_deal + 16u;
            for (int f = tid; f < kDealFine; f += T) {
                const uint32_t above = cur[f], with = f > 0 ? cur[f - 1] : total;
                if (above < rank) {
                    if (with >= rank) misc[40] = (uint32_t)f;
                    if (with - above > crowd) misc[41] = 1u;
                }
            }
            __syncthreads();
            tb = misc[40];
            split = misc[41] != 0u;
            const uint32_t edge = bins.template edge<ELT>(tb);
            if (!split || cut || pass >= 5 || edge <= k_min) break;
            cut = raised = true;  // once more without what lies below the threshold (a range around zero spans every exponent)
            k_min = edge;
        }
        __syncthreads();
        for (int i = tid; i < kDealFine; i += T) cur[i] = 0u;
        __syncthreads();
    }
    uint16_t *table = p.table + r * kDealFine;
    if (!split) {
        for (int f = tid; f < kDealFine; f += T) {
            const uint32_t c = (uint32_t)((u64)cur[f] * (u64)p.n_deal / (u64)rank);  // cur: sampled elements above
            table[f] = (uint32_t)f < tb ? (uint16_t)0xffffu : (uint16_t)min(c, (uint32_t)p.n_deal - 1u);
        }
    } else {
        // Long runs of ties: a part of the sample is sorted, ties by index, and the row cut between its elements.
        __syncthreads();  // (the fine bins have been read)
        regs.each([&](uint32_t bits, int, int en) {
            // (one of every four, but for one four of the lane's eight, another one in each wavefront: no place of the row is left out)
            static_assert(kSplitLane == 7 && kDealSample == 32 * kDealT, "seven of eight fours");
            const int skip = (tid >> 6) & 7, four = en / 4;
            if (en % 4 == four % 4 && four != skip)
                words[(four - (four > skip ? 1 : 0)) * T + tid] =
                    __uint_as_float(bits) == __uint_as_float(bits) ? make_composite(bits, index_at(en)) : 0ull;
        });
        __syncthreads();
        sort_words(words, kSplitSample);
        u64 *low = (u64 *)table;
        for (int b = tid; b < p.n_deal; b += T) {
            const int last = (int)((int64_t)(b + 1) * p.split_rank / p.n_deal) - 1;
            low[b] = max(words[max(last, 0)], 1ull);  // (0: nothing)
        }
    }
    if (tid == 0) {
        DealRow d;
        d.k_min = k_min;
        d.k_max = k_max;
        d.tb = tb;
        d.cursor = 0u;
        d.split = split ? 1u : 0u;
        p.rows[r] = d;
    }
}

template <int ELT>
__global__ void __launch_bounds__(kDealT) ex_deal_kernel(DealParams p) {
    constexpr int VE = ELT == ATK_F32 ? 4 : 8, NV = kDealChunk / kDealT / VE, T = kDealT;
    constexpr int S = kDealStage / T;  // staged candidates per lane
    extern __shared__ __align__(16) unsigned char smem[];
    int2 *passed = (int2 *)smem;                       // (value bits, position), then the same bytes hold the ordered composites
    u64 *staged = (u64 *)smem;
    uint32_t *cnt = (uint32_t *)(staged + kDealStage);  // [n_deal + 1] (at most T + 4)
    uint32_t *misc = cnt + kDealBinsMax + 4;
    uint16_t *tab = (uint16_t *)(misc + kRowMisc);      // [kDealFine], or [n_deal] composites
    const int tid = threadIdx.x, lane = tid & (kWave - 1), n_waves = T >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t r = blockIdx.y;
    const int chunk = blockIdx.x;
    const int rot = (int)(((uintptr_t)p.x + (uintptr_t)(r * p.n) * (16 / VE)) & 15) / (16 / VE);
    const int n_vec = (rot + p.n + VE - 1) / VE;
    const int v0 = min(chunk * (kDealChunk / VE), n_vec - 1);
    const int v1 = chunk * (kDealChunk / VE) < n_vec ? min(v0 + kDealChunk / VE, n_vec) : v0;
    RowRegs<ELT, NV> regs;
    regs.load(p, r, v0, v1, rot);
    const DealRow info = p.rows[r];
    {
        const uint4 *src = (const uint4 *)(p.table + r * kDealFine);
        if (tid < kDealFine / 8) ((uint4 *)tab)[tid] = src[tid];
    }
    for (int i = tid; i <= p.n_deal; i += T) cnt[i] = 0u;
    if (tid == 0) misc[5] = 0u;
    RowBins bins;
    bins.template set<ELT>(info.k_min, info.k_max, p.idx_bits, kDealFine);
    regs.mask_ends(p, v0, v1, rot);
    __syncthreads();
    const u64 *low = (const u64 *)tab;  // split: the lowest composite of each bin
    const float v_lo = __uint_as_float(bits_of_ukey(info.split ? (uint32_t)(low[p.n_deal - 1] >> 32) : bins.template edge<ELT>(info.tb)));
    // ---- what reaches the threshold, side by side in LDS
    uint32_t mine = 0;
    regs.each([&](uint32_t bits, int, int) { mine += __uint_as_float(bits) >= v_lo ? 1u : 0u; });
    const uint32_t incl0 = wave_incl_scan_u32(mine);
    uint32_t at = 0;
    if (lane == kWave - 1) at = atomicAdd(&misc[5], incl0);
    at = (uint32_t)__builtin_amdgcn_readlane((int)at, kWave - 1) + incl0 - mine;
    regs.each([&](uint32_t bits, int pos, int) {
        if (__uint_as_float(bits) >= v_lo) {
            if (at < (uint32_t)kDealStage) passed[at] = make_int2((int)bits, pos);
            ++at;
        }
    });
    __syncthreads();
    const uint32_t n_passed = misc[5];
    const bool fits = n_passed <= (uint32_t)kDealStage;
    auto bin_of = [&](uint32_t bits, int idx) {
        if (info.split) {  // uniform
            const u64 c = make_composite(bits, idx);
            int first = 0, end = p.n_deal;
            while (first < end) {
                const int mid = (first + end) >> 1;
                if (c >= low[mid])
                    end = mid;
                else
                    first = mid + 1;
            }
            return first < p.n_deal ? (uint32_t)first : 0xffffu;
        }
        return (uint32_t)tab[bins.template bin<ELT, true>(ukey_of_bits(bits), 0x7fffffffu - (uint32_t)idx)];  // 0xffff: just below the threshold
    };
    auto index_of = [&](int pos) { return p.xi ? p.xi[r * p.n + pos] : pos; };
    // ---- how many in each bin
    u64 own[S];
    uint32_t own_bin[S], own_pos[S];
    if (fits) {
#pragma unroll
        for (int i = 0; i < S; ++i) {
            own_bin[i] = 0xffffu;
            if (tid + i * T < (int)n_passed) {
                const int2 w = passed[tid + i * T];
                const int idx = index_of(w.y);
                own[i] = make_composite((uint32_t)w.x, idx);
                own_bin[i] = bin_of((uint32_t)w.x, idx);
            }
        }
#pragma unroll
        for (int i = 0; i < S; ++i)
            if (own_bin[i] != 0xffffu) own_pos[i] = atomicAdd(&cnt[own_bin[i]], 1u);
    } else {
        regs.each([&](uint32_t bits, int pos, int) {
            if (__uint_as_float(bits) >= v_lo) {
                const uint32_t b = bin_of(bits, index_of(pos));
                if (b != 0xffffu) atomicAdd(&cnt[b], 1u);
            }
        });
    }
    __syncthreads();
    // ---- places: lane b has bin b
    const uint32_t c = tid < p.n_deal ? cnt[tid] : 0u;
    const uint32_t incl = wave_incl_scan_u32(c);
    if (lane == kWave - 1) misc[8 + wave] = incl;
    __syncthreads();
    const uint32_t tot = lane < n_waves ? misc[8 + lane] : 0u;
    const uint32_t tot_incl = wave_incl_scan_u32(tot);
    uint32_t off = incl - c;
    if (wave > 0) off += (uint32_t)__builtin_amdgcn_readlane((int)tot_incl, wave - 1);
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)tot_incl, n_waves - 1);
    if (tid < p.n_deal) {
        cnt[tid] = off;
        if (c) atomicAdd(&p.totals[r * p.n_deal + tid], c);
    }
    if (tid == 0) misc[6] = atomicAdd(&p.rows[r].cursor, total);
    __syncthreads();
    const int64_t base = misc[6];
    uint32_t *segs = p.segs + (r * p.chunks + chunk) * (p.n_deal + 1);
    if (tid < p.n_deal) segs[tid] = (uint32_t)base + off;
    if (tid == 0) segs[p.n_deal] = (uint32_t)base + total;
    u64 *pool = p.pool + r * p.pool_cap;
    if (fits) {
#pragma unroll
        for (int i = 0; i < S; ++i)
            if (own_bin[i] != 0xffffu) staged[cnt[own_bin[i]] + own_pos[i]] = own[i];
        __syncthreads();
        for (uint32_t i = tid; i < total; i += T)
            if (base + i < p.pool_cap) pool[base + i] = staged[i];
    } else {
        // (every bin's place counts up from here on; the bins' starts have been written)
        regs.each([&](uint32_t bits, int pos, int) {
            if (__uint_as_float(bits) >= v_lo) {
                const int idx = index_of(pos);
                const uint32_t b = bin_of(bits, idx);
                if (b != 0xffffu) {
                    const int64_t to = base + atomicAdd(&cnt[b], 1u);
                    if (to < p.pool_cap) pool[to] = make_composite(bits, idx);
                }
            }
        });
    }
}

// One bin of one row.
template <int ELT>
__global__ void __launch_bounds__(kBinT, 7) ex_bins_kernel(DealParams p) {
    constexpr int T = kBinT, S = kBinCap / T, W = T >> 6;
    __shared__ __align__(16) u64 buf[kBinCap + kBinPeers];
    __shared__ __align__(16) uint32_t cur[kBinSub + 4];
    __shared__ uint32_t misc[kRowMisc];
    __shared__ u64 ends[2 * W];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t r = blockIdx.y;
    // Workgroups go to the eight XCDs in turn; each XCD takes an eighth of the bins side by side (their number is a multiple of
    // eight): the ends of the pieces and the table of their places share lines with the neighbouring bins'.
    const int bin = (int)(blockIdx.x & 7u) * (p.n_deal >> 3) + (int)(blockIdx.x >> 3);
    // (everything that the first steps want is asked for together)
    const uint32_t cursor = p.rows[r].cursor;
    const uint32_t *totals = p.totals + r * p.n_deal;
    const uint32_t count = totals[bin];
    uint32_t before = 0;  // candidates in the bins before this one: where its outputs start
    for (int i = tid; i < bin; i += T) before += totals[i];
    for (int i = tid; i < kBinSub; i += T) cur[i] = 0u;
    if (cursor < (uint32_t)p.k || (int64_t)cursor > p.pool_cap || count == 0u) return;  // (uniform) no bin, or the row is left to the last launch
    before = wave_incl_scan_u32(before);
    if (lane == kWave - 1) misc[4 + wave] = before;
    // f(candidate) for every candidate of the bin, and its place among them: the pieces of 64 chunks at a time (lane i of every
    // wavefront looks up chunk i's), 16 lanes side by side on each, four pieces with two loads each in flight (a piece holds 16
    // candidates on average where a quarter of the row is kept)
    const u64 *pool = p.pool + r * p.pool_cap;
    const uint32_t *segs = p.segs + r * p.chunks * (p.n_deal + 1) + bin;
    auto gather = [&](auto f) {
        constexpr int G = 16;
        const int sl = lane & (G - 1);
        uint32_t carry = 0;
        for (int c0 = 0; c0 < p.chunks; c0 += kWave) {
            uint32_t s0 = 0, len = 0;
            if (c0 + lane < p.chunks) {
                const uint32_t *sg = segs + (int64_t)(c0 + lane) * (p.n_deal + 1);
                s0 = sg[0];
                len = sg[1] - s0;
            }
            const uint32_t incl = wave_incl_scan_u32(len);
            const uint32_t to = carry + incl - len;
            carry += (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
            uint32_t ps[4], pl[4], pt[4];
            u64 v[4][2];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int src = u * (T / G) + wave * (kWave / G) + (lane / G);
                ps[u] = (uint32_t)__shfl((int)s0, src);
                pl[u] = (uint32_t)__shfl((int)len, src);
                pt[u] = (uint32_t)__shfl((int)to, src);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int h = 0; h < 2; ++h) v[u][h] = pool[ps[u] + ((uint32_t)(sl + h * G) < pl[u] ? sl + h * G : 0)];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    if ((uint32_t)(sl + h * G) < pl[u]) f(v[u][h], pt[u] + sl + h * G);
                // the rest of long pieces (rows in order, runs of ties), one after the other by the whole wavefront
                for (u64 more = __ballot(sl == 0 && pl[u] > 2u * G); more; more &= more - 1ull) {
                    const int src = __builtin_ctzll(more);
                    const uint32_t from = (uint32_t)__builtin_amdgcn_readlane((int)ps[u], src), n = (uint32_t)__builtin_amdgcn_readlane((int)pl[u], src);
                    const uint32_t place = (uint32_t)__builtin_amdgcn_readlane((int)pt[u], src);
                    for (uint32_t i = 2u * G + lane; i - lane < n; i += 2 * kWave) {
                        u64 w[2];
#pragma unroll
                        for (int h = 0; h < 2; ++h) w[h] = pool[from + min(i + h * kWave, n - 1u)];
#pragma unroll
                        for (int h = 0; h < 2; ++h)
                            if (i + h * kWave < n) f(w[h], place + i + h * kWave);
                    }
                }
            }
        }
    };
    static_assert(4 * (T / 16) == kWave, "64 chunks at a time");
    const bool fits = count <= (uint32_t)kBinCap;  // uniform
    uint32_t k_min = 0xffffffffu, k_max = 0u;
    gather([&](u64 c, uint32_t place) {
        const uint32_t key = (uint32_t)(c >> 32);
        k_min = min(k_min, key);
        k_max = max(k_max, key);
        if (fits) buf[place] = c;
    });
    k_min = wave_min_u32(k_min);
    k_max = wave_max_u32(k_max);
    if (lane == 0) {
        misc[8 + wave] = k_min;
        misc[24 + wave] = k_max;
    }
    __syncthreads();
    uint32_t start = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        start += misc[4 + w];
        k_min = min(k_min, misc[8 + w]);
        k_max = max(k_max, misc[24 + w]);
    }
    // (the same in every lane: scalars from here on, and what the bins are made of with them)
    k_min = (uint32_t)__builtin_amdgcn_readfirstlane((int)k_min);
    k_max = (uint32_t)__builtin_amdgcn_readfirstlane((int)k_max);
    start = (uint32_t)__builtin_amdgcn_readfirstlane((int)start);
    if (start >= (uint32_t)p.k) return;  // uniform
    const int64_t out = r * p.k + start;
    const uint32_t room = (uint32_t)p.k - start;  // outputs left from here on
    int lg = 8;  // about a bin per candidate
    while ((1 << lg) < kBinSub && (1 << lg) < (int)count) ++lg;
    const int n_sub = 1 << lg;
    RowBins bins;
    bins.template set<ELT>(k_min, k_max, p.idx_bits, n_sub);
    // Sub-bins are linear between the bin's lowest and highest key (ties: in the index, from 0 to the row's length); where that puts
    // dozens into one (one value's ties on a short stretch of the row), between its smallest and its largest composite.
    const RowSqueeze<ELT> sq{p.idx_bits + 1};
    u64 q_min = 0ull;
    int q_shift = -1;
    const int s_idx = __builtin_amdgcn_readfirstlane(bins.s_idx), r_idx = __builtin_amdgcn_readfirstlane(bins.r_idx);
    const uint32_t scale = (uint32_t)__builtin_amdgcn_readfirstlane((int)bins.scale);
    auto sub_of = [&](u64 c) {
        if (q_shift >= 0) return (uint32_t)((sq(c) - q_min) >> q_shift);
        // (RowBins::bin(); an index has 31 bits at most, so s_idx is no more)
        const uint32_t d = ((((uint32_t)(c >> 32) - k_min) >> (ELT == ATK_BF16 ? 16 : 0)) << s_idx) | __builtin_amdgcn_ubfe((uint32_t)c, 1 + r_idx, s_idx);
        return (uint32_t)min(__umulhi(d, scale), (uint32_t)n_sub - 1u);
    };
    // mn, mx: this lane's.  Called by the whole workgroup; ends in a barrier, with the sub-bins cleared.
    auto narrow = [&](u64 mn, u64 mx) {
        wave_min_max_u64(mn, mx);
        if (lane == 0) {
            ends[wave] = mn;
            ends[W + wave] = mx;
        }
        for (int i = tid; i < kBinSub; i += T) cur[i] = 0u;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < W; ++w) {
            mn = ends[w] < mn ? ends[w] : mn;
            mx = ends[W + w] > mx ? ends[W + w] : mx;
        }
        q_min = mn;
        for (q_shift = 0; ((mx - mn) >> q_shift) >= (u64)n_sub;) ++q_shift;
        q_shift = __builtin_amdgcn_readfirstlane(q_shift);
    };
    // Ranks of the ordered-by-sub-bin candidates buf[0 .. n), which are places [first, first + n) of the bin; kBinPeers zeros behind them.  (What lies behind a
    // sub-bin's candidates is smaller than they are, so the first few places from its start on are looked at whosever they are: 128 x 2^20 f32, k = 2^18: 364 us
    // with a choice of each address, 358 without; ranks kept in registers and brought into order in LDS, for wider stores: 380 and 390.)
    auto rank_write = [&](uint32_t n, uint32_t first, auto start_of, auto end_of) {
        for (uint32_t i = tid; i < n; i += T) {
            const u64 c = buf[i];
            const uint32_t b = sub_of(c);
            const uint32_t s = start_of(b) - first, e = end_of(b) - first;
            u64 peer[kBinPeers];
#pragma unroll
            for (int u = 0; u < kBinPeers; ++u) peer[u] = buf[s + u];
            uint32_t rank = first + s;
#pragma unroll
            for (int u = 0; u < kBinPeers; ++u) rank += peer[u] > c ? 1u : 0u;
            for (uint32_t j = s + kBinPeers; j < e; ++j) rank += buf[j] > c ? 1u : 0u;
            if (rank < room) write_composite<ELT>(c, p.out_vals, p.out_idx, out + rank);
        }
    };
    if (!fits) {
        // Stretch by stretch from the top, each cut by a histogram of what is left between its smallest and its largest element.  Where the
        // highest of the 1024 bins alone is more than the LDS holds, the same inside that bin: composites are distinct, so that ends.
        auto stretches = [&]() {
            u64 top = ~0ull, bottom = 0ull;  // (squeezed) what is left lies below top; the stretch is looked for from bottom on
            for (uint32_t first = 0; first < count && first < room;) {
                __syncthreads();  // (buf and misc have been read)
                for (int i = tid; i < kBinSub; i += T) cur[i] = 0u;
                if (tid == 0) misc[5] = 0u;
                u64 mn = ~0ull, mx = 0ull;
                gather([&](u64 c, uint32_t) {
                    const u64 q = sq(c);
                    if (q >= bottom && q < top) {
                        mn = q < mn ? q : mn;
                        mx = q > mx ? q : mx;
                    }
                });
                wave_min_max_u64(mn, mx);
                if (lane == 0) {
                    buf[wave] = mn;
                    buf[W + wave] = mx;
                }
                __syncthreads();
    #pragma unroll
                for (int w = 0; w < W; ++w) {
                    mn = buf[w] < mn ? buf[w] : mn;
                    mx = buf[W + w] > mx ? buf[W + w] : mx;
                }
                int shift = 0;
                while (((mx - mn) >> shift) >= (u64)kBinSub) ++shift;
                auto bin_at = [&](u64 q) { return (uint32_t)((q - mn) >> shift); };
                gather([&](u64 c, uint32_t) {
                    const u64 q = sq(c);
                    if (q >= mn && q <= mx) atomicAdd(&cur[bin_at(q)], 1u);
                });
                __syncthreads();
                row_scan(cur, misc, kBinSub, count);
                // the lowest bin down to which LDS holds them all
                const uint32_t all = misc[3];
                uint32_t low = (uint32_t)kBinSub;
                for (int b = tid; b < kBinSub; b += T)
                    if ((b > 0 ? cur[b - 1] : all) <= (uint32_t)kBinCap) low = min(low, (uint32_t)b);
                low = wave_min_u32(low);
                if (lane == 0) misc[8 + wave] = low;
                __syncthreads();
    #pragma unroll
                for (int w = 0; w < W; ++w) low = min(low, misc[8 + w]);
                const uint32_t n = low < (uint32_t)kBinSub ? (low > 0u ? cur[low - 1u] : all) : 0u;
                if (n == 0u) {  // (uniform)
                    bottom = mn + ((u64)bin_at(mx) << shift);
                    continue;
                }
                const u64 from = mn + ((u64)low << shift);
                gather([&](u64 c, uint32_t) {
                    const u64 q = sq(c);
                    if (q >= from && q <= mx) buf[atomicAdd(&misc[5], 1u)] = c;
                });
                __syncthreads();
                sort_words(buf, (int)n);
                for (uint32_t i = tid; i < n && first + i < room; i += T) write_composite<ELT>(buf[i], p.out_vals, p.out_idx, out + first + i);
                first += n;
                top = from;
                bottom = 0ull;
            }
        };
        // More than the LDS holds (a place of the row that the sample saw too little of): the pieces are read once to count and
        // then once for every stretch of sub-bins that fits.
        __syncthreads();  // (misc has been read)
        gather([&](u64 c, uint32_t) { atomicAdd(&cur[sub_of(c)], 1u); });
        __syncthreads();
        row_scan(cur, misc, n_sub, count);
        if (misc[4] != 0u) {
            u64 mn = ~0ull, mx = 0ull;
            gather([&](u64 c, uint32_t) {
                mn = sq(c) < mn ? sq(c) : mn;
                mx = sq(c) > mx ? sq(c) : mx;
            });
            narrow(mn, mx);
            gather([&](u64 c, uint32_t) { atomicAdd(&cur[sub_of(c)], 1u); });
            __syncthreads();
            row_scan(cur, misc, n_sub, count);
        }
        if (misc[4] != 0u) {  // ties by the dozen
            stretches();
            return;
        }
        // (a sub-bin holds kRowBinMax at most, so those that start inside a window of kBinCap - kRowBinMax places fit)
        constexpr uint32_t window = kBinCap - kRowBinMax;
        uint32_t first = 0;  // the window's first place, and its highest sub-bin
        for (int top = n_sub - 1; top >= 0 && first < room && first < count;) {
            uint32_t low = (uint32_t)top;  // its lowest sub-bin
            for (int b = tid; b <= top; b += T)
                if (cur[b] < first + window) low = min(low, (uint32_t)b);
            low = wave_min_u32(low);
            if (lane == 0) misc[8 + wave] = low;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < W; ++w) low = min(low, misc[8 + w]);
            const uint32_t end = low > 0u ? cur[low - 1u] : count;
            // cur[b] moves from the place where sub-bin b starts to its end, which is where b - 1 starts
            gather([&](u64 c, uint32_t) {
                const uint32_t b = sub_of(c);
                if (b >= low && b <= (uint32_t)top) buf[atomicAdd(&cur[b], 1u) - first] = c;
            });
            if (tid < kBinPeers) buf[end - first + tid] = 0ull;
            __syncthreads();
            rank_write(end - first, first, [&](uint32_t b) { return b == (uint32_t)top ? first : cur[b + 1u]; }, [&](uint32_t b) { return cur[b]; });
            __syncthreads();
            first = end;
            top = (int)low - 1;
        }
        return;
    }
    // ---- into registers and counted
    u64 own[S];
    uint32_t at[S];  // sub-bin, and place among its arrivals in the upper half
#pragma unroll
    for (int i = 0; i < S; ++i) {
        own[i] = 0ull;
        if (i * T < (int)count && tid + i * T < (int)count) own[i] = buf[tid + i * T];
    }
    auto to_sub_bins = [&]() {
#pragma unroll
        for (int i = 0; i < S; ++i)
            if (i * T < (int)count && own[i]) {
                const uint32_t b = sub_of(own[i]);
                at[i] = b | (atomicAdd(&cur[b], 1u) << 16);
            }
        __syncthreads();
        row_scan(cur, misc, n_sub, count);
        return misc[4] != 0u;
    };
    bool crowded = to_sub_bins();
    if (crowded) {
        u64 mn = ~0ull, mx = 0ull;
#pragma unroll
        for (int i = 0; i < S; ++i)
            if (own[i]) {
                mn = sq(own[i]) < mn ? sq(own[i]) : mn;
                mx = sq(own[i]) > mx ? sq(own[i]) : mx;
            }
        narrow(mn, mx);
        crowded = to_sub_bins();
    }
    if (crowded) {
        // many candidates in one place of the bin's range (ties)
        sort_words(buf, (int)count);
        for (uint32_t i = tid; i < count && i < room; i += T) write_composite<ELT>(buf[i], p.out_vals, p.out_idx, out + i);
        return;
    }
#pragma unroll
    for (int i = 0; i < S; ++i)
        if (i * T < (int)count && own[i]) buf[cur[at[i] & 0xffffu] + (at[i] >> 16)] = own[i];
    if (tid < kBinPeers) buf[count + tid] = 0ull;
    __syncthreads();
    rank_write(count, 0u, [&](uint32_t b) { return cur[b]; }, [&](uint32_t b) { return b > 0u ? cur[b - 1u] : count; });
}

// ------------------------------------------------------------------------------------ host
static int64_t align256(int64_t v) { return (v + 255) / 256 * 256; }

// Rows of more than 2 * 32768 elements (shorter ones would be sampled nearly whole) with at most 512 chunks, and k for which
// the sample says something: 64 of its elements or more among the k largest.
bool plan_exact_deal(int64_t m, int64_t n, int64_t k, int dtype, bool ptr16, DealPlan *out) {
    DealPlan p;
    memset(&p, 0, sizeof p);
    const int ve = dtype == ATK_F32 ? 4 : 8;
    if (n < 2 * kDealSample || m > 65535) return false;
    const double q = (double)k / (double)n, expect = q * kDealSample;
    if (expect < 64.0 || q > 0.6) return false;
    // (rows off the 16-byte boundaries: up to ve - 1 more elements)
    p.chunks = (int)((n + (ptr16 && n % ve == 0 ? 0 : ve - 1) + kDealChunk - 1) / kDealChunk);
    if (p.chunks > kDealChunksMax) return false;
    int64_t bins = (k + kDealBinMean - 1) / kDealBinMean;
    bins = (bins + 7) / 8 * 8;
    if (bins > kDealBinsMax) return false;
    p.bins = (int)bins;
    // six standard deviations of the sample's count above what k of n elements make of it; up to four times that where neighbours go
    // together (sixteen to a run: ex_sample_kernel); the pool takes as many again
    const double sd = std::sqrt(expect * (1.0 - q));
    p.expect = (float)expect;
    p.sample_rank = (int)std::ceil(expect + 6.0 * sd + 6.0);
    const double most = (expect + 48.0 * sd + 64.0) / kDealSample;
    // the same for the sample that is sorted, four elements to a run
    const double share = q * kSplitSample, split_sd = 2.0 * std::sqrt(share * (1.0 - q));
    p.split_rank = std::min((int)std::ceil(share + 6.0 * split_sd + 6.0), kSplitSample);
    const double split_most = (share + 12.0 * split_sd + 24.0) / kSplitSample;
    p.pool_cap = std::max<int64_t>(k, std::min<int64_t>(n, (int64_t)(std::max(most, split_most) * (double)n)));
    // the sample's lower bound: 8192 of its 32768 elements, 512 in each wavefront, five deviations below the threshold
    const double part = (double)p.sample_rank / 4.0 / (kDealT / kWave);
    p.rank = std::min(512, (int)std::ceil(part + 5.0 * std::sqrt(part) + 2.0));
    int64_t off = 0;
    auto take = [&](int64_t bytes) {
        const int64_t at = off;
        off += align256(bytes);
        return at;
    };
    p.rows_off = take(m * (int64_t)sizeof(DealRow));
    p.table_off = take(m * kDealFine * 2);
    p.totals_off = take(m * bins * 4);
    p.segs_off = take(m * p.chunks * (bins + 1) * 4);
    p.pool_off = take(m * p.pool_cap * 8);
    p.rest_off = take(m * k * 8);  // for the rows that go digit by digit: one buffer of k, the other is the pool, done with by then
    p.bytes = off;
    *out = p;
    return true;
}

template <int ELT>
static hipError_t launch_deal_t(const DealPlan &pl, const DealParams &prm, int64_t m, hipStream_t stream) {
    const size_t lds = (size_t)kDealStage * 8 + (kDealBinsMax + 4 + kRowMisc) * 4 + kDealFine * 2;
    static_assert(kDealStage * 8 + (kDealBinsMax + 4 + kRowMisc) * 4 + kDealFine * 2 <= 64 * 1024, "dynamic LDS without asking");
    hipLaunchKernelGGL(ex_sample_kernel<ELT>, dim3((unsigned)m), dim3(kDealT), 0, stream, prm);
    hipLaunchKernelGGL(ex_deal_kernel<ELT>, dim3((unsigned)pl.chunks, (unsigned)m), dim3(kDealT), lds, stream, prm);
    hipLaunchKernelGGL(ex_bins_kernel<ELT>, dim3((unsigned)pl.bins, (unsigned)m), dim3(kBinT), 0, stream, prm);
    return hipGetLastError();
}

hipError_t launch_exact_deal(const DealPlan &pl, int64_t m, int64_t n, int64_t k, int64_t idx_n, int dtype, const void *x,
                             const int32_t *xi, void *out_vals, int32_t *out_idx, void *data, hipStream_t stream) {
    DealParams prm;
    memset(&prm, 0, sizeof prm);
    unsigned char *base = (unsigned char *)data;
    prm.x = x;
    prm.xi = xi;
    prm.out_vals = out_vals;
    prm.out_idx = out_idx;
    prm.n = (int)n;
    prm.k = (int)k;
    prm.idx_bits = 1;
    while (((int64_t)1 << prm.idx_bits) < idx_n) ++prm.idx_bits;
    prm.rank = pl.rank;
    prm.rows = (DealRow *)(base + pl.rows_off);
    prm.table = (uint16_t *)(base + pl.table_off);
    prm.totals = (uint32_t *)(base + pl.totals_off);
    prm.segs = (uint32_t *)(base + pl.segs_off);
    prm.pool = (u64 *)(base + pl.pool_off);
    prm.pool_cap = pl.pool_cap;
    prm.n_deal = pl.bins;
    prm.chunks = pl.chunks;
    prm.sample_rank = pl.sample_rank;
    prm.split_rank = pl.split_rank;
    prm.expect = pl.expect;
    const hipError_t e = dtype == ATK_F32 ? launch_deal_t<ATK_F32>(pl, prm, m, stream) : launch_deal_t<ATK_BF16>(pl, prm, m, stream);
    if (e != hipSuccess) return e;
    return launch_exact_rest_rows(m, n, k, prm.idx_bits, dtype, x, xi, prm.rows, pl.pool_cap, (u64 *)(base + pl.rest_off), prm.pool, out_vals,
                                  out_idx, stream);
}

}  // namespace atk
