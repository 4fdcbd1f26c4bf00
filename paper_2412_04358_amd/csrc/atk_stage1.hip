// Fused kernel of approx_topk: Stage 1 (per-bucket top-k_b), the merges needed when one
// bucket is spread over several lanes / workgroups, and Stage 2 (exact top-k of the
// b*k_b candidates) when b*k_b > k.   Section 2 and Appendix A of arxiv 2412.04358.
//
// Mapping.  Bucket j of a row holds the elements i = j (mod b) (Appendix A.1), so the row
// is an L x b row-major matrix whose column j is bucket j.  A lane owns V adjacent columns
// (one 16-byte load per matrix row) and keeps, per column, the k_b largest elements seen
// so far in registers ("a max priority queue of size k_b ... in per-thread registers",
// Appendix A).  Lanes side by side read consecutive addresses, so the interleaved layout
// costs nothing.  When b is small, several lanes (row phases) share a column group, and
// when m*b is too small to fill the chip, several workgroups (row splits) do; their sorted
// lists are merged once at the end (Appendix A, mode (2): "merge the per-thread queues
// once"), first in LDS, then - across workgroups - by whichever workgroup of the row
// finishes last (a ticket counter), which also runs Stage 2.
#include <algorithm>
#include <cstdlib>
#include <cstring>

#include <type_traits>

#include "atk_common.h"
#include "atk_packed.h"
#include "atk_select.h"
#include "atk_sort_select.h"
#include "atk_stream.h"

namespace atk {

struct S1Params {
    const void *x;
    void *out_vals;
    int32_t *out_idx;
    u64 *lists;          // scratch: [row][split][column][k_b] composites
    uint32_t *tickets;   // scratch: one counter per row (kTicketStride words apart), zero between calls
    int64_t n;
    int b, L, G, Gw, P, colblocks, S, rows_per_split;
    int rem, extra_ph;   // n mod b, and the row phase that takes the ragged last matrix row
    int idx_bits;        // column indices are below 2^idx_bits
    int k, k_b;
    int stage2, direct, use_scratch, vec_store;
    int staged;          // direct: a wavefront's outputs go through LDS, to be stored side by side
    int wave_merge;      // Gw < 64 and a power of two: lanes of one wavefront share columns
    int nparts;          // partial lists per column left after the wavefront merge
    int lds_xch_off, lds_cand_off;  // byte offsets of the exchange and candidate areas in LDS
    int cb_shift, s_shift, gw_shift;  // log2 of colblocks, S, Gw when those are powers of two, else -1
    int tail_tpc_shift;  // log2 of the lanes that share a column in the last workgroup's merge
    int wgs_per_ticket;  // workgroups that share a ticket: a row's (Stage 2), else a column block's row splits
    // contiguous assignment only
    int Gs, gs_shift;    // lanes per bucket (a power of two) and its log2
    int bblocks;         // workgroups side by side across the b buckets
    int chunks_per_split;
    int NB;              // short buckets: buckets a lane group takes in turn (0: one bucket per group)
    int lds_max;         // k_b = 1, no scratch: the lanes' running maxima meet in LDS by atomic maximum (see the kernel)
    int bound_ok;        // ... and the lower bound on the smallest candidate that comes with that merge is tight enough for select_binned()
    int refresh;         // eight unpacked slots: the lanes of a column pool their queues' floors after four times this many matrix rows each, then four times as many, ... (0: never)
    u64 *trace;          // measurement build only: phase timestamps, [workgroup][wavefront][phase]
};

// The scans count ahead of their last matrix row (contiguous buckets: load) in 32 bits, by up to three batches of sixteen for each
// of 1024 lanes.  Only rows of one bucket are long enough for that to pass 2^31; what they have beyond this row is taken one by one.  (The host
// sees to it that no split starts near it.)
constexpr int kRowsAhead = 0x7fffffff - (1 << 16);

// Insert (v, t) into the descending list (val, tt); later elements never displace equal
// earlier ones ("!(v <= slot)" is "v > slot" for numbers and true for the NaN that marks
// an empty slot).
template <int KB>
__device__ __forceinline__ void insert(float (&val)[KB], int (&tt)[KB], float v, int t) {
    bool c[KB];
#pragma unroll
    for (int j = 0; j < KB; ++j) c[j] = !(v <= val[j]);
#pragma unroll
    for (int j = KB - 1; j >= 1; --j) {
        val[j] = c[j - 1] ? val[j - 1] : (c[j] ? v : val[j]);
        tt[j] = c[j - 1] ? tt[j - 1] : (c[j] ? t : tt[j]);
    }
    val[0] = c[0] ? v : val[0];
    tt[0] = c[0] ? t : tt[0];
}

// ---- batch scan for long queues (k_b > 4) -------------------------------------------------------------------------
// Inserting element by element costs about five lane operations per slot and element.  Where most elements enter
// the queue (short buckets: the top quarter of every bucket is kept when b*k_b = k = n/4) it is cheaper to take
// k_b matrix rows at a time, sort them with a network, and fold the sorted batch into the queue with the
// bitonic merge that also joins the lanes' queues.  A network has no notion of "earlier element wins ties", so the queues
// hold words that are distinct: [63:32] the float's own bits (-0 as +0), [31:0] 0x7fffffff - the element's number among the lane's
// rows, inverted where the float is negative.  The order of the words is their order as doubles: sign and magnitude order a
// double's high word as they order a float, and among equal floats the earlier element has the larger magnitude where that is the
// larger double, the smaller one where it is not.  The exponent field of +-inf comes out as 0x7f8 (and that of a small float as zero:
// denormals are kept), so every number makes a finite double, and a compare-exchange is v_max_f64 and v_min_f64, two
// instructions at full rate, instead of a 64-bit compare and four selects (128 x 65536 f32, k = 16384: k_b = 16:
// 27.5 -> 20.2 us; k_b = 8, element by element before: 19.1 -> 17.4; one row of 2^20, b = 1024, k_b = 8: 132 -> 30; 64 x 2^20,
// k = 1024, b = 1024, k_b = 8: 140 -> 88).  A word is three instructions to make; with the value's order
// key and "was -0" in it, it took twelve, which with a select for every element of every batch came to half of the scan: 128 x 65536, k = 16384,
// b = 2048, k_b = 8: 16.9 -> 15.6 us.  Which zeros were -0 is looked up in the row at the end.
__device__ __forceinline__ double word_max(double a, double b) {
    double d;
    asm("v_max_f64 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));  // (fmax() would quiet its operands first)
    return d;
}
__device__ __forceinline__ double word_min(double a, double b) {
    double d;
    asm("v_min_f64 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
    return d;
}
__device__ __forceinline__ double row_word(uint32_t bits, uint32_t s) {
    const int hi = __float_as_int(__uint_as_float(bits) + 0.0f);
    return __hiloint2double(hi, (int)(0x7fffffffu - s) ^ (hi >> 31));
}
// What marks an empty slot lies below -inf and is a NaN as a float: for bf16 its high half alone.
constexpr uint32_t kNoWordBits = 0xffef0000u;
__device__ __forceinline__ double no_word() { return __hiloint2double((int)kNoWordBits, -1); }
__device__ __forceinline__ uint32_t word_bits(double w) { return (uint32_t)__double2hiint(w); }
__device__ __forceinline__ bool is_word(double w) { return word_bits(w) <= 0xff800000u; }
__device__ __forceinline__ uint32_t word_number(double w) {
    return 0x7fffffffu - (uint32_t)(__double2loint(w) ^ (__double2hiint(w) >> 31));
}
__device__ __forceinline__ uint32_t word_key(double w) { return is_word(w) ? ukey_of_bits(word_bits(w)) : 0u; }
// Batcher's odd-even merge sort of N words, largest first (N a power of two; 19 compare-exchanges for 8, 63 for 16).
template <int N>
__device__ __forceinline__ void sort_desc(double (&a)[N]) {
#pragma unroll
    for (int p = 1; p < N; p *= 2)
#pragma unroll
        for (int k = p; k >= 1; k /= 2)
#pragma unroll
            for (int j = k % p; j + k < N; j += 2 * k)
#pragma unroll
                for (int i = 0; i < k; ++i)
                    if (i + j + k < N && (i + j) / (2 * p) == (i + j + k) / (2 * p)) {
                        const double x = a[i + j], y = a[i + j + k];
                        a[i + j] = word_max(x, y);
                        a[i + j + k] = word_min(x, y);
                    }
}
// mine <- the N largest of (mine U theirs); both sorted descending, result sorted descending.
template <int N>
__device__ __forceinline__ void merge_words(double (&mine)[N], const double (&theirs)[N]) {
#pragma unroll
    for (int j = 0; j < N; ++j) mine[j] = word_max(mine[j], theirs[N - 1 - j]);
#pragma unroll
    for (int stride = N / 2; stride >= 1; stride >>= 1)
#pragma unroll
        for (int i = 0; i < N; ++i)
            if ((i & stride) == 0) {
                const double x = mine[i], y = mine[i + stride];
                mine[i] = word_max(x, y);
                mine[i + stride] = word_min(x, y);
            }
}
// one word into a queue sorted largest first
template <int N>
__device__ __forceinline__ void insert_word(double (&q)[N], double c) {
#pragma unroll
    for (int j = N - 1; j >= 1; --j) q[j] = word_max(q[j], word_min(q[j - 1], c));  // (q[j-1] >= q[j]: c clamped between them)
    q[0] = word_max(q[0], c);
}

// ---- queues that elements enter rarely (pooled floors) ----------------------------------------------------------------
// A queue of words (as above, numbered by the lane's matrix rows) and one element that waits for it: an element that beats `last` - a
// comparison, and two selects where any lane of the wavefront has one - is put by, and only where a lane has one already do all lanes work
// theirs into the queues, some thirty instructions; with 64 lanes that is about one time in ten.  Where a queue of values and rows took its
// elements one by one, the 40 instructions that some lane needed two times in three bounded these rows (82 % of the SIMDs' cycles).  `last` may
// lag behind the queue (what waits has not raised it yet), which lets an element too many through and never one too few; the words put them
// in order.  While elements enter often - rows that rise along their length, every row at its start - a batch of matrix rows is sorted and
// merged in instead, 15 instructions an element where working them in one by one takes 40: rising rows of 2048 x 65536, b = 16 take 137 us so,
// 240 one by one and 129 without floors; 128 x 2^20, b = 128: 128, 222, 125; without order 95, 113 and 129; 108, 116 and 129.
template <int KB>
struct LazyQueue {
    double q[KB];
    float last;     // an element has to beat it: the value in the last slot, or a floor above that (NaN: anything enters)
    uint32_t wait;  // the waiting element,
    int wait_t;     // and its number (kEmptyT: none)
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int j = 0; j < KB; ++j) q[j] = no_word();
        last = __uint_as_float(0x7fc00000u);
        wait = 0u;
        wait_t = kEmptyT;
    }
    __device__ __forceinline__ void raise() {
        last = fmaxf(last, __uint_as_float(word_bits(q[KB - 1])));  // (empty: a NaN, and `last` stays)
    }
    __device__ __forceinline__ void flush() {
        const double c = row_word(wait, (uint32_t)wait_t);
        insert_word<KB>(q, wait_t != kEmptyT ? c : no_word());
        wait_t = kEmptyT;
        raise();
    }
    __device__ __forceinline__ void feed(uint32_t bits, int t, int &flushed) {
        const bool in = !(__uint_as_float(bits) <= last);
        if (__ballot(in) == 0ull) return;
        if (__ballot(in && wait_t != kEmptyT) != 0ull) {
            flush();
            ++flushed;
        }
        wait = in ? bits : wait;
        wait_t = in ? t : wait_t;
    }
    // KB matrix rows numbered t, t + 1, ... at once: sorted, and merged into the queue.  Whether some lane had half of them to put in: elements
    // still enter often (three and more to six and more measure the same).
    __device__ __forceinline__ bool feed_sorted(const uint32_t (&bits)[KB], int t) {
        int n = 0;
#pragma unroll
        for (int u = 0; u < KB; ++u) n += __uint_as_float(bits[u]) <= last ? 0 : 1;
        if (__ballot(n != 0) == 0ull) return false;
        if (__ballot(wait_t != kEmptyT) != 0ull) flush();
        double c[KB];
#pragma unroll
        for (int u = 0; u < KB; ++u) c[u] = row_word(bits[u], (uint32_t)(t + u));
        sort_desc<KB>(c);
        merge_words<KB>(q, c);
        raise();
        return __ballot(n >= KB / 2) != 0ull;
    }
};

// mine <- the N largest of (mine U theirs), as multisets; both sorted descending, result sorted descending.
template <int N>
__device__ __forceinline__ void merge_keys(uint32_t (&mine)[N], const uint32_t (&theirs)[N]) {
#pragma unroll
    for (int j = 0; j < N; ++j) mine[j] = max(mine[j], theirs[N - 1 - j]);
#pragma unroll
    for (int stride = N / 2; stride >= 1; stride >>= 1)
#pragma unroll
        for (int i = 0; i < N; ++i)
            if ((i & stride) == 0) {
                const uint32_t a = mine[i], c = mine[i + stride];
                mine[i] = max(a, c);
                mine[i + stride] = min(a, c);
            }
}

// Feed the V elements of one load into the lane's V queues.  With k_b > 1 the insertion costs
// about 5*k_b lane operations per element, so it is skipped whenever no lane of the wavefront
// holds an element that beats the last slot of its queue (one compare per element and a
// wavefront-uniform branch): on long buckets almost every load is rejected that way.
template <int ELT, int V, int KB>
__device__ __forceinline__ void scan_vec(float (&val)[V][KB], int (&tt)[V][KB], const RowVec<ELT, V> &v, int t) {
    float x[V];
#pragma unroll
    for (int e = 0; e < V; ++e) x[e] = __uint_as_float(elem_bits<ELT, V>(v, e));
    if (KB > 1) {
        bool any = false;
#pragma unroll
        for (int e = 0; e < V; ++e) any = any || !(x[e] <= val[e][KB - 1]);
        if (__ballot(any) == 0ull) return;
    }
#pragma unroll
    for (int e = 0; e < V; ++e) insert<KB>(val[e], tt[e], x[e], t);
}

// Stage-1 result of bucket `col`, as seen by row split `sp` of row r: to the scratch lists (when
// several workgroups share the row), to the candidate area in LDS (Stage 2 inside this
// workgroup), or straight to the output.
template <int ELT, int KB>
__device__ __forceinline__ void emit_list(const S1Params &p, int r, int sp, int col, const u64 (&list)[KB], u64 *cand) {
    if (p.use_scratch) {
        // agent-scope atomic stores: written through to memory, not left in this XCD's L2
        u64 *dst = p.lists + (((int64_t)r * p.S + sp) * p.b + col) * p.k_b;
#pragma unroll
        for (int j = 0; j < KB; ++j)
            if (j < p.k_b) __hip_atomic_store(&dst[j], list[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else if (p.stage2) {
#pragma unroll
        for (int j = 0; j < KB; ++j)
            if (j < p.k_b) cand[col * p.k_b + j] = list[j];
    } else {
        const int64_t o = (int64_t)r * p.k + (int64_t)col * p.k_b;
#pragma unroll
        for (int j = 0; j < KB; ++j)
            if (j < p.k_b) write_composite<ELT>(list[j], p.out_vals, p.out_idx, o + j);
    }
}

// What follows the last emit_list() of a workgroup: the hand-over between the workgroups that
// share a ticket, and Stage 2.  Every thread calls it.
// With Stage 2 the whole row shares one ticket (one workgroup must see all b*k_b candidates);
// without it every block of columns [c_lo, c_hi) has its own (ticket number `tk`), and whoever
// draws the last one merges the row splits of just those columns.  Column c of the block is
// bucket c - rot (mod b).
template <int ELT, int KB, bool TR = false>
__device__ __forceinline__ void row_tail(const S1Params &p, int r, int64_t tk, int c_lo, int c_hi, int rot,
                                         unsigned char *smem) {
    const int tid = threadIdx.x, T = blockDim.x;
    u64 *cand = (u64 *)(smem + p.lds_cand_off);
    if (!p.use_scratch) {
        if (!p.stage2) return;
        __syncthreads();
    } else {
        // ------------------------------------------------------------ ticket
        // Cross-workgroup hand-over without cache-wide fences: the lists were written, and are
        // read below, with agent-scope atomic accesses (they go through to memory instead of
        // staying in one XCD's L2, so there is nothing for a cache write-back or invalidate to do);
        // every lane waits until its own stores have been acknowledged (a barrier alone does not:
        // inside a workgroup the compiler lets global stores stay in flight across it), and only
        // after the barrier one lane takes the ticket.  Whoever draws the last one knows that every
        // other workgroup's lists are complete.  The wait is an asm statement with a memory clobber,
        // so the compiler can move neither the stores below it nor the ticket above it.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        uint32_t *flag = (uint32_t *)smem;
        uint32_t *ticket_word = p.tickets + tk * kTicketStride;
        if (tid == 0) {
            uint32_t ticket = __hip_atomic_fetch_add(ticket_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            flag[0] = (ticket == (uint32_t)(p.wgs_per_ticket - 1)) ? 1u : 0u;
        }
        __syncthreads();
        if (flag[0] == 0) return;
        trace_mark<TR>(p.trace, 10);  // drew the last ticket
        if (tid == 0)  // ready for the next call
            __hip_atomic_store(ticket_word, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

        // The last workgroup merges the splits of its columns, SU splits per batch of loads.
        constexpr int SU = tail_split_batch(KB);
        const int ncols = c_hi - c_lo;
        const u64 *src = p.lists + (int64_t)r * p.S * p.b * p.k_b;
        // The lists of NB consecutive splits from s0 on, merged into acc.  All NB loads are issued
        // before the first merge; the k_b <= KB slots that exist are loaded, the rest stay empty.
        // (Loads under a per-load condition would each sit in a branch of their own and wait for
        // one another.)
        auto batch = [&](auto nb_tag, int col, int s0, u64(&acc)[KB]) {
            constexpr int NB = decltype(nb_tag)::value;
            u64 th[NB][KB];
#pragma unroll
            for (int u = 0; u < NB; ++u)
#pragma unroll
                for (int j = 0; j < KB; ++j)
                    th[u][j] = __hip_atomic_load(&src[((int64_t)(s0 + u) * p.b + col) * p.k_b + (j < p.k_b ? j : p.k_b - 1)],
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int u = 0; u < NB; ++u) {
#pragma unroll
                for (int j = 0; j < KB; ++j)
                    if (j >= p.k_b) th[u][j] = 0ull;
                merge_topk<KB>(acc, th[u]);
            }
        };
        // lists of the splits [s0, s0 + SU) for s0 = s_first, s_first + s_step, ... of column `col`, merged
        // into acc; a batch cut short by the last split goes in pieces of 4, 2 and 1
        auto gather = [&](int col, int s_first, int s_step, u64(&acc)[KB]) {
            int s0 = s_first;
            for (; s0 + SU <= p.S; s0 += s_step) batch(std::integral_constant<int, SU>(), col, s0, acc);
            if (s0 < p.S) {  // s_step >= SU: at most one batch is cut short
                const int rem = p.S - s0;
                if (SU > 4 && (rem & 4)) {
                    batch(std::integral_constant<int, 4>(), col, s0, acc);
                    s0 += 4;
                }
                if (SU > 2 && (rem & 2)) {
                    batch(std::integral_constant<int, 2>(), col, s0, acc);
                    s0 += 2;
                }
                if (rem & 1) batch(std::integral_constant<int, 1>(), col, s0, acc);
            }
        };
        auto put = [&](int col, const u64(&acc)[KB]) {
            if (p.stage2) {
#pragma unroll
                for (int j = 0; j < KB; ++j)
                    if (j < p.k_b) cand[col * p.k_b + j] = acc[j];
            } else {
                const int64_t o = (int64_t)r * p.k + (int64_t)col * p.k_b;
#pragma unroll
                for (int j = 0; j < KB; ++j)
                    if (j < p.k_b) write_composite<ELT>(acc[j], p.out_vals, p.out_idx, o + j);
            }
        };
        if (p.tail_tpc_shift == 0) {
            // one lane per column (a plain loop: the compiler may overlap its iterations)
            for (int ci = tid; ci < ncols; ci += T) {
                u64 acc[KB];
#pragma unroll
                for (int j = 0; j < KB; ++j) acc[j] = 0ull;
                const int col = c_lo + ci - rot + (c_lo + ci < rot ? p.b : 0);
                gather(col, 0, SU, acc);
                put(col, acc);
            }
        } else {
            // Fewer columns than lanes and many splits: tpc lanes side by side share a column,
            // each merges every tpc-th batch, then a butterfly of shuffles joins them.
            const int tpc_shift = p.tail_tpc_shift, tpc = 1 << tpc_shift;  // chosen on the host: tpc * ncols <= T
            const int part = tid & (tpc - 1);
            const int ci = tid >> tpc_shift;
            const bool ok = ci < ncols;
            u64 acc[KB];
#pragma unroll
            for (int j = 0; j < KB; ++j) acc[j] = 0ull;
            const int col = c_lo + ci - rot + (c_lo + ci < rot ? p.b : 0);
            if (ok) gather(col, part * SU, tpc * SU, acc);
            for (int off = 1; off < tpc; off <<= 1) {
                u64 theirs[KB];
#pragma unroll
                for (int j = 0; j < KB; ++j) theirs[j] = shfl_xor_u64(acc[j], off);
                merge_topk<KB>(acc, theirs);
            }
            if (ok && part == 0) put(col, acc);
        }
        trace_mark<TR>(p.trace, 11);  // the other workgroups' lists are merged
        if (!p.stage2) return;
        __syncthreads();
    }

    // ---------------------------------------------------------------- Stage 2 in LDS
    trace_mark<TR>(p.trace, 3);  // all candidates of the row are in LDS
    if (sort_select_fits<ELT>(p.b * p.k_b, p.k, p.idx_bits)) {
        if (sort_select(cand, p.b * p.k_b, p.k, p.out_vals, p.out_idx, (int64_t)r)) {
            trace_mark<TR>(p.trace, 8);
            return;
        }
        __syncthreads();  // (few positive candidates)
    }
    select_write<ELT, TR>(cand, p.b * p.k_b, p.k, p.idx_bits, p.out_vals, p.out_idx, (int64_t)r, p.trace);
    trace_mark<TR>(p.trace, 8);  // outputs written
}

template <int ELT, int V, int KB, int U, int MAXT, bool PKF, bool TR = false, bool RF = false>
// (pooled floors: the launches are laid out for four wavefronts per SIMD, and three are two rounds: 128 x 2^20, b = 128: 116 -> 159 us)
__global__ void __launch_bounds__(MAXT, RF && V <= 2 ? 4 : 1) stage1_kernel(S1Params p) {
    extern __shared__ __align__(16) unsigned char smem[];
    trace_mark<TR>(p.trace, 0);  // the wavefront has started
    constexpr int ES = (ELT == ATK_F32) ? 4 : 2;
    constexpr bool PK = PKF && ELT == ATK_BF16 && KB >= 2;  // packed 32-bit queues (host: rows per split < 65534)
    // queues of distinct 64-bit words, fed k_b matrix rows at a time (the pooled floors work on the other form)
    constexpr bool BATCH = KB >= 8 && !PK && !RF;
    const int tid = threadIdx.x, T = blockDim.x;
    int wg = blockIdx.x, cb, sp, r, cgl, ph;
    divmod(wg, p.colblocks, p.cb_shift, wg, cb);
    divmod(wg, p.S, p.s_shift, r, sp);
    divmod(tid, p.Gw, p.gw_shift, ph, cgl);
    const int cg = cb * p.Gw + cgl;
    const bool active = (ph < p.P) && (cg < p.G);
    const int col0 = cg * V;
    // Rows whose first element is not aligned to a V-element load (n not a multiple of V) are
    // read from the aligned address just before: the row is taken as a virtual row that starts
    // `rot` elements early, so virtual column c holds bucket c - rot (mod b) and element
    // (t, c) of the virtual matrix is column t*b + c - rot of the row.  The first `rot` virtual
    // elements belong to the previous row and are skipped.
    const int rot = (V > 1) ? (int)(((int64_t)r * p.n) & (V - 1)) : 0;
    const bool carry = p.rem + rot >= p.b;       // the virtual row has one more full matrix row
    const int Lr = p.L + (carry ? 1 : 0);       // full matrix rows of the virtual row
    const int remr = p.rem + rot - (carry ? p.b : 0);  // columns of its ragged last matrix row
    int eph = p.extra_ph + (carry ? 1 : 0);     // the row phase that takes the ragged row
    if (eph >= p.P) eph -= p.P;
    const int t0 = sp * p.rows_per_split;
    const int t_end = (sp == p.S - 1) ? Lr : min(Lr - t0, p.rows_per_split) + t0;
    const int t1 = min(t_end, kRowsAhead);  // (where the scans stop that look ahead)
    auto bucket_of = [&](int c) { return c - rot + (c < rot ? p.b : 0); };

    // One slot per bucket, no hand-over through memory: the lanes that share a column meet in LDS by
    // atomic maximum on the composite (the merge of Appendix A's per-thread queues, for queues of one
    // slot), straight into the candidate array that Stage 2 selects from.  The array - and the counts
    // of Stage 2's histogram - are cleared here, while nothing else is going on.
    if constexpr (KB == 1) {
        if (p.lds_max) {
            u64 *cand = (u64 *)(smem + p.lds_cand_off);
            const int wcols = min(p.Gw * V, p.b - cb * p.Gw * V);
            for (int i = tid; i < wcols; i += T) cand[i] = 0ull;
            if (p.stage2 && binned_fits(wcols) && p.bound_ok) {
                uint32_t *cnt = binned_cnt(cand, wcols), *misc = binned_misc(cand, wcols);
                for (int i = tid; i < (1 << binned_lg_bins(wcols)); i += T) cnt[i] = 0u;
                if (tid < 8) misc[tid] = (tid == 1) ? 0xffffffffu : 0u;  // (see select_binned: flag, range, lower bounds)
            }
            __syncthreads();
        }
    }

    float val[V][KB];
    int tt[V][KB];
    int32_t pk[PK ? V : 1][PK ? KB : 1];
    double qw[BATCH ? V : 1][BATCH ? KB : 1];  // BATCH: the queues, as row words
    float last_f[BATCH ? V : 1];            // ... and the value of each queue's last slot (NaN while it is empty)
    LazyQueue<KB> lazy[RF ? V : 1];
    int flushed = KB * V;  // RF: times that waiting elements were worked in of late (at the start all elements enter)
    if constexpr (RF) {
#pragma unroll
        for (int e = 0; e < V; ++e) lazy[e].clear();
    }
#pragma unroll
    for (int e = 0; e < V; ++e)
#pragma unroll
        for (int j = 0; j < KB; ++j) {
            val[e][j] = __uint_as_float(0x7fc00000u);
            tt[e][j] = kEmptyT;
            if constexpr (PK) pk[e][j] = kEmptyPk;
            if constexpr (BATCH) {
                qw[e][j] = no_word();
                last_f[e] = __uint_as_float(0x7fc00000u);
            }
        }
#define ATK_FEED_ELEM(e, xb, row)                                                                    \
    do {                                                                                             \
        if constexpr (PK)                                                                            \
            insert_pk<KB>(pk[e], pack_bf16(xb, (uint32_t)(0xffff - ((row) - t0))));                  \
        else if constexpr (RF)                                                                       \
            lazy[e].feed(xb, pooled_rows + ((row) - t_resume), flushed);                             \
        else if constexpr (BATCH)                                                                    \
            insert_word<KB>(qw[e], row_word(xb, (uint32_t)(((row) - t0 - ph) / p.P)));               \
        else                                                                                         \
            insert<KB>(val[e], tt[e], __uint_as_float(xb), (row));                                   \
    } while (0)
#define ATK_FEED_VEC(vec, row)                                                                       \
    do {                                                                                             \
        if constexpr (PK)                                                                            \
            scan_vec_pk<ELT, V, KB>(pk, vec, (row) - t0);                                            \
        else if constexpr (BATCH || RF) {                                                            \
            _Pragma("unroll") for (int e_ = 0; e_ < V; ++e_) ATK_FEED_ELEM(e_, (elem_bits<ELT, V>(vec, e_)), (row)); \
        } else                                                                                       \
            scan_vec<ELT, V, KB>(val, tt, vec, (row));                                               \
    } while (0)

    // ---------------------------------------------------------------- pooled floors (instances of their own: RF)
    // Eight unpacked slots, several lanes of the workgroup on a column, many matrix rows per lane, rows that start on a
    // load boundary (rot = 0; the host sees to all of it).  What a lane has seen alone is a poor bound on what still
    // matters: after t rows one element in t/8 still enters its queue, and with 128 lane-columns per wavefront some
    // lane always needs the insertion.  So after `stop` load batches of U matrix rows - the same number in every lane, and every lane
    // has at least that many - the lanes of a column pool what they hold: between them they have seen all elements of
    // a stretch of the row; the eighth best of that stretch bounds the column's final eighth best from below, and every
    // element still to come has a higher index than all of the stretch, so it has to beat that value outright.
    // The lanes pool their queues' value keys: a butterfly
    // inside the wavefront where lanes of a column sit side by side, then through the exchange area in LDS (free
    // until the lists are merged at the end).  Again after four times as many batches, and so on: as elements wait for the queues, a
    // floor that lags costs little (stops at 32 matrix rows of a lane, 128, 512, ... against 16, 64, ...: 128 x 2^20, b = 512 119 -> 107 us, its
    // rising rows 129 -> 126 and constant ones 114 -> 107; 512 x 65536, b = 16 37.6 -> 36.7, 48.6 -> 45.9, 37.2 -> 35.3).
    const int64_t row_bytes = (int64_t)p.b * ES;
    int pooled_rows = 0;  // matrix rows that a lane feeds here: they are numbered 0, 1, ..., and the later ones pooled_rows + (row - t_resume)
    if constexpr (RF) {
        static_assert(!RF || (KB == 8 && U == KB && !PKF), "pooled floors: eight unpacked slots");
        const int step = p.P;
        const int nfull = ((t1 - t0) / p.P) / U;  // full batches that every row phase has
        pooled_rows = nfull * U;
        // (the next batch's loads are issued before the current one is worked on, and before the lanes meet)
        int stop = max(1, 4 * p.refresh / U);
        constexpr int kCrowd = 5 * V;  // (4 and 6 a column and batch measure the same)
        RowVec<ELT, V> v[U], w[U];
        const int64_t stride_bytes = (int64_t)step * row_bytes;
        // (scalar addresses and one offset for all of a lane's loads; the host sees to it that it fits)
        const unsigned char *next = (const unsigned char *)p.x + ((int64_t)r * p.n * ES + t0 * row_bytes);
        const uint32_t lane_off = (uint32_t)ph * (uint32_t)row_bytes + (uint32_t)col0 * ES;
        auto load = [&](RowVec<ELT, V> (&to)[U]) {
            uint32_t off = lane_off;
            asm volatile("" : "+v"(off));
#pragma unroll
            for (int u = 0; u < U; ++u) to[u] = load_vec<ELT, V>(next + u * stride_bytes + off);
        };
        if (active && nfull > 0) load(v);
        for (int i = 1; i <= nfull; ++i) {
            if (i < nfull) next += U * stride_bytes;  // (else the last batch again)
            if (active) {
                const bool sorted = __builtin_amdgcn_readfirstlane(flushed) >= kCrowd;  // (uniform: all active lanes count the same)
                if (!sorted) load(w);  // (sorting takes the registers of a batch)
                if (sorted) {
                    flushed = 0;
#pragma unroll
                    for (int e = 0; e < V; ++e) {
                        uint32_t bits[U];
#pragma unroll
                        for (int u = 0; u < U; ++u) bits[u] = elem_bits<ELT, V>(v[u], e);
                        if (lazy[e].feed_sorted(bits, (i - 1) * U)) flushed = kCrowd;
                    }
                    load(w);
                } else {
                    flushed = 0;
#pragma unroll
                    for (int u = 0; u < U; ++u)
#pragma unroll
                        for (int e = 0; e < V; ++e) lazy[e].feed(elem_bits<ELT, V>(v[u], e), (i - 1) * U + u, flushed);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = w[u];
            }
            if (i != stop || i == nfull) continue;  // uniform
            stop *= 4;
            uint32_t keys[V][KB];
#pragma unroll
            for (int e = 0; e < V; ++e) lazy[e].flush();
#pragma unroll
            for (int e = 0; e < V; ++e)
#pragma unroll
                for (int j = 0; j < KB; ++j)
                    keys[e][j] = word_key(lazy[e].q[j]);
            if (p.wave_merge) {
                for (int off = p.Gw; off < kWave; off <<= 1) {
#pragma unroll
                    for (int e = 0; e < V; ++e) {
                        uint32_t theirs[KB];
#pragma unroll
                        for (int j = 0; j < KB; ++j) theirs[j] = (uint32_t)__shfl_xor((int)keys[e][j], off, kWave);
                        merge_keys<KB>(keys[e], theirs);
                    }
                }
            }
            if (p.nparts > 1) {
                uint32_t *xk = (uint32_t *)(smem + p.lds_xch_off);  // [part][column of the workgroup][slot]
                const int part = p.wave_merge ? (tid >> 6) : ph;
                const bool holder = active && (!p.wave_merge || (tid & (kWave - 1)) < p.Gw);
                const int64_t pstride = (int64_t)p.Gw * V;
                if (holder) {
#pragma unroll
                    for (int e = 0; e < V; ++e)
#pragma unroll
                        for (int j = 0; j < KB; ++j) xk[((int64_t)part * pstride + cgl * V + e) * KB + j] = keys[e][j];
                }
                __syncthreads();
                if (active) {
#pragma unroll
                    for (int e = 0; e < V; ++e) {
#pragma unroll
                        for (int j = 0; j < KB; ++j) keys[e][j] = xk[((int64_t)cgl * V + e) * KB + j];
                        for (int q = 1; q < p.nparts; ++q) {
                            uint32_t theirs[KB];
#pragma unroll
                            for (int j = 0; j < KB; ++j) theirs[j] = xk[((int64_t)q * pstride + cgl * V + e) * KB + j];
                            merge_keys<KB>(keys[e], theirs);
                        }
                    }
                }
                __syncthreads();  // (the area is written again at the next stop, and by the merge at the end)
            }
            if (active) {
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const uint32_t fk = keys[e][KB - 1];
                    if (fk != 0u)  // eight elements of the column have been seen
                        lazy[e].last = fmaxf(lazy[e].last, __uint_as_float(bits_of_ukey(fk)));
                }
            }
        }
    }

    // ---------------------------------------------------------------- streaming scan
    const int t_resume = t0 + ph + pooled_rows * p.P;  // the lane's next matrix row
    if (active) {
        const unsigned char *base = (const unsigned char *)p.x + ((int64_t)r * p.n - rot + (int64_t)col0) * ES;
        const int step = p.P;
        int t = t_resume;
        if (V > 1 && rot > 0 && cg == 0 && t == 0 && t < t1) {
            // the head of the virtual row: its first `rot` elements are not this row's
            RowVec<ELT, V> v = load_vec<ELT, V>(base);
#pragma unroll
            for (int e = 0; e < V; ++e)
                if (e >= rot) ATK_FEED_ELEM(e, (elem_bits<ELT, V>(v, e)), 0);
            t += step;
        }
        if constexpr (BATCH) {
            // k_b matrix rows at a time; the next batches' loads (two with eight slots) are issued before this one is worked on.  Rows past
            // the end re-read the batch's first row and are dropped.  A second batch ahead is for launches of two wavefronts per SIMD,
            // whose lanes wait for memory together: 256 x 65536, k = 16384, b = 2048, k_b = 8: 29.2 -> 27.2 us; 128 rows 17.4 -> 16.9,
            // 64 rows 13.4 -> 12.5; 128 x 2^20, b = 1024: 138 -> 130.
            constexpr int D = KB == 8 ? 2 : 1;  // batches ahead
            RowVec<ELT, V> v[KB], w[D][KB];
            uint32_t seq = (uint32_t)((t - t0 - ph) / step);  // number of the batch's first row among the lane's
            bool have = t < t1;
            auto fetch = [&](RowVec<ELT, V> (&to)[KB], int tb) {
#pragma unroll
                for (int u = 0; u < KB; ++u) {
                    const int tu = tb + u * step;
                    to[u] = load_vec<ELT, V>(base + (int64_t)(tu < t1 ? tu : tb) * row_bytes);
                }
            };
            if (have) {
                fetch(v, t);
                if (D == 2 && t + KB * step < t1) fetch(w[0], t + KB * step);
            }
            while (have) {
                const int tn = t + KB * step;
                const bool more = tn < t1;
                if (tn + (D - 1) * KB * step < t1) fetch(w[D - 1], tn + (D - 1) * KB * step);
                if (__ballot(t + (KB - 1) * step >= t1) != 0ull) {  // (a lane's last rows)
#pragma unroll
                    for (int u = 1; u < KB; ++u)
                        if (t + u * step >= t1) {
#pragma unroll
                            for (int w = 0; w < RowVec<ELT, V>::kWords; ++w) v[u].w[w] = ELT == ATK_F32 ? kNoWordBits : (kNoWordBits | (kNoWordBits >> 16));
                        }
                }
                // one compare per element, and a wavefront-uniform skip, keep long buckets cheap: an element enters
                // only if it beats the queue's last slot (equal values never displace earlier ones)
                bool any = false;
#pragma unroll
                for (int u = 0; u < KB; ++u)
#pragma unroll
                    for (int e = 0; e < V; ++e) any = any || !(__uint_as_float(elem_bits<ELT, V>(v[u], e)) <= last_f[e]);
                if (__ballot(any) != 0ull) {
                    const bool first = __ballot(is_word(qw[V - 1][0])) == 0ull;  // (the head of a virtual row holds its last column at least)
#pragma unroll
                    for (int e = 0; e < V; ++e) {
                        double bt[KB];
#pragma unroll
                        for (int u = 0; u < KB; ++u) bt[u] = row_word(elem_bits<ELT, V>(v[u], e), seq + (uint32_t)u);
                        sort_desc<KB>(bt);
                        if (first) {
#pragma unroll
                            for (int j = 0; j < KB; ++j) qw[e][j] = bt[j];
                        } else {
                            merge_words<KB>(qw[e], bt);
                        }
                        last_f[e] = __uint_as_float(word_bits(qw[e][KB - 1]));
                    }
                }
                seq += KB;
#pragma unroll
                for (int u = 0; u < KB; ++u) {
                    v[u] = w[0][u];
                    if (D == 2) w[0][u] = w[D - 1][u];
                }
                t = tn;
                have = more;
            }
        } else if (KB == 8) {
            // The next batch's loads are issued before the current one is worked on (measured:
            // 4-7 % at eight slots, nothing or a loss at other queue lengths).
            RowVec<ELT, V> v[U], w[U];
            bool have = t + (U - 1) * step < t1;
            if (have) {
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = load_vec<ELT, V>(base + (int64_t)(t + u * step) * row_bytes);
            }
            while (have) {
                const int tn = t + U * step;
                const bool more = tn + (U - 1) * step < t1;
                if (more) {
#pragma unroll
                    for (int u = 0; u < U; ++u) w[u] = load_vec<ELT, V>(base + (int64_t)(tn + u * step) * row_bytes);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) ATK_FEED_VEC(v[u], t + u * step);
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = w[u];
                t = tn;
                have = more;
            }
        } else {
            if (KB == 1 && ELT == ATK_BF16) {
                // One pointer per lane, advanced by a batch at a time, the batch's loads at fixed strides
                // from it, and the whole batch in flight before the first row is looked at: the barrier
                // keeps the scheduler from starting on the first rows while the addresses of the last are
                // still being worked out, as it does for bf16 in the plain form below (2048 x 8192:
                // 8.6 -> 8.3 us).  For f32 and with queues the plain form schedules as well or better.
                const int64_t stride_bytes = (int64_t)step * row_bytes;
                const unsigned char *ptr = base + (int64_t)t * row_bytes;
                for (; t + (U - 1) * step < t1; t += U * step, ptr += U * stride_bytes) {
                    RowVec<ELT, V> v[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) v[u] = load_vec<ELT, V>(ptr + u * stride_bytes);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < U; ++u) ATK_FEED_VEC(v[u], t + u * step);
                }
            } else {
                for (; t + (U - 1) * step < t1; t += U * step) {
                    RowVec<ELT, V> v[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) v[u] = load_vec<ELT, V>(base + (int64_t)(t + u * step) * row_bytes);
#pragma unroll
                    for (int u = 0; u < U; ++u) ATK_FEED_VEC(v[u], t + u * step);
                }
            }
        }
        if (t < t1) {
            // Fewer than U rows are left: they go in pieces of U/2, U/4, ... 1 rows, each piece's loads
            // issued together.  One row at a time, every load would wait out a full memory latency, which
            // on rows of a few batches per lane is most of the kernel (n = 128256 against 131072: +3 us).
            int nr = (t1 - t + step - 1) / step;
            if (KB == 1 && U >= 8 && nr > U / 2) {
                // more than half a batch: a whole batch at once, the loads past the end re-reading row t
                // (for a running maximum a row fed twice changes nothing) - one memory latency, not three
                RowVec<ELT, V> v[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int tu = t + u * step;
                    v[u] = load_vec<ELT, V>(base + (int64_t)(tu < t1 ? tu : t) * row_bytes);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int tu = t + u * step;
                    ATK_FEED_VEC(v[u], tu < t1 ? tu : t);
                }
                nr = 0;
            }
#define ATK_PIECE(NP)                                                                                          \
    if (NP < U && (nr & NP)) {                                                                                 \
        RowVec<ELT, V> v[NP];                                                                                  \
        _Pragma("unroll") for (int u = 0; u < NP; ++u) v[u] = load_vec<ELT, V>(base + (int64_t)(t + u * step) * row_bytes); \
        _Pragma("unroll") for (int u = 0; u < NP; ++u) ATK_FEED_VEC(v[u], t + u * step);                       \
        t += NP * step;                                                                                        \
    }
            ATK_PIECE(8)
            ATK_PIECE(4)
            ATK_PIECE(2)
            ATK_PIECE(1)
#undef ATK_PIECE
        }
        if (t1 < t_end) {  // (uniform)
            for (uint32_t tr = (uint32_t)(t0 + ph) + (uint32_t)((t1 - t0 - ph + step - 1) / step) * (uint32_t)step; tr < (uint32_t)t_end; tr += (uint32_t)step) {
                RowVec<ELT, V> v = load_vec<ELT, V>(base + (int64_t)tr * row_bytes);
                ATK_FEED_VEC(v, (int)tr);
            }
        }
        // The (virtual) row does not end on a matrix row: the last matrix row holds only its
        // first `remr` columns (the short buckets of Figure 2).  It has the highest indices, so
        // it is fed last.
        if (remr > 0 && sp == p.S - 1 && ph == eph && col0 < remr) {
            const unsigned char *last = base + (int64_t)Lr * row_bytes;
            if (col0 + V <= remr) {
                RowVec<ELT, V> v = load_vec<ELT, V>(last);
                ATK_FEED_VEC(v, Lr);
            } else {
#pragma unroll
                for (int e = 0; e < V; ++e)
                    if (col0 + e < remr) {
                        RowVec<ELT, 1> one = load_vec<ELT, 1>(last + e * ES);
                        ATK_FEED_ELEM(e, (elem_bits<ELT, 1>(one, 0)), Lr);
                    }
            }
        }
    }

#undef ATK_FEED_VEC
#undef ATK_FEED_ELEM
    trace_mark<TR>(p.trace, 1);  // its share of the row is in
    if constexpr (BATCH) {
#pragma unroll
        for (int e = 0; e < V; ++e)
#pragma unroll
            for (int j = 0; j < KB; ++j)
                if (is_word(qw[e][j])) {
                    val[e][j] = __uint_as_float(word_bits(qw[e][j]));
                    tt[e][j] = t0 + ph + (int)word_number(qw[e][j]) * p.P;
                }
    }
    if constexpr (RF) {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            lazy[e].flush();
#pragma unroll
            for (int j = 0; j < KB; ++j)
                if (is_word(lazy[e].q[j])) {
                    val[e][j] = __uint_as_float(word_bits(lazy[e].q[j]));
                    const int t = (int)word_number(lazy[e].q[j]);
                    tt[e][j] = t < pooled_rows ? t0 + ph + t * p.P : t_resume + (t - pooled_rows);
                }
        }
    }
    if (BATCH || RF || (PK && p.direct)) {
        bool zero = false;
#pragma unroll
        for (int e = 0; e < V; ++e)
#pragma unroll
            for (int j = 0; j < KB; ++j) {
                if constexpr (PK) unpack_bf16(pk[e][j], t0, val[e][j], tt[e][j]);
                zero = zero || __float_as_uint(val[e][j]) == 0u;
            }
        if (__ballot(zero) != 0ull) {  // +0 or -0: the element itself says (a column's loads in flight together)
            typedef typename std::conditional<ELT == ATK_F32, uint32_t, uint16_t>::type word_t;
            const word_t *row = (const word_t *)p.x + (int64_t)r * p.n;
#pragma unroll
            for (int e = 0; e < V; ++e) {
                uint32_t own[KB];
#pragma unroll
                for (int j = 0; j < KB; ++j)
                    own[j] = row[__float_as_uint(val[e][j]) == 0u ? (int64_t)tt[e][j] * p.b + col0 + e - rot : 0];
#pragma unroll
                for (int j = 0; j < KB; ++j)
                    if (__float_as_uint(val[e][j]) == 0u) val[e][j] = __uint_as_float(own[j] << (ELT == ATK_F32 ? 0 : 16));
            }
        }
    }

    // ---------------------------------------------------------------- every lane owns whole buckets
    if (p.direct) {
        if (!active) return;
        const int64_t o = (int64_t)r * p.k + (int64_t)col0 * p.k_b;
        if (p.vec_store && rot == 0 && p.k_b == KB && (V * KB) % ((ELT == ATK_F32) ? 4 : 8) == 0) {
            constexpr int N = V * KB;  // contiguous outputs of this lane
            uint32_t ob[N];
            int32_t oi[N];
#pragma unroll
            for (int e = 0; e < V; ++e)
#pragma unroll
                for (int j = 0; j < KB; ++j) {
                    ob[e * KB + j] = __float_as_uint(val[e][j]);
                    oi[e * KB + j] = tt[e][j] * p.b + col0 + e;
                }
            typedef uint32_t v4u __attribute__((ext_vector_type(4)));
            constexpr int NV = ELT == ATK_F32 ? N / 4 : N / 8;
            v4u wi[N < 4 ? 1 : N / 4], wv[NV < 1 ? 1 : NV];
#pragma unroll
            for (int q = 0; q < N / 4; ++q) wi[q] = v4u{(uint32_t)oi[4 * q], (uint32_t)oi[4 * q + 1], (uint32_t)oi[4 * q + 2], (uint32_t)oi[4 * q + 3]};
#pragma unroll
            for (int q = 0; q < NV; ++q)
                if (ELT == ATK_F32)
                    wv[q] = v4u{ob[4 * q], ob[4 * q + 1], ob[4 * q + 2], ob[4 * q + 3]};
                else
                    wv[q] = v4u{(ob[8 * q] >> 16) | (ob[8 * q + 1] & 0xffff0000u), (ob[8 * q + 2] >> 16) | (ob[8 * q + 3] & 0xffff0000u),
                                (ob[8 * q + 4] >> 16) | (ob[8 * q + 5] & 0xffff0000u), (ob[8 * q + 6] >> 16) | (ob[8 * q + 7] & 0xffff0000u)};
            // A wavefront's outputs lie side by side, but a lane has up to 128 bytes of them: stored from the lanes, sixteen bytes at a time, every store
            // touches as many lines as there are lanes, and the address units have them one by one.  They go through LDS first, a wavefront's
            // own part of it, in an order that spreads over the banks.  f32, 128 x 65536, k = 16384, b = 2048, k_b = 8: 16.3 -> 14.5 us; 256 rows
            // 25.8 -> 21.0; 128 x 2^20, k = 2^18, b = 2^15: 146 -> 132.
            auto put = [&](auto &w, v4u *to) {
                constexpr int NW = sizeof(w) / sizeof(w[0]), kTurn = NW >= 16 ? 0 : NW >= 8 ? 1 : NW >= 4 ? 2 : 3;  // (lanes to the 64 banks, as a power of two)
                if constexpr (NW > 1 && N >= 16) {
                    if (p.staged && __ballot(true) == ~0ull) {
                        const int lane = tid & (kWave - 1);
                        v4u *own = (v4u *)smem + (tid - lane) * (N / 4);  // (values and indices in turn)
                        __builtin_amdgcn_wave_barrier();
#pragma unroll
                        for (int q = 0; q < NW; ++q) own[lane * NW + (q ^ ((lane >> kTurn) & (NW - 1)))] = w[q];
                        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                        __builtin_amdgcn_wave_barrier();
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
                        for (int q = 0; q < NW; ++q) {
                            const int at = q * kWave + lane, of = at / NW;
                            w[q] = own[of * NW + ((at % NW) ^ ((of >> kTurn) & (NW - 1)))];
                        }
                        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                        __builtin_amdgcn_wave_barrier();
                        v4u *first = to - lane * NW;
#pragma unroll
                        for (int q = 0; q < NW; ++q) first[q * kWave + lane] = w[q];
                        return;
                    }
                }
#pragma unroll
                for (int q = 0; q < NW; ++q) to[q] = w[q];
            };
            put(wv, (v4u *)((unsigned char *)p.out_vals + o * ES));
            put(wi, (v4u *)(p.out_idx + o));
        } else {
#pragma unroll
            for (int e = 0; e < V; ++e)
#pragma unroll
                for (int j = 0; j < KB; ++j)
                    if (j < p.k_b) {
                        const int64_t pos = (int64_t)r * p.k + (int64_t)bucket_of(col0 + e) * p.k_b + j;
                        store_val<ELT>(p.out_vals, pos, __float_as_uint(val[e][j]));
                        p.out_idx[pos] = tt[e][j] * p.b + col0 + e - rot;
                    }
        }
        return;
    }

    // ---------------------------------------------------------------- one slot, one workgroup per row or column block
    if constexpr (KB == 1) {
        if (p.lds_max) {
            u64 *cand = (u64 *)(smem + p.lds_cand_off);
            const int colbase = cb * p.Gw * V;
            const int wcols = min(p.Gw * V, p.b - colbase), groups = wcols / V;  // (a last column block may be narrower: fewer than Gw)
            const bool binned = p.stage2 && binned_fits(wcols) && p.bound_ok;
            uint32_t k_min = 0xffffffffu, k_max = 0u;
            bool whole = active;  // this lane holds an element of every one of its V columns
            if (active) {
#pragma unroll
                for (int e = 0; e < V; ++e) whole = whole && tt[e][0] != kEmptyT;
#pragma unroll
                for (int e = 0; e < V; ++e)
                    if (tt[e][0] != kEmptyT) {
                        const u64 c = make_composite(__float_as_uint(val[e][0]), tt[e][0] * p.b + col0 + e - rot);
                        // column e of column group cgl sits at e * groups + cgl: side-by-side lanes, side-by-side words, wcols of them
                        __hip_atomic_fetch_max(&cand[e * groups + cgl], c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        const uint32_t key = (uint32_t)(c >> 32);
                        k_min = key < k_min ? key : k_min;
                        k_max = key > k_max ? key : k_max;
                    }
            }
            if (binned) {
                // the range of the value keys that Stage 2 spreads its bins over: the lanes' maxima span at least
                // the range of the columns' maxima.  Folded here, before the barrier, it costs the wavefronts that
                // finish reading early nothing.
                uint32_t *misc = binned_misc(cand, wcols);
                k_min = wave_min_u32(k_min);
                k_max = wave_max_u32(k_max);
                // a wavefront whose 64 lanes between them hold an element of every column of the row: its minimum is
                // a lower bound on the smallest candidate, usually far tighter than the minimum over all lanes
                const bool cover = p.Gw <= kWave && __ballot(whole) == ~0ull;
                if ((tid & (kWave - 1)) == 0) {
                    atomicMin(&misc[1], k_min);
                    atomicMax(&misc[2], k_max);
                    if (cover) atomicMax(&misc[4], k_min);
                }
            }
            trace_mark<TR>(p.trace, 2);  // this wavefront's maxima are in
            __syncthreads();
            if (!p.stage2) {
                for (int lc = tid; lc < wcols; lc += T)
                    write_composite<ELT>(cand[(lc % V) * groups + lc / V], p.out_vals, p.out_idx,
                                         (int64_t)r * p.k + bucket_of(colbase + lc));
                trace_mark<TR>(p.trace, 9);
                return;
            }
            trace_mark<TR>(p.trace, 3);  // all candidates of the row are in LDS, their key range is known
            if (binned)
                select_binned<ELT, TR>(cand, wcols, p.k, p.idx_bits, p.out_vals, p.out_idx, (int64_t)r, p.trace);
            else
                select_write<ELT, TR>(cand, wcols, p.k, p.idx_bits, p.out_vals, p.out_idx, (int64_t)r, p.trace);
            trace_mark<TR>(p.trace, 8);
            trace_mark<TR>(p.trace, 9);
            return;
        }
    }

    // ---------------------------------------------------------------- packed queues meet as they are
    // The words of the lanes that share a column count the same split's matrix rows, so their queues are merged as words of 32 bits, and only
    // what is left of them becomes values, rows and composites.
    if constexpr (PK) {
        u64 *cand = (u64 *)(smem + p.lds_cand_off);
        auto emit = [&](int c, const auto &q) {  // columns c, c + 1, ... of the (virtual) matrix, a queue each
            constexpr int N = sizeof(q) / sizeof(q[0]);
            float v[N][KB];
            int t[N][KB];
            bool zero = false;
#pragma unroll
            for (int e = 0; e < N; ++e)
#pragma unroll
                for (int j = 0; j < KB; ++j) {
                    unpack_bf16(q[e][j], t0, v[e][j], t[e][j]);
                    zero = zero || __float_as_uint(v[e][j]) == 0u;
                }
            // +0 or -0: the element itself says (the loads of all columns in flight together: 6 x 222784, k = 15104, b = 1888, k_b = 8, mostly zeros:
            // 10.0 us with a wait for each column, 9.0)
            if (__ballot(zero) != 0ull) {
                const uint16_t *row = (const uint16_t *)p.x + (int64_t)r * p.n;
                uint32_t own[N][KB];
#pragma unroll
                for (int e = 0; e < N; ++e)
#pragma unroll
                    for (int j = 0; j < KB; ++j) own[e][j] = row[__float_as_uint(v[e][j]) == 0u ? (int64_t)t[e][j] * p.b + c + e - rot : 0];
#pragma unroll
                for (int e = 0; e < N; ++e)
#pragma unroll
                    for (int j = 0; j < KB; ++j)
                        if (__float_as_uint(v[e][j]) == 0u) v[e][j] = __uint_as_float(own[e][j] << 16);
            }
#pragma unroll
            for (int e = 0; e < N; ++e) {
                u64 list[KB];
#pragma unroll
                for (int j = 0; j < KB; ++j) list[j] = t[e][j] != kEmptyT ? make_composite(__float_as_uint(v[e][j]), t[e][j] * p.b + c + e - rot) : 0ull;
                emit_list<ELT, KB>(p, r, sp, bucket_of(c + e), list, cand);
            }
        };
        if (p.wave_merge) {
            for (int off = p.Gw; off < kWave; off <<= 1) {
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    int32_t theirs[KB];
#pragma unroll
                    for (int j = 0; j < KB; ++j) theirs[j] = __shfl_xor(pk[e][j], off, kWave);
                    merge_pk<KB>(pk[e], theirs);
                }
            }
        }
        if (p.nparts > 1) {
            int32_t *xch = (int32_t *)(smem + p.lds_xch_off);  // [part][column of the workgroup][slot]
            const int part = p.wave_merge ? (tid >> 6) : ph, colbase = cb * p.Gw * V, wcols = min(p.Gw * V, p.b - colbase), stride = p.Gw * V;
            if (active && (!p.wave_merge || (tid & (kWave - 1)) < p.Gw)) {
#pragma unroll
                for (int e = 0; e < V; ++e)
#pragma unroll
                    for (int j = 0; j < KB; ++j) xch[((int64_t)part * stride + cgl * V + e) * KB + j] = pk[e][j];
            }
            __syncthreads();
            for (int c = tid; c < wcols; c += T) {
                int32_t acc[1][KB];
#pragma unroll
                for (int j = 0; j < KB; ++j) acc[0][j] = xch[(int64_t)c * KB + j];
                for (int q = 1; q < p.nparts; ++q) {
                    int32_t theirs[KB];
#pragma unroll
                    for (int j = 0; j < KB; ++j) theirs[j] = xch[((int64_t)q * stride + c) * KB + j];
                    merge_pk<KB>(acc[0], theirs);
                }
                emit(colbase + c, acc);
            }
        } else if (active && (!p.wave_merge || (tid & (kWave - 1)) < p.Gw)) {
            emit(col0, pk);
        }
        trace_mark<TR>(p.trace, 2);
        const bool all = p.stage2 != 0;
        row_tail<ELT, KB, TR>(p, r, all ? (int64_t)r : (int64_t)r * p.colblocks + cb, all ? 0 : cb * p.Gw * V,
                              all ? p.b : min(p.b, (cb + 1) * p.Gw * V), all ? 0 : rot, smem);
        trace_mark<TR>(p.trace, 9);
        return;
    }

    if constexpr (!PK) {
    // ---------------------------------------------------------------- to composites
    u64 comp[V][KB];
#pragma unroll
    for (int e = 0; e < V; ++e)
#pragma unroll
        for (int j = 0; j < KB; ++j)
            comp[e][j] = (tt[e][j] != kEmptyT)
                             ? make_composite(__float_as_uint(val[e][j]), tt[e][j] * p.b + col0 + e - rot)
                             : 0ull;

    // ---------------------------------------------------------------- merge inside the wavefront
    // With fewer than 64 column groups the lanes l, l+Gw, l+2Gw, ... of a wavefront share
    // their columns: a butterfly over those lane strides leaves the merged list in all of them.
    if (p.wave_merge) {
        for (int off = p.Gw; off < kWave; off <<= 1) {
#pragma unroll
            for (int e = 0; e < V; ++e) {
                u64 theirs[KB];
#pragma unroll
                for (int j = 0; j < KB; ++j) theirs[j] = shfl_xor_u64(comp[e][j], off);
                merge_topk<KB>(comp[e], theirs);
            }
        }
    }

    // ---------------------------------------------------------------- where finished lists go
    u64 *cand = (u64 *)(smem + p.lds_cand_off);
    auto emit = [&](int col, const u64(&list)[KB]) { emit_list<ELT, KB>(p, r, sp, col, list, cand); };

    // ---------------------------------------------------------------- merge across wavefronts (LDS, one barrier)
    if (p.nparts > 1) {
        // columns are numbered from the first one of this workgroup's column block
        u64 *xch = (u64 *)(smem + p.lds_xch_off);  // [part][column][slot]
        const int lane = tid & (kWave - 1);
        const int part = p.wave_merge ? (tid >> 6) : ph;
        const bool holder = active && (!p.wave_merge || lane < p.Gw);
        const int colbase = cb * p.Gw * V;
        const int wcols = min(p.Gw * V, p.b - colbase);
        const int64_t pstride = (int64_t)p.Gw * V;  // columns per part
        if (holder) {
#pragma unroll
            for (int e = 0; e < V; ++e)
#pragma unroll
                for (int j = 0; j < KB; ++j) xch[((int64_t)part * pstride + cgl * V + e) * KB + j] = comp[e][j];
        }
        __syncthreads();
        for (int c = tid; c < wcols; c += T) {
            u64 acc[KB];
#pragma unroll
            for (int j = 0; j < KB; ++j) acc[j] = xch[(int64_t)c * KB + j];
            for (int q = 1; q < p.nparts; ++q) {
                u64 theirs[KB];
#pragma unroll
                for (int j = 0; j < KB; ++j) theirs[j] = xch[((int64_t)q * pstride + c) * KB + j];
                merge_topk<KB>(acc, theirs);
            }
            emit(bucket_of(colbase + c), acc);
        }
    } else if (active && (!p.wave_merge || (tid & (kWave - 1)) < p.Gw)) {
#pragma unroll
        for (int e = 0; e < V; ++e) emit(bucket_of(col0 + e), comp[e]);
    }

    trace_mark<TR>(p.trace, 2);  // this workgroup's lists are merged and handed on
    const bool whole = p.stage2 != 0;
    row_tail<ELT, KB, TR>(p, r, whole ? (int64_t)r : (int64_t)r * p.colblocks + cb, whole ? 0 : cb * p.Gw * V,
                          whole ? p.b : min(p.b, (cb + 1) * p.Gw * V), whole ? 0 : rot, smem);
    trace_mark<TR>(p.trace, 9);  // done
    }
}

// ------------------------------------------------------------------------------------------------
// Contiguous assignment (Appendix A.1): bucket j is the run of elements i with floor(b*i/n) = j,
// that is [ceil(j*n/b), ceil((j+1)*n/b)).  Gs lanes side by side share a bucket: lane q reads the
// V-element chunks q, q+Gs, q+2Gs, ... of the run (consecutive lanes, consecutive addresses) into
// one queue, and the Gs queues are merged by a butterfly of shuffles (and, when a bucket takes
// more than one wavefront, once through LDS).  Long buckets of small batches are also split
// over S workgroups.  From the finished per-bucket lists on, everything is shared with the
// interleaved kernel (emit_list, row_tail).
// V > 1 is used only when every bucket has the same length L = n/b, V divides L and the rows
// are aligned; otherwise V = 1 and the runs may differ in length by one.
template <int ELT, int V, int KB, int U, int MAXT>
__global__ void __launch_bounds__(MAXT) contig_kernel(S1Params p) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int ES = (ELT == ATK_F32) ? 4 : 2;
    const int tid = threadIdx.x, T = blockDim.x;
    int wg = blockIdx.x, bb, sp, r;
    divmod(wg, p.bblocks, -1, wg, bb);
    divmod(wg, p.S, p.s_shift, r, sp);
    const int g = tid >> p.gs_shift, q = tid & (p.Gs - 1);
    const int bpw = T >> p.gs_shift;  // buckets the workgroup works on at a time

    // ---- short buckets: a bucket is one load per lane of its group; the group takes NB buckets in turn
    if (p.NB > 0) {
        const int first = bb * bpw * p.NB;  // first bucket of this workgroup
        u64 *cand = (u64 *)(smem + p.lds_cand_off);
        for (int i0 = 0; i0 < p.NB; i0 += U) {
            RowVec<ELT, V> v[U];
            int bj[U];
            int64_t r0[U];
            bool has[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int jj = first + (i0 + u) * bpw + g;
                const bool ok = (i0 + u < p.NB) && jj < p.b;
                int64_t a0 = 0, a1 = 0;
                if (ok) {
                    if (p.rem == 0) {
                        a0 = (int64_t)jj * p.L;
                        a1 = a0 + p.L;
                    } else {
                        a0 = ((int64_t)jj * p.n + p.b - 1) / p.b;
                        a1 = ((int64_t)(jj + 1) * p.n + p.b - 1) / p.b;
                    }
                }
                bj[u] = ok ? jj : -1;
                r0[u] = a0;
                has[u] = ok && (int64_t)q * V < a1 - a0;
            }
            // all loads of the batch are issued together; a lane without an element of its own re-reads the
            // start of the row and drops it (a load under a condition would wait for the one before it)
#pragma unroll
            for (int u = 0; u < U; ++u)
                v[u] = load_vec<ELT, V>((const unsigned char *)p.x +
                                        ((int64_t)r * p.n + (has[u] ? r0[u] + (int64_t)q * V : 0)) * ES);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float val[KB];
                int tt[KB];
#pragma unroll
                for (int i = 0; i < KB; ++i) {
                    val[i] = __uint_as_float(0x7fc00000u);
                    tt[i] = kEmptyT;
                }
                if (has[u]) {
#pragma unroll
                    for (int e = 0; e < V; ++e) insert<KB>(val, tt, __uint_as_float(elem_bits<ELT, V>(v[u], e)), q * V + e);
                }
                u64 comp[KB];
#pragma unroll
                for (int i = 0; i < KB; ++i)
                    comp[i] = (tt[i] != kEmptyT) ? make_composite(__float_as_uint(val[i]), (int32_t)(r0[u] + tt[i])) : 0ull;
                if (KB == 1) {
                    // one slot: the merge is a maximum over the group's lanes; inside a row of 16 lanes
                    // it goes through DPP (register to register), only groups of 32 and 64 lanes need
                    // a cross-row exchange on top
                    u64 v = comp[0], t;
                    if (p.Gs >= 2) { t = dpp_u64<0xB1>(v); v = t > v ? t : v; }
                    if (p.Gs >= 4) { t = dpp_u64<0x4E>(v); v = t > v ? t : v; }
                    if (p.Gs >= 8) { t = dpp_u64<0x141>(v); v = t > v ? t : v; }
                    if (p.Gs >= 16) { t = dpp_u64<0x140>(v); v = t > v ? t : v; }
                    if (p.Gs >= 32) { t = shfl_xor_u64(v, 16); v = t > v ? t : v; }
                    if (p.Gs >= 64) { t = shfl_xor_u64(v, 32); v = t > v ? t : v; }
                    comp[0] = v;
                } else {
                    for (int off = 1; off < p.Gs; off <<= 1) {
                        u64 theirs[KB];
#pragma unroll
                        for (int i = 0; i < KB; ++i) theirs[i] = shfl_xor_u64(comp[i], off);
                        merge_topk<KB>(comp, theirs);
                    }
                }
                if (q == 0 && bj[u] >= 0) emit_list<ELT, KB>(p, r, 0, bj[u], comp, cand);
            }
        }
        row_tail<ELT, KB>(p, r, (int64_t)r, 0, p.b, 0, smem);  // no row splits here: a ticket only with Stage 2
        return;
    }

    const int j = bb * bpw + g;       // this lane's bucket
    const bool active = j < p.b;

    float val[KB];
    int tt[KB];
#pragma unroll
    for (int i = 0; i < KB; ++i) {
        val[i] = __uint_as_float(0x7fc00000u);
        tt[i] = kEmptyT;
    }
    // the run of bucket j, in elements of the row
    int64_t run0 = 0, run1 = 0;
    if (active) {
        run0 = ((int64_t)j * p.n + p.b - 1) / p.b;
        run1 = ((int64_t)(j + 1) * p.n + p.b - 1) / p.b;
    }
    if (active) {
        const int chunks = (int)((run1 - run0) / V);
        const int c0 = sp * p.chunks_per_split;
        const int c_end = min(chunks - c0, p.chunks_per_split) + c0;
        const int c1 = min(c_end, kRowsAhead);  // (where the scan stops that looks ahead)
        const unsigned char *base = (const unsigned char *)p.x + ((int64_t)r * p.n + run0) * ES;
        auto feed = [&](const RowVec<ELT, V> &v, int c) {
            float x[V];
#pragma unroll
            for (int e = 0; e < V; ++e) x[e] = __uint_as_float(elem_bits<ELT, V>(v, e));
            if (KB > 1) {
                bool any = false;
#pragma unroll
                for (int e = 0; e < V; ++e) any = any || !(x[e] <= val[KB - 1]);
                if (__ballot(any) == 0ull) return;
            }
#pragma unroll
            for (int e = 0; e < V; ++e) insert<KB>(val, tt, x[e], c * V + e);
        };
        int c = c0 + q;
        for (; c + (U - 1) * p.Gs < c1; c += U * p.Gs) {
            RowVec<ELT, V> v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = load_vec<ELT, V>(base + (int64_t)(c + u * p.Gs) * (V * ES));
#pragma unroll
            for (int u = 0; u < U; ++u) feed(v[u], c + u * p.Gs);
        }
        if (c < c1) {  // fewer than U loads left: in pieces of U/2 ... 1, each piece's loads issued together
            const int nr = (c1 - c + p.Gs - 1) >> p.gs_shift;
#define ATK_PIECE(NP)                                                                                                  \
    if (NP < U && (nr & NP)) {                                                                                         \
        RowVec<ELT, V> v[NP];                                                                                          \
        _Pragma("unroll") for (int u = 0; u < NP; ++u) v[u] = load_vec<ELT, V>(base + (int64_t)(c + u * p.Gs) * (V * ES)); \
        _Pragma("unroll") for (int u = 0; u < NP; ++u) feed(v[u], c + u * p.Gs);                                       \
        c += NP * p.Gs;                                                                                                \
    }
            ATK_PIECE(8)
            ATK_PIECE(4)
            ATK_PIECE(2)
            ATK_PIECE(1)
#undef ATK_PIECE
        }
        if (c1 < c_end)
            for (uint32_t cr = (uint32_t)(c0 + q) + (uint32_t)((c1 - c0 - q + p.Gs - 1) >> p.gs_shift) * (uint32_t)p.Gs; cr < (uint32_t)c_end; cr += (uint32_t)p.Gs)
                feed(load_vec<ELT, V>(base + (int64_t)cr * (V * ES)), (int)cr);
    }
    u64 comp[KB];
#pragma unroll
    for (int i = 0; i < KB; ++i)
        comp[i] = (tt[i] != kEmptyT) ? make_composite(__float_as_uint(val[i]), (int32_t)(run0 + tt[i])) : 0ull;

    // ---- merge the Gs queues of a bucket: butterfly inside the wavefront ...
    const int span = p.Gs < kWave ? p.Gs : kWave;
    for (int off = 1; off < span; off <<= 1) {
        u64 theirs[KB];
#pragma unroll
        for (int i = 0; i < KB; ++i) theirs[i] = shfl_xor_u64(comp[i], off);
        merge_topk<KB>(comp, theirs);
    }
    // ... and across the wavefronts of the workgroup when the bucket owns all of it
    if (p.Gs > kWave) {
        u64 *xch = (u64 *)(smem + p.lds_xch_off);  // [wavefront][slot]
        const int lane = tid & (kWave - 1), wave = tid >> 6, n_waves = T >> 6;
        if (lane == 0) {
#pragma unroll
            for (int i = 0; i < KB; ++i) xch[wave * KB + i] = comp[i];
        }
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int i = 0; i < KB; ++i) comp[i] = (lane < n_waves) ? xch[lane * KB + i] : 0ull;
            for (int off = 1; off < n_waves; off <<= 1) {
                u64 theirs[KB];
#pragma unroll
                for (int i = 0; i < KB; ++i) theirs[i] = shfl_xor_u64(comp[i], off);
                merge_topk<KB>(comp, theirs);
            }
        }
    }
    u64 *cand = (u64 *)(smem + p.lds_cand_off);
    if (active && q == 0) emit_list<ELT, KB>(p, r, sp, j, comp, cand);
    const bool whole = p.stage2 != 0;
    row_tail<ELT, KB>(p, r, whole ? (int64_t)r : (int64_t)r * p.bblocks + bb, whole ? 0 : bb * bpw,
                      whole ? p.b : min(p.b, (bb + 1) * bpw), 0, smem);
}

// ------------------------------------------------------------------------------------------------
// Matrix rows whose loads a lane with packed queues has in flight, for V columns: 128 bytes' worth of registers at most (with eight slots
// twice that: the next batch is loaded while one is worked on).  The instances' own batches are about unpacked queues and smaller ones left the
// lanes waiting (128 x 65536, k = 16384, b = 1024, k_b = 16: two rows 24.8 us, eight 15.6, sixteen 14.2; 128 x 2^20, b = 64, k_b = 16: 247, 173, 157).
constexpr int packed_batch(int V) { return V == 8 ? 4 : 16; }

template <int ELT, int V, int KB, int U>
static hipError_t launch_one(const Plan &pl, const S1Params &params, hipStream_t stream) {
    constexpr int MAXT = max_threads_for_kb(KB);
    if (pl.T > MAXT) return hipErrorInvalidValue;
    S1Params prm = params;
    size_t lds = (size_t)pl.lds_bytes;
    constexpr size_t kStage = V * KB * 4;  // bytes of a lane's indices
    // (32 bytes and less from a lane: 0.97 to 1.02 times as long through LDS)
    if (pl.direct && params.vec_store && pl.k_b == KB && kStage >= 64 && pl.T * kStage <= 64 * 1024) {
        prm.staged = 1;
        lds = std::max(lds, pl.T * kStage);
    }
    if constexpr (ELT == ATK_BF16 && KB >= 2) {
        if (pl.packed) {
            // (packed queues leave registers for more loads in flight than the instance's U, which is about the unpacked ones)
            constexpr int UP = packed_batch(V);
            hipLaunchKernelGGL((stage1_kernel<ELT, V, KB, UP, MAXT, true>), dim3((unsigned)pl.grid),
                               dim3((unsigned)pl.T), lds, stream, prm);
            return hipGetLastError();
        }
    }
    if (prm.trace) return hipErrorNotSupported;  // the measurement build exists for the lean kernels only
    if constexpr (KB == 8) {
        if (pl.refresh) {
            constexpr int UF = KB;  // matrix rows in flight, and sorted at a time
            hipLaunchKernelGGL((stage1_kernel<ELT, V, KB, UF, MAXT, false, false, true>), dim3((unsigned)pl.grid),
                               dim3((unsigned)pl.T), lds, stream, prm);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((stage1_kernel<ELT, V, KB, U, MAXT, false>), dim3((unsigned)pl.grid), dim3((unsigned)pl.T), lds, stream, prm);
    return hipGetLastError();
}

static int log2_exact(int v) {
    if (v < 1 || (v & (v - 1))) return -1;
    int s = 0;
    while ((1 << s) < v) ++s;
    return s;
}

hipError_t launch_approx(const Plan &pl, const void *x, void *out_vals, int32_t *out_idx, void *state, void *data,
                         hipStream_t stream, void *trace) {
    S1Params prm;
    memset(&prm, 0, sizeof prm);
    prm.trace = (u64 *)trace;
    prm.x = x;
    prm.out_vals = out_vals;
    prm.out_idx = out_idx;
    prm.tickets = (uint32_t *)state;
    prm.lists = (u64 *)data;
    prm.n = pl.n;
    prm.b = (int)pl.b;
    prm.L = (int)pl.L;
    prm.G = (int)pl.G;
    prm.Gw = pl.Gw;
    prm.P = pl.P;
    prm.colblocks = pl.colblocks;
    prm.S = pl.S;
    prm.rows_per_split = pl.rows_per_split;
    prm.rem = (int)(pl.n % pl.b);
    prm.extra_ph = (int)(pl.L % pl.P);
    prm.idx_bits = 1;
    while (((int64_t)1 << prm.idx_bits) < pl.n) ++prm.idx_bits;
    prm.k = (int)pl.k;
    prm.k_b = pl.k_b;
    prm.stage2 = pl.stage2;
    prm.direct = pl.direct;
    prm.use_scratch = pl.use_scratch;
    prm.wave_merge = pl.wave_merge;
    prm.nparts = pl.nparts;
    prm.lds_xch_off = pl.lds_xch_off;
    prm.lds_cand_off = pl.lds_cand_off;
    prm.lds_max = pl.lds_max;
    prm.bound_ok = pl.bound_ok;
    prm.refresh = pl.refresh;
    prm.wgs_per_ticket = pl.stage2 ? pl.S * pl.colblocks : pl.S;
    prm.tail_tpc_shift = log2_exact(pl.tail_tpc);
    prm.cb_shift = log2_exact(pl.colblocks);
    prm.s_shift = log2_exact(pl.S);
    prm.gw_shift = log2_exact(pl.Gw);
    const uintptr_t ov = (uintptr_t)out_vals, oi = (uintptr_t)out_idx;
    prm.vec_store = ((ov | oi) & 15u) == 0;
#define ATK_CASE(ELT, VV, KK, UU) \
    if (pl.dtype == ELT && pl.V == VV && pl.KB == KK) return launch_one<ELT, VV, KK, UU>(pl, prm, stream);
    ATK_STAGE1_INSTANCES(ATK_CASE)
#undef ATK_CASE
    return hipErrorInvalidValue;
}

template <int ELT, int V, int KB, int U>
static hipError_t launch_contig_one(const Plan &pl, const S1Params &prm, hipStream_t stream) {
    constexpr int MAXT = max_threads_for_kb(KB);
    if (pl.T > MAXT) return hipErrorInvalidValue;
    hipLaunchKernelGGL((contig_kernel<ELT, V, KB, U, MAXT>), dim3((unsigned)pl.grid), dim3((unsigned)pl.T),
                       (size_t)pl.lds_bytes, stream, prm);
    return hipGetLastError();
}

hipError_t launch_approx_contig(const Plan &pl, const void *x, void *out_vals, int32_t *out_idx, void *state,
                                void *data, hipStream_t stream) {
    S1Params prm;
    memset(&prm, 0, sizeof prm);
    prm.x = x;
    prm.out_vals = out_vals;
    prm.out_idx = out_idx;
    prm.tickets = (uint32_t *)state;
    prm.lists = (u64 *)data;
    prm.n = pl.n;
    prm.b = (int)pl.b;
    prm.L = (int)pl.L;
    prm.S = pl.S;
    prm.s_shift = log2_exact(pl.S);
    prm.idx_bits = 1;
    while (((int64_t)1 << prm.idx_bits) < pl.n) ++prm.idx_bits;
    prm.k = (int)pl.k;
    prm.k_b = pl.k_b;
    prm.stage2 = pl.stage2;
    prm.use_scratch = pl.use_scratch;
    prm.lds_xch_off = pl.lds_xch_off;
    prm.lds_cand_off = pl.lds_cand_off;
    prm.wgs_per_ticket = pl.stage2 ? pl.S * pl.bblocks : pl.S;
    prm.tail_tpc_shift = log2_exact(pl.tail_tpc);
    prm.Gs = pl.Gs;
    prm.gs_shift = log2_exact(pl.Gs);
    prm.bblocks = pl.bblocks;
    prm.chunks_per_split = pl.chunks_per_split;
    prm.NB = pl.NB;
    prm.rem = (int)(pl.n % pl.b);
    if (prm.gs_shift < 0) return hipErrorInvalidValue;
#define ATK_CASE(ELT, VV, KK, UU) \
    if (pl.dtype == ELT && pl.V == VV && pl.KB == KK) return launch_contig_one<ELT, VV, KK, UU>(pl, prm, stream);
    ATK_CONTIG_INSTANCES(ATK_CASE)
#undef ATK_CASE
    return hipErrorInvalidValue;
}

}  // namespace atk
