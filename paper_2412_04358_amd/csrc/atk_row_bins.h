// The bins of exact_topk's row kernels: a header without device code of its own, so that host tests can compile it.
#pragma once

#include <stdint.h>

#include "../../include/approx_topk.h"

#ifdef __HIPCC__
#define ATK_HD __host__ __device__ __forceinline__
#else
#define ATK_HD inline
#endif

namespace atk {

// Bins linear in the order key (ties: in the index) between two keys.  d grows with the composite: the value key relative
// to the lower end without the low bits that bf16 leaves constant, then as many index bits as 32 bits have room for.
struct RowBins {
    uint32_t k_min, span, scale;
    int n_bins, s_idx, r_idx;
    uint32_t i_mask;
    float inv_scale;
    template <int ELT>
    ATK_HD void set(uint32_t lo, uint32_t hi, int idx_bits, int bins) {
        constexpr int tz = (ELT == ATK_BF16) ? 16 : 0;
        k_min = lo;
        n_bins = bins;
        span = (hi - lo) >> tz;
        const int span_bits = span ? 32 - __builtin_clz(span) : 0;
        s_idx = 32 - span_bits < idx_bits ? 32 - span_bits : idx_bits;
        r_idx = idx_bits - s_idx;
        i_mask = idx_bits >= 31 ? 0x7fffffffu : ((1u << idx_bits) - 1u);
        const uint32_t d_max = (uint32_t)((((unsigned long long)span + 1ull) << s_idx) - 1ull);  // < 2^32: span < 2^span_bits, s_idx <= 32 - span_bits
        const float d1 = (float)d_max + 1.0f;
        // a little under bins * 2^32 / (d_max + 1): the conversion's rounding must not push the largest d past the last bin
        const float s = ((float)bins * 4294967296.0f / d1) * 0.999999f;
        scale = s >= 4294967040.0f ? 0xffffffffu : (uint32_t)s;
        inv_scale = 4294967296.0f / (float)scale;
    }
    // key >= k_min; inv_idx: 0x7fffffff - index.  ABOVE: keys past the upper end (which is a sample's largest, say) lie in the
    // last bin whatever their index: no bin of a composite is above that of a larger one.  Without it there must be none (where the
    // bins of a row's every element are worked out in unrolled code, an instruction more is 3 % of the call).
    template <int ELT, bool ABOVE = false>
    ATK_HD uint32_t bin(uint32_t key, uint32_t inv_idx) const {
        constexpr int tz = (ELT == ATK_BF16) ? 16 : 0;
        const uint32_t off = (key - k_min) >> tz;
        uint32_t d = s_idx >= 32 ? 0u : (off << s_idx);
        d |= (inv_idx & i_mask) >> r_idx;
        if (ABOVE) d = off > span ? 0xffffffffu : d;
        const uint32_t b = (uint32_t)(((unsigned long long)d * scale) >> 32);
        return b < (uint32_t)n_bins ? b : (uint32_t)n_bins - 1u;
    }
    // a key at or a little below the lowest of bin b
    template <int ELT>
    ATK_HD uint32_t edge(uint32_t b) const {
        constexpr int tz = (ELT == ATK_BF16) ? 16 : 0;
        float d = (float)b * inv_scale;
        d = d - d * 4.0e-7f - 2.0f;
        if (!(d > 0.0f)) return k_min;
        const uint32_t di = d >= 4294967040.0f ? 0xffffff00u : (uint32_t)d;
        return k_min + ((s_idx >= 32 ? 0u : (di >> s_idx)) << tz);
    }
};

}  // namespace atk
