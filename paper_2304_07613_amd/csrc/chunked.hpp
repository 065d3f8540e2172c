// chunked.hpp -- shared by the translation units of the paper's chunked layout
// (Section 5): the pattern list and a wave's own LDS ordering.
#pragma once
#include "common.hpp"

namespace {

__host__ __device__ inline int p_binom(int m, int n) {
    int64_t v = 1;
    for (int i = 1; i <= n; ++i) {
        v = v * (m - n + i) / i;
        if (v > 4096) return 4097;
    }
    return (int)v;
}

// Offsets (ascending) of pattern `idx` of the revolving-door list of the
// n-subsets of {0 .. m-1}: the list of (m, n) is the list of (m-1, n)
// followed by the list of (m-1, n-1) reversed, each with m-1 added; (m, m)
// holds the single full set.  Unranked from the top: every binomial on the way
// is at most C(m, n).
__host__ __device__ inline void p_unrank(int m, int n, int idx, uint8_t *out) {
    while (n > 0) {
        if (n == m) {
            for (int i = 0; i < n; ++i) out[i] = (uint8_t)i;
            return;
        }
        const int first = p_binom(m - 1, n);
        if (idx >= first) {  // in the second half: m-1 is in the pattern
            idx = p_binom(m - 1, n - 1) - 1 - (idx - first);
            out[n - 1] = (uint8_t)(m - 1);
            --n;
        }
        --m;
    }
}

// Division of e < 2^16 by 1 <= d < 2^16 through a multiply-high: with
// mul = ceil(2^32 / d), floor(e mul / 2^32) = floor(e / d) since e d < 2^32.
__device__ __forceinline__ uint32_t magic_u16(uint32_t d) {
    return d > 1 ? (uint32_t)(0xffffffffu / d + 1u) : 0u;
}
__device__ __forceinline__ uint32_t div_u16(uint32_t e, uint32_t mul, uint32_t d) {
    return d > 1 ? __umulhi(e, mul) : e;
}

__device__ __forceinline__ void p_wave_sync() {
    // this wave's LDS writes are done before its later LDS reads
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace
