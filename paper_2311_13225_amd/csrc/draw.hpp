// The random draw of one sampled row (Philox4x32-10 and the partial Fisher-Yates shuffle of its edge positions), shared by
// the sampler's hop kernel and the pre-sampling kernel.
#pragma once
#include "common.hpp"

namespace no {

__device__ __forceinline__ uint64_t philox_random64(uint32_t k0, uint32_t k1, uint32_t c0, uint32_t c1, uint32_t c2,
                                                    uint32_t c3) {
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
        uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
        uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return ((uint64_t)c1 << 32) | (uint64_t)c0;
}

// Position, inside the d entries of vertex v's row, of slot j of a draw of min(d, k) of them: the whole row in stored
// order when d <= k, else slot j of the shuffle. A group of G lanes (G >= k, lane j = slot j) serves one row; every lane of
// the wavefront calls this together (row_ok = false for lanes without a row), and only lanes with j < min(d, k) use the result.
template <int G>
__device__ __forceinline__ int64_t draw_position(bool row_ok, int32_t v, int64_t d, int32_t k, int32_t j, uint32_t key0,
                                                 uint32_t key1, uint32_t c3) {
    int64_t pos = j;
    const bool take_all = d <= (int64_t)k;
    // The swap partner of slot j: r_j = j + floor(x * (d - j) / 2^64) in [j, d).
    int64_t r = -1 - (int64_t)j;          // distinct negative sentinels for idle lanes
    if (row_ok && !take_all && j < k) {
        uint64_t x = philox_random64(key0, key1, (uint32_t)v, 0u, (uint32_t)j, c3);
        r = (int64_t)j + (int64_t)__umul64hi(x, (uint64_t)(d - j));
    }
    // Whole groups with nothing to shuffle still take part in the cross-lane reads below.
    if (__ballot(row_ok && !take_all) != 0ull) {
        // a = latest earlier step that displaced position j; b = latest earlier step that hit r_j
        int32_t a = -1, b = -1;
        for (int32_t t = 0; t < k; ++t) {
            int64_t rt = __shfl(r, t, G);
            if (t < j) {
                if (rt == (int64_t)j) a = t;
                if (rt == r) b = t;
            }
        }
        // w_j = content of position j just before step j: j itself unless displaced, else w_a.
        int64_t w = j;
        bool done = a < 0;
        while (true) {
            int64_t wa = __shfl(w, a < 0 ? 0 : a, G);
            int da = __shfl((int)done, a < 0 ? 0 : a, G);
            if (!done && da) { w = wa; done = true; }
            if (__ballot(!done) == 0ull) break;
        }
        int64_t wb = __shfl(w, b < 0 ? 0 : b, G);
        if (!take_all) pos = b < 0 ? r : wb;
    }
    return pos;
}

}  // namespace no
