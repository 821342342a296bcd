// The random draw of one sampled row (Philox4x32-10 and the partial Fisher-Yates shuffle of its edge positions), shared by
// the sampler's hop kernel and the pre-sampling kernel.
#pragma once
#include "common.hpp"

namespace no {

__device__ __forceinline__ uint64_t philox_random64(uint32_t k0, uint32_t k1, uint32_t c0, uint32_t c1, uint32_t c2,
                                                    uint32_t c3) {
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;      // (one instruction each)
        const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0, n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
        c0 = n0; c1 = (uint32_t)p1; c2 = n2; c3 = (uint32_t)p0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return ((uint64_t)c1 << 32) | (uint64_t)c0;
}

// The value that lane t of every group of G lanes holds, in all lanes of the group (t the same in the whole wavefront and
// known when the caller's loop is unrolled). Groups of up to 16 lanes lie within a row of the DPP network and need no LDS round trip (a
// shuffle through LDS takes some 60 cycles, and a draw has a chain of 2 k of them).
template <int G, int T>
__device__ __forceinline__ uint32_t group_lane(uint32_t v) {
    static_assert(G == 8 || G == 16 || G == 32 || G == 64, "group width");
    if (G == 16) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x150 + (T & 15), 0xf, 0xf, true);        // row_newbcast
    if (G == 8) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x150 + (T & 7), 0xf, 0xf, true);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x158 + (T & 7), 0xf, 0xf, true);
        return (threadIdx.x & 8) ? hi : lo;
    }
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)v, T);
    if (G == 64) return lo;
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)v, 32 + (T & 31));
    return (threadIdx.x & 32) ? hi : lo;
}

// The swap partner of slot j: j + floor(x (d - j) / 2^64) in [j, d), for a row of d < 2^32 entries.
__device__ __forceinline__ uint32_t swap_partner(uint64_t x, uint32_t d, uint32_t j) {
    const uint32_t left = d - j;
    const uint64_t low = (uint64_t)(uint32_t)x * left;
    return j + (uint32_t)(((uint64_t)(uint32_t)(x >> 32) * left + (low >> 32)) >> 32);
}

// One step of the shuffle as slot j sees it: step T swapped position r_T with position T. `put` is what stands in position j
// (what step j will move to its partner), `pos` what stands in the partner's; both are final once the steps before j are done,
// so step T may hand out its own.
template <int G, int T>
__device__ __forceinline__ void draw_steps(int32_t k, uint32_t j, uint32_t r, uint32_t& put, uint32_t& pos) {
    if constexpr (T < G) {
        if (T + 1 >= k) return;
        const uint32_t rt = group_lane<G, T>(r), pt = group_lane<G, T>(put);
        if ((uint32_t)T < j) {
            if (rt == j) put = pt;
            if (rt == r) pos = pt;
        }
        draw_steps<G, T + 1>(k, j, r, put, pos);
    }
}

// Position, inside the d entries of vertex v's row, of slot j of a draw of min(d, k) of them: the whole row in stored
// order when d <= k, else slot j of the shuffle. A group of G lanes (G >= k, lane j = slot j) serves one row; every lane of
// the wavefront calls this together (row_ok = false for lanes without a row), and only lanes with j < min(d, k) use the result.
// d < 2^32: a graph has no more edges.
template <int G>
__device__ __forceinline__ uint32_t draw_position(bool row_ok, int32_t v, uint32_t d, int32_t k, int32_t j, uint32_t key0,
                                                  uint32_t key1, uint32_t c3) {
    const bool shuffle = row_ok && d > (uint32_t)k;
    if (__ballot(shuffle) == 0ull) return (uint32_t)j;
    uint32_t r = 0;
    if (shuffle && j < k) r = swap_partner(philox_random64(key0, key1, (uint32_t)v, 0u, (uint32_t)j, c3), d, (uint32_t)j);
    uint32_t put = (uint32_t)j, pos = r;
    draw_steps<G, 0>(k, (uint32_t)j, r, put, pos);
    return shuffle ? pos : (uint32_t)j;
}

// All slots of a row by one thread (k <= K): positions of a draw of k of the row's d > k entries. The steps in order: step j
// finds in its own position, and in its partner's, what the latest step that had that position for a partner put there. (That is always
// one of the first k positions: a byte.)
template <int K>
__device__ __forceinline__ void draw_row(int32_t v, uint32_t d, int32_t k, uint32_t key0, uint32_t key1, uint32_t c3, uint32_t (&pos)[K]) {
    uint32_t r[K], put[K / 4];
#pragma unroll
    for (int j = 0; j < K; ++j) {
        if (j < k) {
            r[j] = swap_partner(philox_random64(key0, key1, (uint32_t)v, 0u, (uint32_t)j, c3), d, (uint32_t)j);
            uint32_t mine = (uint32_t)j, p = r[j];
#pragma unroll
            for (int t = 0; t < j; ++t) {
                const uint32_t pt = (put[t / 4] >> (8 * (t & 3))) & 0xffu;
                mine = r[t] == (uint32_t)j ? pt : mine;
                p = r[t] == r[j] ? pt : p;
            }
            pos[j] = p;
            put[j / 4] = (j & 3) == 0 ? mine : put[j / 4] | mine << (8 * (j & 3));
        }
    }
}

}  // namespace no
