// Stable LSD radix sort of (key, value) pairs of 32-bit words, digit by digit (up to 9 bits each).
//
// A pass is three launches over tiles of 8192 pairs. rs_hist: a block walks a chunk of consecutive tiles and writes, per tile
// and digit, the chunk's count so far, and at the end the chunk's totals (at most 512 chunks). rs_chunks: prefix of the
// totals over the chunks, per digit, and the digits' totals. rs_scatter: a tile ranks its pairs (wavefront matches by
// ballot, stable), puts them in digit order in LDS and stores runs of equal digits contiguously.
// Bound by memory: a pass has to read and write 8 bytes a pair and reads the keys once more for the counts. Stored straight
// from the registers (no order in LDS, 16-pair runs at 4096-pair tiles) a pass took 3.4-4.2 ms on 124 M pairs; like this
// 0.40-0.46 ms for the scatter (4.3 to 4.9 TB/s; a large copy reaches 4.78) and 0.13 ms for the counts. With the tiles dealt
// to the dies in turn the scatter took 0.75 ms. Digits of 11 bits, four values a thread, would save one pass in five, but
// leave 4-pair runs: 0.81 ms (0.87 with tiles of 16384 pairs and 1024 threads), so 9 bits are the most.
#pragma once
#include "primitives.hpp"

namespace no {

constexpr int RS_THREADS = 512, RS_WAVES = RS_THREADS / 64, RS_ITEMS = 16, RS_TILE = RS_THREADS * RS_ITEMS;
constexpr int RS_MAX_BITS = 9, RS_RADIX = 1 << RS_MAX_BITS;        // one digit value per thread
constexpr int64_t RS_MAX_CHUNKS = 512;
static_assert(RS_RADIX == RS_THREADS, "one digit value per thread");

// One digit of a pass: bits [shift, shift + bits) of the key, or, with up > 0, of the 64-bit number whose low `up + shift`
// bits are the key and whose upper ones are the value.
struct Digit {
    int shift, bits, up;
    __device__ __forceinline__ uint32_t of(uint32_t key) const { return (key >> shift) & ((1u << bits) - 1u); }
    __device__ __forceinline__ uint32_t of(uint32_t key, uint32_t val) const { return ((key >> shift) | (val << up)) & ((1u << bits) - 1u); }
};

struct RadixPlan {      // how n pairs are cut up; the scratch of one pass (any number of passes may share it)
    int64_t n, n_tiles, tiles_per_chunk, n_chunks;
    explicit RadixPlan(int64_t n_) : n(n_) {
        n_tiles = ceil_div(n, RS_TILE);
        if (n_tiles < 1) n_tiles = 1;
        tiles_per_chunk = ceil_div(n_tiles, RS_MAX_CHUNKS);
        n_chunks = ceil_div(n_tiles, tiles_per_chunk);
    }
    size_t ws_words() const { return (size_t)(n_tiles + n_chunks + 1) * RS_RADIX; }
    uint32_t* tile_excl(void* ws) const { return (uint32_t*)ws; }                                     // [n_tiles][RS_RADIX]
    uint32_t* chunk(void* ws) const { return (uint32_t*)ws + n_tiles * RS_RADIX; }                    // [n_chunks][RS_RADIX]
    uint32_t* totals(void* ws) const { return (uint32_t*)ws + (n_tiles + n_chunks) * RS_RADIX; }      // [RS_RADIX]
};

// k[0 .. here) = a[i .. i + here), in 16-byte loads where a whole, aligned run is there.
template <typename T>
__device__ __forceinline__ void load_run(const T* a, int64_t i, int here, T (&k)[RS_ITEMS]) {
    constexpr int PER = 16 / sizeof(T);
    typedef T vec __attribute__((ext_vector_type(PER)));
    if (here == RS_ITEMS && ((uintptr_t)(a + i) & 15) == 0) {
#pragma unroll
        for (int q = 0; q < RS_ITEMS / PER; ++q) {
            const vec v = *reinterpret_cast<const vec*>(a + i + q * PER);
#pragma unroll
            for (int e = 0; e < PER; ++e) k[q * PER + e] = v[e];
        }
    } else {
#pragma unroll
        for (int it = 0; it < RS_ITEMS; ++it) k[it] = it < here ? a[i + it] : (T)0;
    }
}

// Where a pass's pairs come from: two arrays of words.
struct PairArrays {
    const uint32_t* keys; const uint32_t* vals;
    __device__ __forceinline__ uint32_t key(int64_t i) const { return keys[i]; }
    __device__ __forceinline__ void keys_checked(int64_t i, int here, uint32_t (&k)[RS_ITEMS]) const { load_run(keys, i, here, k); }
    __device__ __forceinline__ uint32_t val(int64_t i) const { return vals[i]; }
};

template <typename Source, bool BOTH>
__global__ void __launch_bounds__(RS_THREADS) rs_hist_kernel(Source in, int64_t n, int64_t n_tiles, int64_t tiles_per_chunk, Digit digit,
                                                             uint32_t* __restrict__ tile_excl, uint32_t* __restrict__ chunk) {
    __shared__ uint32_t cnt[RS_RADIX];
    cnt[threadIdx.x] = 0;
    __syncthreads();
    const int64_t t0 = (int64_t)blockIdx.x * tiles_per_chunk, t1 = min(n_tiles, t0 + tiles_per_chunk);
    for (int64_t t = t0; t < t1; ++t) {
        // A thread takes consecutive pairs and adds a run of equal digits at once: after the first passes equal keys stand
        // together, and 64 lanes that add to one counter queue up (a popular vertex: 340 us instead of 140 for such a pass).
        uint32_t k[RS_ITEMS];
        const int64_t first = t * RS_TILE + (int64_t)threadIdx.x * RS_ITEMS;
        const int here = (int)max((int64_t)0, min((int64_t)RS_ITEMS, n - first));
        in.keys_checked(first, here, k);
        if constexpr (BOTH) {
            uint32_t v[RS_ITEMS];
            load_run(in.vals, first, here, v);
#pragma unroll
            for (int it = 0; it < RS_ITEMS; ++it) k[it] = digit.of(k[it], v[it]);
        } else {
#pragma unroll
            for (int it = 0; it < RS_ITEMS; ++it) k[it] = digit.of(k[it]);
        }
        tile_excl[t * RS_RADIX + threadIdx.x] = cnt[threadIdx.x];
        __syncthreads();                   // (the tile's counts come on top only after they were read)
        if (here > 0) {
            uint32_t d = k[0], run = 1;
#pragma unroll
            for (int it = 1; it < RS_ITEMS; ++it) {
                const uint32_t e = k[it];
                if (it < here && e == d) { ++run; continue; }
                if (it < here) {
                    atomicAdd(&cnt[d], run);
                    d = e;
                    run = 1;
                }
            }
            atomicAdd(&cnt[d], run);
        }
        __syncthreads();
    }
    chunk[(int64_t)blockIdx.x * RS_RADIX + threadIdx.x] = cnt[threadIdx.x];
}

// chunk[c][d] becomes the sum of chunk[0 .. c)[d]; totals[d] their sum. A block owns 64 digits; its eight wavefronts own
// consecutive ranges of chunks.
__global__ void __launch_bounds__(RS_THREADS) rs_chunks_kernel(uint32_t* chunk, int64_t n_chunks, uint32_t* totals);

template <typename Source, bool BOTH>
__global__ void __launch_bounds__(RS_THREADS) rs_scatter_kernel(Source in, int64_t n, int64_t n_tiles, int64_t tiles_per_chunk, Digit digit,
                                                                const uint32_t* __restrict__ tile_excl, const uint32_t* __restrict__ chunk,
                                                                const uint32_t* __restrict__ totals, uint32_t* __restrict__ keys_out,
                                                                uint32_t* __restrict__ vals_out) {
    // counts, per wavefront: of a digit, then the local position of its first pair; once every pair knows its place, the pairs
    __shared__ uint32_t buf[RS_TILE];
    __shared__ uint32_t gbase[RS_RADIX];              // global minus local position of a digit's run
    __shared__ uint32_t smem[RS_WAVES + 1];
    uint32_t (*const cnt)[RS_RADIX] = reinterpret_cast<uint32_t (*)[RS_RADIX]>(buf);
    static_assert(RS_WAVES * RS_RADIX <= RS_TILE, "the counts fit where the pairs go");
    const int lane = lane_id(), wave = (int)(threadIdx.x >> 6);
    // a workgroup's die is its id modulo 8: consecutive tiles, whose runs of a digit lie next to each other, go to one die,
    // so that the lines where two runs meet are put together in its L2
    const int64_t per_die = (n_tiles + 7) / 8, tile = blockIdx.x % 8 * per_die + blockIdx.x / 8;
    if (tile >= n_tiles) return;
    const int64_t base = tile * RS_TILE, wave_base = base + (int64_t)wave * (RS_ITEMS * 64) + lane;
    uint32_t key[RS_ITEMS], val[RS_ITEMS];
#pragma unroll
    for (int it = 0; it < RS_ITEMS; ++it) key[it] = wave_base + it * 64 < n ? in.key(wave_base + it * 64) : 0u;
    if constexpr (BOTH)
#pragma unroll
        for (int it = 0; it < RS_ITEMS; ++it) val[it] = wave_base + it * 64 < n ? in.val(wave_base + it * 64) : 0u;
    const uint32_t total = totals[threadIdx.x];
    const uint32_t before = chunk[tile / tiles_per_chunk * RS_RADIX + threadIdx.x] + tile_excl[tile * RS_RADIX + threadIdx.x];
#pragma unroll
    for (int w = 0; w < RS_WAVES; ++w) cnt[w][threadIdx.x] = 0;
    uint32_t all;
    const uint32_t digit_base = block_exclusive_scan<uint32_t, RS_THREADS>(total, &all, smem);
    auto digit_of = [&](int it) { if constexpr (BOTH) return digit.of(key[it], val[it]); else return digit.of(key[it]); };
    volatile uint32_t* my_cnt = cnt[wave];
    uint32_t rank[RS_ITEMS];
#pragma unroll
    for (int it = 0; it < RS_ITEMS; ++it) {
        const bool valid = wave_base + it * 64 < n;
        const uint32_t d = digit_of(it);
        // lanes of the same digit: those that agree in every bit (the bit as a mask of all ones or none)
        const uint64_t here = __ballot(valid);
        uint32_t lo = (uint32_t)here, hi = (uint32_t)(here >> 32);
#pragma unroll
        for (int b = 0; b < RS_MAX_BITS; ++b) {
            const uint32_t bit = (uint32_t)__builtin_amdgcn_sbfe((int32_t)d, b, 1);
            const uint64_t m = __ballot(bit != 0);
            lo &= ~((uint32_t)m ^ bit);
            hi &= ~((uint32_t)(m >> 32) ^ bit);
        }
        const uint32_t ahead = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0)), group = (uint32_t)(__popc(lo) + __popc(hi));
        const uint32_t prev = valid ? my_cnt[d] : 0u;
        rank[it] = prev + ahead;
        __builtin_amdgcn_wave_barrier();
        if (valid && ahead == group - 1) my_cnt[d] = prev + group;   // the last lane of a group publishes
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    {
        uint32_t c[RS_WAVES], sum = 0;
#pragma unroll
        for (int w = 0; w < RS_WAVES; ++w) { c[w] = cnt[w][threadIdx.x]; sum += c[w]; }
        uint32_t run = block_exclusive_scan<uint32_t, RS_THREADS>(sum, &all, smem);
        gbase[threadIdx.x] = digit_base + before - run;
#pragma unroll
        for (int w = 0; w < RS_WAVES; ++w) { cnt[w][threadIdx.x] = run; run += c[w]; }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < RS_ITEMS; ++it) rank[it] += cnt[wave][digit_of(it)];
    __syncthreads();
    const int32_t here = (int32_t)min((int64_t)RS_TILE, n - base);
    if constexpr (!BOTH)          // (not before they are needed: the ranking has the registers)
#pragma unroll
        for (int it = 0; it < RS_ITEMS; ++it) val[it] = wave_base + it * 64 < n ? in.val(wave_base + it * 64) : 0u;
    uint32_t to[RS_ITEMS];
    if constexpr (BOTH) {            // (the digits first: neither word of a pair has the whole of one)
#pragma unroll
        for (int it = 0; it < RS_ITEMS; ++it)
            if (wave_base + it * 64 < n) buf[rank[it]] = digit_of(it);
        __syncthreads();
#pragma unroll
        for (int it = 0; it < RS_ITEMS; ++it) {
            const int32_t i = it * RS_THREADS + (int32_t)threadIdx.x;
            if (i < here) to[it] = gbase[buf[i]] + (uint32_t)i;
        }
        __syncthreads();
    }
#pragma unroll
    for (int it = 0; it < RS_ITEMS; ++it)
        if (wave_base + it * 64 < n) buf[rank[it]] = key[it];
    __syncthreads();
#pragma unroll
    for (int it = 0; it < RS_ITEMS; ++it) {
        const int32_t i = it * RS_THREADS + (int32_t)threadIdx.x;
        if (i < here) {
            const uint32_t k = buf[i];
            if constexpr (!BOTH) to[it] = gbase[digit.of(k)] + (uint32_t)i;
            keys_out[to[it]] = k;
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < RS_ITEMS; ++it)
        if (wave_base + it * 64 < n) buf[rank[it]] = val[it];
    __syncthreads();
#pragma unroll
    for (int it = 0; it < RS_ITEMS; ++it) {
        const int32_t i = it * RS_THREADS + (int32_t)threadIdx.x;
        if (i < here) vals_out[to[it]] = buf[i];
    }
}

template <typename Source, bool BOTH>
void radix_launches(const Source& in, const RadixPlan& plan, Digit digit, uint32_t* keys_out, uint32_t* vals_out, void* ws, hipStream_t st) {
    hipLaunchKernelGGL((rs_hist_kernel<Source, BOTH>), dim3((unsigned)plan.n_chunks), dim3(RS_THREADS), 0, st, in, plan.n, plan.n_tiles,
                       plan.tiles_per_chunk, digit, plan.tile_excl(ws), plan.chunk(ws));
    hipLaunchKernelGGL(rs_chunks_kernel, dim3(RS_RADIX / 64), dim3(RS_THREADS), 0, st, plan.chunk(ws), plan.n_chunks, plan.totals(ws));
    hipLaunchKernelGGL((rs_scatter_kernel<Source, BOTH>), dim3((unsigned)(ceil_div(plan.n_tiles, 8) * 8)), dim3(RS_THREADS), 0, st, in, plan.n,
                       plan.n_tiles, plan.tiles_per_chunk, digit, (const uint32_t*)plan.tile_excl(ws), (const uint32_t*)plan.chunk(ws),
                       (const uint32_t*)plan.totals(ws), keys_out, vals_out);
}

// One pass: pairs of `in` ordered by bits [shift, shift + bits) of their keys. The outputs must not be the input's arrays.
template <typename Source>
int32_t radix_pass(const Source& in, const RadixPlan& plan, int shift, int bits, uint32_t* keys_out, uint32_t* vals_out, void* ws,
                   hipStream_t st) {
    radix_launches<Source, false>(in, plan, Digit{shift, bits, 0}, keys_out, vals_out, ws, st);
    return launch_status("radix_pass");
}

// The same by a digit that begins in the key, of key_bits bits, and ends in the value.
static inline int32_t radix_pass_across(const PairArrays& in, const RadixPlan& plan, int shift, int bits, int key_bits, uint32_t* keys_out,
                                        uint32_t* vals_out, void* ws, hipStream_t st) {
    radix_launches<PairArrays, true>(in, plan, Digit{shift, bits, key_bits - shift}, keys_out, vals_out, ws, st);
    return launch_status("radix_pass_across");
}

// Passes for keys of `bits` bits, and the digit width that spreads the bits evenly over them.
static inline int radix_passes(int bits) { const int p = (bits + RS_MAX_BITS - 1) / RS_MAX_BITS; return p < 1 ? 1 : p; }
static inline int radix_digit_bits(int bits) { const int p = radix_passes(bits), w = (bits + p - 1) / p; return w < 1 ? 1 : w; }

}  // namespace no
