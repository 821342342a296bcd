// no_select_hot and the embedding cache (Section 4.1.2): hotness = how often a vertex lands in
// V^1 (the set whose layer-1 embedding could be reused) while pre-sampling the training batches;
// the hot set is the top floor(fraction * V) by (count descending, id ascending).
#include <algorithm>
#include <mutex>
#include <type_traits>
#include <unordered_set>
#include "primitives.hpp"
#include "draw.hpp"
#include "handles.hpp"

#include <math.h>

namespace no {

// The vertices of V^1 of one batch, each counted once. The first n_seeds ids are the batch's own, which the caller may have repeated:
// last[v] is the stamp of the last batch that held v (a vertex further down the list stands there once). n_vertices > 0: the
// ids come straight from the caller; one outside [0, V) is not counted and raises *bad_flag.
__global__ void count_members_kernel(const int32_t* ids, const int32_t* d_n, int32_t n_seeds, int32_t* last, int32_t stamp, int32_t* freq,
                                     int32_t n_vertices, int32_t* bad_flag) {
    const int32_t n = d_n ? *d_n : n_seeds;
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t v = ids[i];
    if (n_vertices > 0 && (uint32_t)v >= (uint32_t)n_vertices) { *bad_flag = 1; return; }
    if (i < n_seeds && atomicExch(&last[v], stamp) == stamp) return;
    atomicAdd(&freq[v], 1);       // integer count: order independent
}

// One workgroup pre-samples one whole batch, all hops in one launch: V^1 is only wanted as a set, so a vertex is a bit of the
// batch's bitmap and the order in which the lanes meet it does not matter; the draws themselves depend on nothing but (stream, vertex,
// slot, hop). Hops above the last also append every vertex they meet for the first time to the batch's list, the destinations of
// the next hop. Batches are independent (train ids job % n_batches): workgroups take them in turn.
//
// The bitmap stands in LDS, in up to PRESAMPLE_RANGES parts of PRESAMPLE_RANGE vertices one after the other: a vertex of a later part
// waits in the `later` list while the first part is filled (4 bytes written and read in order; as a bit of a bitmap in memory it
// was a 64-byte sector read and written at random, and those were 60 % of the 52 M L2 misses of 508 batches). A thread draws whole
// rows, whose column entries it requests together.
// Measured (2.4 M vertices, 124 M edges, 1523 batches of 1024 seeds, fanouts 15 and 10), the pre-sampling alone: 3774 us with
// the bitmaps in memory, 1665 like this (278 us a batch and compute unit); it reads 47 G random sectors a second of the 54 G that independent
// 4-byte reads from 1 GB reach here.
constexpr int PRESAMPLE_THREADS = 1024;
constexpr int PRESAMPLE_RANGE = 152 * 1024 * 8;      // vertices; 152 of the 160 KB of a compute unit
constexpr int PRESAMPLE_RANGES = 4;
constexpr int PRESAMPLE_WORKERS = 256;               // workgroups of a launch: one a compute unit
constexpr int64_t PRESAMPLE_LIST_WORDS = 2ll << 28;  // and what their lists may take together (2 GiB; above, batches are few and large)
struct PresampleHops { int32_t fanout[NO_MAX_LAYERS]; int32_t n; };
// The batches of one launch: train ids, streams, and the vertices' range.
struct PresampleJobs {
    const int32_t* train; int64_t n_train; int32_t batch; int64_t n_batches, first_job; int32_t n_jobs; uint64_t seed; PresampleHops hops;
    int32_t n_vertices; int32_t* bad_flag;
};

template <int K, typename RowT>
__global__ void __launch_bounds__(PRESAMPLE_THREADS) presample_lds_kernel(PresampleJobs in, const RowT* __restrict__ rowptr,
                                                                          const int32_t* __restrict__ col, uint32_t* __restrict__ bitmaps,
                                                                          int64_t words, int32_t range, int32_t n_ranges, int32_t* lists,
                                                                          int64_t list_cap, int32_t* laters, int64_t later_cap) {
    extern __shared__ __attribute__((aligned(16))) uint32_t bits[];      // the current part's bitmap
    __shared__ int32_t n_list, n_later;
    int32_t* list = lists + (int64_t)blockIdx.x * list_cap;
    int32_t* later = laters + (int64_t)blockIdx.x * later_cap;
    const int lane = lane_id(), tid = (int)threadIdx.x;
    const int32_t range_words = range / 32;
    auto clear = [&] {
        for (int32_t w = tid; w < range_words / 4; w += PRESAMPLE_THREADS) reinterpret_cast<uint4*>(bits)[w] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
    };
    // the list's first n entries that lie in the part from `lo` on
    auto mark_list = [&](int32_t n, int32_t lo) {
        for (int32_t i = tid; i < n; i += PRESAMPLE_THREADS) {
            const uint32_t at = (uint32_t)(list[i] - lo);
            if (at < (uint32_t)range) atomicOr(&bits[at >> 5], 1u << (at & 31));
        }
        __syncthreads();
    };
    auto append = [&](bool on, int32_t u, int32_t* to, int32_t* count) {      // (every lane of the wavefront; one counter access for it)
        const uint64_t m = __ballot(on);
        int32_t at = 0;
        if (m && lane == 0) at = atomicAdd(count, __popcll(m));
        at = __builtin_amdgcn_readfirstlane(at);
        if (on) to[at + __popcll(m & ((1ull << lane) - 1ull))] = u;
    };
    // a vertex of the part from `lo` on: marked, and where it was not marked before and `keep`, it joins the list
    auto visit = [&](bool on, int32_t u, int32_t lo, bool keep) {
        const uint32_t at = (uint32_t)(u - lo), bit = 1u << (at & 31);
        if (!keep) {
            if (on) atomicOr(&bits[at >> 5], bit);
            return;
        }
        const bool fresh = on && !(atomicOr(&bits[at >> 5], bit) & bit);
        append(fresh, u, list, &n_list);
    };
    for (int32_t b = (int32_t)blockIdx.x; b < in.n_jobs; b += (int32_t)gridDim.x) {
        const int64_t job = in.first_job + b, first = (job % in.n_batches) * in.batch;
        const int32_t n_seeds = (int32_t)min((int64_t)in.batch, in.n_train - first);
        uint32_t* out = bitmaps + (int64_t)b * words;
        const uint64_t key = in.seed + (uint64_t)job;
        const uint32_t key0 = (uint32_t)key, key1 = (uint32_t)(key >> 32);
        __syncthreads();                              // (the batch before is done with the counters)
        if (tid == 0) n_list = 0;
        for (int32_t stage = 0; stage <= in.hops.n; ++stage) {      // the seeds, then the hops
            const bool keep = stage < in.hops.n;
            if (tid == 0) n_later = 0;
            if (stage == 0 || n_ranges > 1) clear(); else __syncthreads();
            const int32_t n_before = n_list;
            if (n_ranges > 1) mark_list(n_before, 0);
            __syncthreads();                          // (everybody has read the count before it grows)
            if (stage == 0) {
                for (int32_t i0 = 0; i0 < n_seeds; i0 += PRESAMPLE_THREADS) {
                    const int32_t i = i0 + tid;
                    const int32_t v = i < n_seeds ? in.train[first + i] : 0;
                    const bool ok = i < n_seeds && (uint32_t)v < (uint32_t)in.n_vertices;
                    if (i < n_seeds && !ok) *in.bad_flag = 1;       // never followed; the caller gets an error and no cache
                    visit(ok && v < range, v, 0, true);
                    if (n_ranges > 1) append(ok && v >= range, v, later, &n_later);
                }
            } else {
                const int32_t h = stage - 1, k = in.hops.fanout[h];
                const uint32_t c3 = (1u << 8) | (uint32_t)h;
                for (int32_t i0 = 0; i0 < n_before; i0 += PRESAMPLE_THREADS) {
                    const int32_t i = i0 + tid;
                    int64_t begin = 0;
                    uint32_t d = 0;
                    int32_t v = 0;
                    if (i < n_before) {
                        v = list[i];
                        begin = (int64_t)rowptr[v];
                        d = (uint32_t)((int64_t)rowptr[v + 1] - begin);
                    }
                    uint32_t pos[K];
#pragma unroll
                    for (int j = 0; j < K; ++j) pos[j] = (uint32_t)j;
                    if (d > (uint32_t)k) draw_row<K>(v, d, k, key0, key1, c3, pos);
                    const int32_t n = (int32_t)min(d, (uint32_t)k);
                    int32_t n_out = 0;
#pragma unroll
                    for (int j = 0; j < K; ++j) {      // (the vertex in the place of its position)
                        pos[j] = j < n ? (uint32_t)col[begin + pos[j]] : ~0u;
                        if (K > 16 && j % 8 == 7) __builtin_amdgcn_sched_barrier(0);      // (not all the addresses at a time: they spill)
                    }
#pragma unroll
                    for (int j = 0; j < K; ++j) {
                        if (j < k) visit(pos[j] < (uint32_t)range, (int32_t)pos[j], 0, keep);
                        n_out += (int32_t)pos[j] >= range ? 1 : 0;
                    }
                    if (n_ranges > 1) {
                        int32_t at = wave_inclusive_scan(n_out);
                        const int32_t all = __builtin_amdgcn_readlane(at, 63);
                        int32_t base = 0;
                        if (all && lane == 0) base = atomicAdd(&n_later, all);
                        at += __builtin_amdgcn_readfirstlane(base) - n_out;
#pragma unroll
                        for (int j = 0; j < K; ++j)
                            if ((int32_t)pos[j] >= range) later[at++] = (int32_t)pos[j];
                    }
                }
            }
            __syncthreads();
            for (int32_t r = 0; r < n_ranges; ++r) {
                const int32_t lo = r * range;
                if (r > 0) {
                    clear();
                    mark_list(n_before, lo);
                    const int32_t n = n_later;
                    for (int32_t i0 = 0; i0 < n; i0 += PRESAMPLE_THREADS) {
                        const int32_t i = i0 + tid;
                        const int32_t u = i < n ? later[i] : -1;
                        visit(i < n && u >= lo && u - lo < range, u, lo, keep);
                    }
                    __syncthreads();
                }
                if (!keep) {
                    const int32_t n4 = (int32_t)min((int64_t)range_words, words - lo / 32) / 4;
                    uint4* to = reinterpret_cast<uint4*>(out + lo / 32);
                    for (int32_t w = tid; w < n4; w += PRESAMPLE_THREADS) to[w] = reinterpret_cast<const uint4*>(bits)[w];
                    __syncthreads();
                }
            }
        }
    }
}

// The same with the bitmaps in memory, for more vertices than PRESAMPLE_RANGES parts hold, for wider fanouts and for small batches: workgroup-scope atomics
// (they end in the L2 of the die the workgroup runs on), a group of G lanes to a row, so that many workgroups share a compute
// unit. Bound by the latency of the dependent reads list -> row pointers -> column entry -> bitmap, hidden by 32 waves per compute
// unit (two workgroups, which is what the bound on the registers is for: with 106 scalar ones there was room for one, and 260 batches of 256 seeds,
// fanouts 40, 20 and 5, took 806 us; like this 597). In place of batches one after another through the training sampler: 117 -> 4.3 ms on the graph above.
template <int G, typename RowT>
__global__ void __launch_bounds__(PRESAMPLE_THREADS, 8) presample_kernel(PresampleJobs in, const RowT* __restrict__ rowptr,
                                                                      const int32_t* __restrict__ col, uint32_t* bitmaps, int64_t words,
                                                                      int32_t* lists, int64_t list_cap) {
    __shared__ int32_t n_list;
    const int64_t job = in.first_job + blockIdx.x;
    const int64_t lo = (job % in.n_batches) * in.batch;
    const int32_t n_seeds = (int32_t)min((int64_t)in.batch, in.n_train - lo);
    const PresampleHops& hops = in.hops;
    uint32_t* bm = bitmaps + (int64_t)blockIdx.x * words;
    int32_t* list = lists + (int64_t)blockIdx.x * list_cap;
    const uint64_t key = in.seed + (uint64_t)job;
    const uint32_t key0 = (uint32_t)key, key1 = (uint32_t)(key >> 32);
    const int lane = lane_id();
    // marks u; where it was not marked before and `keep`, it joins the list (one counter access per wavefront)
    auto visit = [&](bool on, int32_t u, bool keep) {
        bool fresh = false;
        if (on) {
            const uint32_t bit = 1u << (u & 31);
            fresh = !(__hip_atomic_fetch_or(&bm[u >> 5], bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) & bit);
        }
        if (!keep) return;
        const uint64_t m = __ballot(fresh);
        int32_t at = 0;
        if (m && lane == 0) at = atomicAdd(&n_list, __popcll(m));
        at = __shfl(at, 0, 64);
        if (fresh) list[at + __popcll(m & ((1ull << lane) - 1ull))] = u;
    };
    if (threadIdx.x == 0) n_list = 0;
    __syncthreads();
    for (int32_t i0 = 0; i0 < n_seeds; i0 += PRESAMPLE_THREADS) {
        const int32_t i = i0 + (int32_t)threadIdx.x;
        int32_t v = i < n_seeds ? in.train[lo + i] : 0;
        const bool ok = i < n_seeds && (uint32_t)v < (uint32_t)in.n_vertices;
        if (i < n_seeds && !ok) *in.bad_flag = 1;       // never followed; the caller gets an error and no cache
        visit(ok, v, true);
    }
    __syncthreads();
    constexpr int ROWS = PRESAMPLE_THREADS / G;
    const int32_t j = (int32_t)threadIdx.x % G;
    for (int32_t h = 0; h < hops.n; ++h) {
        const int32_t n_dst = n_list, k = hops.fanout[h];
        const uint32_t c3 = (1u << 8) | (uint32_t)h;
        const bool keep = h + 1 < hops.n;
        __syncthreads();                              // (everybody has read the count before it grows)
        for (int32_t i0 = 0; i0 < n_dst; i0 += ROWS) {
            const int32_t i = i0 + (int32_t)threadIdx.x / G;
            const bool row_ok = i < n_dst;
            int32_t v = 0;
            int64_t begin = 0;
            uint32_t d = 0;
            if (row_ok) {
                v = list[i];
                begin = (int64_t)rowptr[v];
                d = (uint32_t)((int64_t)rowptr[v + 1] - begin);
            }
            const uint32_t pos = draw_position<G>(row_ok, v, d, k, j, key0, key1, c3);
            const bool on = row_ok && j < k && (uint32_t)j < d;
            visit(on, on ? col[begin + pos] : 0, keep);
        }
        __syncthreads();
    }
}

// freq[v] += number of bitmaps that hold v. A thread adds one word of the bitmaps up in bit planes, two operations a plane for 32
// vertices at once, and takes the planes apart at the end. Where the bitmaps are long a wavefront owns 64 words of all of them, and a
// vertex that any of them holds costs one atomic: bound by the bitmaps' bytes (89 of 27.75 M vertices, 309 MB: 89 us).
// SHARED: where that leaves the chip idle, the eight wavefronts of a block share 64 words and deal the bitmaps out evenly; their counts meet in
// LDS, and no other block has these vertices. Every wavefront takes planes apart, however few its bitmaps are, and the block goes
// through all its counts: long bitmaps, and few of them, are the other form's. How few depends on how many atomics that one needs (`large`:
// batches such as are drawn in LDS; most counts are not zero). Measured, us, one wavefront / shared, bitmaps of large batches: 8 of 10 K
// vertices 16 / 6; 12 of 2.4 M 11 / 16, 60 24 / 19, 400 82 / 36; 400 of 3.7 M 85 / 54. Of small ones: 100 of 2.4 M 13 / 16, 250
// 24 / 21; 400 of 3.7 M 32 / 50. 89 of 27.75 M: 89 / 250.
constexpr int COUNT_FLIGHT = 16;
constexpr int count_planes(bool shared) { return shared ? 7 : 9; }
constexpr int count_waves(bool shared) { return shared ? 8 : 4; }      // (long bitmaps: small blocks, dealt more evenly)
static inline bool count_shared(int64_t words, int64_t n_maps, bool large) {
    return words < (large ? 64 * 2560 : 64 * 1536) && n_maps >= words / (large ? 3000 : 800);
}
template <bool SHARED>
__global__ void __launch_bounds__(64 * count_waves(SHARED), 8) count_bitmaps_kernel(const uint32_t* __restrict__ bitmaps, int64_t words, int32_t n_maps,
                                                                         int64_t n_vertices, int32_t* freq) {
    constexpr int WAVES = count_waves(SHARED), PLANES = count_planes(SHARED), MAPS = (1 << PLANES) - 1;
    __shared__ int32_t sums[SHARED ? 64 * 33 : 1];
    const int lane = lane_id(), wave = (int)(threadIdx.x >> 6);
    const int64_t w0 = ((int64_t)blockIdx.x * (SHARED ? 1 : WAVES) + (SHARED ? 0 : wave)) * 64, w = w0 + lane;
    if constexpr (SHARED) {
        for (int i = (int)threadIdx.x; i < 64 * 33; i += 64 * WAVES) sums[i] = 0;
        __syncthreads();
    }
    const int32_t share = SHARED ? (n_maps + WAVES - 1) / WAVES : n_maps;
    const int32_t begin = SHARED ? wave * share : 0, end = min(n_maps, begin + share);
    for (int32_t first = begin; w < words && first < end; first += MAPS) {
        const int32_t last = min(end, first + MAPS);
        uint32_t plane[PLANES] = {0};
        auto add = [&](uint32_t c) {
#pragma unroll
            for (int p = 0; p < PLANES; ++p) {
                const uint32_t carry = plane[p] & c;
                plane[p] ^= c;
                c = carry;
            }
        };
        int32_t m = first;
        uint32_t x[COUNT_FLIGHT];
        for (; m + COUNT_FLIGHT <= last; m += COUNT_FLIGHT) {
#pragma unroll
            for (int q = 0; q < COUNT_FLIGHT; ++q) x[q] = bitmaps[(int64_t)(m + q) * words + w];
#pragma unroll
            for (int q = 0; q < COUNT_FLIGHT; ++q) add(x[q]);
        }
        if (m < last) {      // the rest together too (past the last bitmap: that one again, not added)
#pragma unroll
            for (int q = 0; q < COUNT_FLIGHT; ++q) x[q] = bitmaps[(int64_t)min(m + q, last - 1) * words + w];
#pragma unroll
            for (int q = 0; q < COUNT_FLIGHT; ++q) add(m + q < last ? x[q] : 0u);
        }
#pragma unroll
        for (int b = 0; b < 32; ++b) {
            int32_t n = 0;
#pragma unroll
            for (int p = 0; p < PLANES; ++p) n |= (int32_t)((plane[p] >> b) & 1u) << p;
            if constexpr (SHARED) {
                if (n) atomicAdd(&sums[lane * 33 + b], n);
            } else {
                if (n && w * 32 + b < n_vertices) atomicAdd(&freq[w * 32 + b], n);
            }
        }
    }
    if constexpr (SHARED) {
        __syncthreads();
        for (int i = (int)threadIdx.x; i < 2048; i += 64 * WAVES) {
            const int64_t v = w0 * 32 + i;
            const int32_t n = sums[(i >> 5) * 33 + (i & 31)];
            if (n && v < n_vertices) freq[v] += n;
        }
    }
}

__global__ void hot_keys_kernel(const int32_t* freq, int64_t n, uint32_t max_count, uint32_t* keys, uint32_t* ids) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) { keys[i] = max_count - (uint32_t)freq[i]; ids[i] = (uint32_t)i; }
}

__global__ void hot_slots_kernel(const uint32_t* order, int64_t n_hot, int32_t* hot_ids, int32_t* slot_of_vertex) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_hot) { int32_t v = (int32_t)order[i]; hot_ids[i] = v; slot_of_vertex[v] = (int32_t)i; }
}

}  // namespace no

using namespace no;

namespace no {
static std::mutex g_cache_mutex;
static std::unordered_set<no_cache_s*> g_live_caches;
static uint64_t g_next_cache_uid = 1;
void cache_register(no_cache_s* c) { std::lock_guard<std::mutex> l(g_cache_mutex); c->uid = g_next_cache_uid++; g_live_caches.insert(c); }
void cache_unregister(no_cache_s* c) { std::lock_guard<std::mutex> l(g_cache_mutex); g_live_caches.erase(c); }
bool cache_is_live(no_cache_s* c) { std::lock_guard<std::mutex> l(g_cache_mutex); return g_live_caches.count(c) != 0; }
}  // namespace no

// Whether a batch keeps a workgroup busy while its bitmap stands in LDS. Every stage empties the bitmap's parts and goes through the list for each, and a
// thread draws the slots of its row one after the other, which few rows leave without cover: batches of few seeds, in memory, share a
// compute unit and take a group of lanes to a row. Measured, time of a call in memory over that in LDS: one part, fanouts 10 and 5,
// 64 seeds 0.93, 256 1.18; 15, 10 and 5, 16 seeds 0.88, 64 1.27; 25 and 10, 64 seeds 0.69, 256 1.01, 1024 1.46. Four parts, 10 and 5, 256
// seeds 0.90, 1024 1.15; 15, 10 and 5, 64 seeds 0.89, 256 1.32; 25 and 10, 256 seeds 0.82, 1024 1.09.
static bool presample_fills_workgroup(int32_t batch, int64_t slots_per_batch, int32_t widest, int64_t n_ranges) {
    if (batch >= 256) return n_ranges <= 2 || slots_per_batch >= (widest <= 16 ? 10000 : 40000);
    return widest <= 16 ? batch >= 32 * n_ranges && slots_per_batch >= 1250 * n_ranges : batch >= 32 && slots_per_batch >= 12000 + 6000 * n_ranges;
}

// Whether whole batches are pre-sampled by one workgroup each, a group of them per launch, or one after the other with the
// training sampler, every hop spread over the chip. A batch takes the sampler a dozen launches (about 80 us) however small it
// is, and a workgroup about 2 us per 1024 slots, as many of them at a time as the chip holds (bitmaps in LDS: one a compute unit): few but very
// large batches stay with the sampler. Measured, sampler / workgroups, us a call on 2.4 M vertices, fanouts 15, 10 and 5: 4 batches of 4096
// 387 / 542, 16 1111 / 679; 6 of 60,000 1385 / 5114; fanouts 10 and 5, 4 of 4096 229 / 174, 6 of 60,000 481 / 790, 20 1248 / 814.
static bool presample_by_group(int64_t n_batches, int64_t slots_per_batch, int64_t at_a_time) {
    const double rounds = (double)ceil_div(n_batches, at_a_time);
    return rounds * (20.0 + 2.0 * (double)slots_per_batch / 1024.0) < 80.0 * (double)n_batches;
}

extern "C" int32_t no_select_hot(no_graph_t g, const int32_t* d_train_ids, int64_t n_train, int32_t batch,
                                 const int32_t* h_fanouts, int32_t n_layers, int32_t presample_epochs,
                                 double hot_fraction, int32_t staleness, int32_t emb_dim, uint64_t seed, void* stream,
                                 no_cache_t* out) {
    clear_error();
    NO_REQUIRE(out != nullptr, NO_ERR_INVALID_ARG, "no_select_hot: out is NULL");
    *out = nullptr;
    NO_REQUIRE(g && d_train_ids && h_fanouts, NO_ERR_INVALID_ARG, "no_select_hot: NULL argument");
    NO_REQUIRE(n_train >= 1 && batch >= 1, NO_ERR_INVALID_ARG, "no_select_hot: n_train and batch must be positive");
    NO_REQUIRE(n_layers >= 1 && n_layers <= NO_MAX_LAYERS, NO_ERR_INVALID_ARG, "no_select_hot: bad n_layers");
    for (int32_t h = 0; h < n_layers; ++h)
        NO_REQUIRE(h_fanouts[h] >= 1 && h_fanouts[h] <= NO_MAX_FANOUT, NO_ERR_INVALID_ARG, "no_select_hot: bad fanout[%d]", h);
    NO_REQUIRE(presample_epochs >= 1, NO_ERR_INVALID_ARG, "no_select_hot: presample_epochs must be >= 1");
    NO_REQUIRE(hot_fraction >= 0.0 && hot_fraction <= 1.0, NO_ERR_INVALID_ARG, "no_select_hot: hot_fraction outside [0,1]");
    NO_REQUIRE(staleness >= 0, NO_ERR_INVALID_ARG, "no_select_hot: staleness must be >= 0");
    NO_REQUIRE(emb_dim >= 1, NO_ERR_INVALID_ARG, "no_select_hot: emb_dim must be positive");
    NO_REQUIRE(batch <= g->n_vertices, NO_ERR_INVALID_ARG, "no_select_hot: batch larger than the graph");
    hipStream_t st = (hipStream_t)stream;
    const int64_t V = g->n_vertices;
    const int64_t nb = ceil_div(n_train, batch);
    const int64_t max_count = (int64_t)presample_epochs * nb;
    NO_REQUIRE(max_count < (1ll << 31), NO_ERR_OVERFLOW, "no_select_hot: too many pre-sampling batches");

    no_cache_s* c = new no_cache_s();
    struct Guard { no_cache_s* c; ~Guard() { if (c) { c->release(); delete c; } } } guard{c};
    c->n_vertices = V;
    c->staleness = staleness;
    c->emb_dim = emb_dim;
    c->n_hot = (int64_t)floor(hot_fraction * (double)V);
    NO_CHECK(c->freq.alloc((size_t)V));
    NO_CHECK(c->slot_of_vertex.alloc((size_t)V));
    NO_CHECK(c->hot_ids.alloc((size_t)c->n_hot));
    NO_CHECK(c->version.alloc((size_t)c->n_hot));
    NO_CHECK(c->emb.alloc((size_t)c->n_hot * emb_dim));
    NO_CHECK(fill_i32(c->freq.p, 0, V, st));
    NO_CHECK(fill_i32(c->slot_of_vertex.p, -1, V, st));
    NO_CHECK(fill_i32(c->version.p, -1, c->n_hot, st));
    NO_CHECK(fill_i32((int32_t*)c->emb.p, 0, c->n_hot * emb_dim, st));

    // pre-sampling: hops 0 .. L-2 of every batch, Philox domain 1
    no_blocks_s* b = nullptr;
    struct BGuard { no_blocks_s*& b; ~BGuard() { if (b) { b->release(); delete b; } } } bguard{b};
    // bad_flag: an id outside [0, V) among the train ids. arena: bitmaps and lists of a group of batches, then the sort's arrays.
    DevBuf<int32_t> bad_flag, arena;
    struct FGuard { DevBuf<int32_t>* f[2]; ~FGuard() { ReleaseScope scope; f[0]->release(); f[1]->release(); } } fguard{{&bad_flag, &arena}};
    NO_CHECK(bad_flag.alloc(1));
    NO_CHECK(fill_i32(bad_flag.p, 0, 1, st));
    // slots a batch draws at most (in all, and in one stage: the seeds, a hop), and destinations of its last pre-sampled hop at most
    int64_t slots = 0, last_slots = batch, dst_cap = batch;
    int32_t widest = 1;
    for (int32_t h = 0; h + 1 < n_layers; ++h) {
        slots += dst_cap * h_fanouts[h];
        last_slots = std::max(last_slots, dst_cap * h_fanouts[h]);
        if (h + 2 < n_layers) dst_cap = std::min<int64_t>(V, dst_cap * (h_fanouts[h] + 1));
        widest = std::max(widest, h_fanouts[h]);
    }
    // A group is as many batches as fit 192 MiB (larger device allocations take the runtime some 250 us to give back), more
    // where that would make more than 16 groups; groups are of equal size.
    // Bitmaps in LDS: lists and waiting vertices are per workgroup, and a group is a whole number of batches for each of them where it
    // takes several.
    const int64_t n_ranges = ceil_div(V, PRESAMPLE_RANGE);
    const int32_t range = (int32_t)(ceil_div(ceil_div(V, n_ranges), 128) * 128);
    const int64_t later_cap = n_ranges > 1 ? last_slots : 0;
    const bool fits_lds = n_ranges <= PRESAMPLE_RANGES && widest <= 32 && presample_fills_workgroup(batch, slots, widest, n_ranges) &&
                          std::min<int64_t>(max_count, PRESAMPLE_WORKERS) * (dst_cap + later_cap) <= PRESAMPLE_LIST_WORDS;
    const bool by_group = n_layers >= 2 && presample_by_group(max_count, slots, (fits_lds ? 1 : 2) * PRESAMPLE_WORKERS);
    const bool in_lds = by_group && fits_lds;
    const int64_t words = ceil_div(V, 128) * 4, per_batch = words + (in_lds ? 0 : dst_cap);       // (32-bit words)
    int64_t group = 0, arena_words = 0, workers = 0;
    if (by_group) {
        const int64_t room = std::max<int64_t>(192ll << 18, std::min<int64_t>(4ll << 28, max_count * per_batch / 16));
        group = std::max<int64_t>(1, std::min<int64_t>(max_count, room / per_batch));
        group = ceil_div(max_count, ceil_div(max_count, group));
        if (in_lds) {
            workers = std::min<int64_t>(group, PRESAMPLE_WORKERS);
            group = ceil_div(group, workers) * workers;
        }
        arena_words = group * per_batch + workers * (dst_cap + later_cap);
    }
    const int64_t sort_words = c->n_hot > 0 ? 6 * V + (int64_t)(radix_ws_bytes(V) + 15) / 4 : 0;
    NO_CHECK(arena.alloc((size_t)std::max(arena_words, sort_words)));
    if (by_group) {
        uint32_t* bitmaps = (uint32_t*)arena.p;
        int32_t* lists = arena.p + group * words;
        int32_t* laters = lists + workers * dst_cap;
        PresampleJobs in{d_train_ids, n_train, batch, nb, 0, 0, seed, {}, (int32_t)V, bad_flag.p};
        in.hops.n = n_layers - 1;
        for (int32_t h = 0; h < in.hops.n; ++h) in.hops.fanout[h] = h_fanouts[h];
        const size_t lds = (size_t)range / 8;
        for (int64_t job = 0; job < max_count; job += group) {
            const int32_t n = (int32_t)std::min<int64_t>(group, max_count - job);
            in.first_job = job;
            in.n_jobs = n;
            auto launch = [&](auto rp) -> int32_t {
                using RowT = std::remove_const_t<std::remove_pointer_t<decltype(rp)>>;
                if (in_lds) {
                    auto kernel = widest <= 16 ? presample_lds_kernel<16, RowT> : presample_lds_kernel<32, RowT>;
                    NO_HIP_CHECK(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
                    hipLaunchKernelGGL(kernel, dim3((unsigned)std::min<int64_t>(n, workers)), dim3(PRESAMPLE_THREADS), lds, st, in, rp, g->col.p,
                                       bitmaps, words, range, (int32_t)n_ranges, lists, dst_cap, laters, later_cap);
                    return NO_OK;
                }
                NO_CHECK(fill_i32((int32_t*)bitmaps, 0, n * words, st));
                auto kernel = widest <= 8 ? presample_kernel<8, RowT> : widest <= 16 ? presample_kernel<16, RowT>
                            : widest <= 32 ? presample_kernel<32, RowT> : presample_kernel<64, RowT>;
                hipLaunchKernelGGL(kernel, dim3((unsigned)n), dim3(PRESAMPLE_THREADS), 0, st, in, rp, g->col.p, bitmaps, words, lists, dst_cap);
                return NO_OK;
            };
            if (g->rowptr_bits == 64) NO_CHECK(launch((const int64_t*)g->rowptr64.p));
            else NO_CHECK(launch((const int32_t*)g->rowptr32.p));
            if (count_shared(words, n, in_lds))
                hipLaunchKernelGGL(count_bitmaps_kernel<true>, dim3((unsigned)ceil_div(words, 64)), dim3(64 * count_waves(true)), 0, st,
                                   (const uint32_t*)bitmaps, words, n, V, c->freq.p);
            else
                hipLaunchKernelGGL(count_bitmaps_kernel<false>, dim3((unsigned)ceil_div(words, 64 * count_waves(false))), dim3(64 * count_waves(false)), 0,
                                   st, (const uint32_t*)bitmaps, words, n, V, c->freq.p);
        }
    } else {
        if (n_layers >= 2) NO_CHECK(blocks_create_impl(g, batch, h_fanouts, n_layers - 1, false, &b));
        int32_t* last = c->slot_of_vertex.p;      // (filled after the ranking)
        for (int64_t job = 0; job < max_count; ++job) {
            const int64_t lo = job % nb * batch;
            const int32_t n = (int32_t)std::min<int64_t>(batch, n_train - lo);
            if (n_layers >= 2) {
                NO_CHECK(sample_blocks_impl(g, d_train_ids + lo, n, seed + (uint64_t)job, 1u, n_layers - 1, nullptr, 0, b, st));
                const HopBuffers& H = b->hop[n_layers - 2];
                hipLaunchKernelGGL(count_members_kernel, dim3((unsigned)ceil_div(H.n_src_cap, 256)), dim3(256), 0, st,
                                   (const int32_t*)H.src_global.p, (const int32_t*)(b->counts.p + 4 * (n_layers - 2) + 1), n, last,
                                   (int32_t)job, c->freq.p, 0, (int32_t*)nullptr);
            } else {
                hipLaunchKernelGGL(count_members_kernel, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, st, d_train_ids + lo,
                                   (const int32_t*)nullptr, n, last, (int32_t)job, c->freq.p, (int32_t)V, bad_flag.p);
            }
        }
        NO_CHECK(fill_i32(last, -1, V, st));
    }
    NO_CHECK(launch_status("presample"));

    // rank: stable sort of ids by (max_count - freq) keeps ascending id among equal counts
    if (c->n_hot > 0) {
        uint32_t* a = (uint32_t*)arena.p;
        uint32_t *k_in = a, *v_in = a + V, *k_out = a + 2 * V, *v_out = a + 3 * V, *k_tmp = a + 4 * V, *v_tmp = a + 5 * V;
        void* ws = (void*)(((uintptr_t)(a + 6 * V) + 15) & ~(uintptr_t)15);
        int64_t blocks = ceil_div(V, 256 * 4);
        if (blocks > 65536) blocks = 65536;
        hipLaunchKernelGGL(hot_keys_kernel, dim3((unsigned)blocks), dim3(256), 0, st, (const int32_t*)c->freq.p, V,
                           (uint32_t)max_count, k_in, v_in);
        int bits = ilog2_ceil((uint64_t)max_count + 1);
        if (bits < 1) bits = 1;
        NO_CHECK(radix_sort_pairs(k_in, v_in, k_out, v_out, k_tmp, v_tmp, V, bits, ws, st));
        hipLaunchKernelGGL(hot_slots_kernel, dim3((unsigned)ceil_div(c->n_hot, 256)), dim3(256), 0, st,
                           (const uint32_t*)v_out, c->n_hot, c->hot_ids.p, c->slot_of_vertex.p);
        NO_CHECK(launch_status("hot ranking"));
    }
    NO_HIP_CHECK(hipStreamSynchronize(st));
    {
        // the private blocks start with zeroed flag words, so anything in them was raised by one of the batches above
        int32_t flags[4] = {0, 0, 0, 0};
        if (b) NO_HIP_CHECK(hipMemcpy(flags, b->counts.p + 4 * (n_layers - 1) + 5, 2 * sizeof(int32_t), hipMemcpyDeviceToHost));
        NO_HIP_CHECK(hipMemcpy(flags + 2, bad_flag.p, sizeof(int32_t), hipMemcpyDeviceToHost));
        NO_REQUIRE(flags[1] == 0, NO_ERR_TIMEOUT, "no_select_hot: a scan gave up waiting for an earlier tile");
        NO_REQUIRE(flags[0] == 0 && flags[2] == 0, NO_ERR_OUT_OF_RANGE, "no_select_hot: a train id lies outside [0, V)");
    }
    guard.c = nullptr;
    no::cache_register(c);
    handle_created();
    *out = c;
    return NO_OK;
}

extern "C" int32_t no_cache_view(no_cache_t c, int64_t* n_hot, int32_t* staleness, int32_t* emb_dim,
                                 const int32_t** d_hot_ids, const int32_t** d_slot_of_vertex, int32_t** d_version,
                                 float** d_emb, const int32_t** d_freq) {
    clear_error();
    NO_REQUIRE(c != nullptr, NO_ERR_INVALID_ARG, "no_cache_view: cache is NULL");
    if (n_hot) *n_hot = c->n_hot;
    if (staleness) *staleness = c->staleness;
    if (emb_dim) *emb_dim = c->emb_dim;
    if (d_hot_ids) *d_hot_ids = c->hot_ids.p;
    if (d_slot_of_vertex) *d_slot_of_vertex = c->slot_of_vertex.p;
    if (d_version) *d_version = c->version.p;
    if (d_emb) *d_emb = c->emb.p;
    if (d_freq) *d_freq = c->freq.p;
    return NO_OK;
}

extern "C" int32_t no_cache_set_staleness(no_cache_t c, int32_t staleness) {
    clear_error();
    NO_REQUIRE(c != nullptr, NO_ERR_INVALID_ARG, "no_cache_set_staleness: cache is NULL");
    NO_REQUIRE(staleness >= 0, NO_ERR_INVALID_ARG, "no_cache_set_staleness: staleness must be >= 0");
    c->staleness = staleness;
    ++c->generation;
    return NO_OK;
}

extern "C" int32_t no_cache_set_layer_form(no_cache_t c, no_arch form) {
    clear_error();
    NO_REQUIRE(c != nullptr, NO_ERR_INVALID_ARG, "no_cache_set_layer_form: cache is NULL");
    NO_REQUIRE(form == NO_ARCH_GCN || form == NO_ARCH_GCN_SUM || form == NO_ARCH_GCN_SYM, NO_ERR_INVALID_ARG,
               "no_cache_set_layer_form: not a GCN-style form");
    NO_REQUIRE(!(c->refresh && c->refresh->pending), NO_ERR_INVALID_ARG, "no_cache_set_layer_form: a refresh is pending");
    c->gcn_form = form;
    return NO_OK;
}

extern "C" int32_t no_cache_invalidate(no_cache_t c, void* stream) {
    clear_error();
    NO_REQUIRE(c != nullptr, NO_ERR_INVALID_ARG, "no_cache_invalidate: cache is NULL");
    ++c->generation;
    ++c->contents;
    return fill_i32(c->version.p, -1, c->n_hot, (hipStream_t)stream);
}

extern "C" int32_t no_cache_destroy(no_cache_t c) {
    clear_error();
    if (!c) return NO_OK;
    no::cache_unregister(c);
    c->release();
    delete c;
    handle_destroyed();
    return NO_OK;
}
