// no_sample_blocks: reverse multi-hop fanout sampling over the in-neighbour CSR (the sample()
// loop of Algorithm 1), de-duplication / relabelling of each frontier, the block transpose used
// by the backward pass, and the hot-vertex lookup that removes reusable vertices from the bottom
// hop (Section 4.1.2, Stage 1 of Section 4.2).
//
// One hop is four kernels over a fixed-stride ("padded") edge array, slot q = row * fanout + j:
//   1. sample_rows   a sub-wave group of G lanes (G = 8/16/32/64 >= fanout) serves one destination;
//                    lane j draws slot j with Philox4x32-10 keyed by (stream; vertex, slot, domain,
//                    hop), the group hands the partial Fisher-Yates swap chain from lane to lane
//                    by DPP, and every sampled id does atomicMin(map[id], n_dst + q): the first
//                    occurrence of an id in (row, slot) order wins, whatever the execution order;
//   2. edge_tile_sums  per 1024-slot tile: number of sampled edges and of first occurrences
//                    (many tiles: tile_offsets adds them up);
//   3. edge_assign   tile prefix + block scan: compact edge ids, row pointers, new local ids in
//                    first-occurrence order, map[id] = local id;
//   4. edge_indices  indices[e] = map[id]; counts per source for the transpose.
// `map` is a direct-address table int32[V] (HBM is plentiful; no hashing, no probing order to
// reason about). It carries the local ids from one hop to the next and is wiped after the last.
// The transpose (hops above the bottom one) is a counting sort: scan of the per-source counts,
// unordered fill in order of arrival at the counts, then every edge ranks itself inside its (short) column so
// that columns end up in ascending edge id regardless of the fill order.
// 4 and the transpose are side tasks: extra blocks of the launches that follow (side.hpp).
#include "side.hpp"
#include "draw.hpp"
#include "handles.hpp"
#include "layers.hpp"

#include <algorithm>
#include <type_traits>

namespace no {

// Tiles of the slot scans: 1024 slots (four per thread). Measured on three hops of 15 K / 34 K / 122 K slots: sampling
// stage 232 / 190 / 173 / 171 / 179 us at 4096 / 2048 / 1024 / 512 / 256 slots per tile (a thread's dependent loads and
// its scattered stores are the latency of the kernel; more tiles are more sums for every block to add up).
constexpr int ETHREADS = 256, EITEMS = 4, ETILE = ETHREADS * EITEMS;

// ---------------------------------------------------------------------------- 1. sampling

template <int G, typename RowT>
__global__ void __launch_bounds__(256) sample_rows_kernel(const RowT* __restrict__ rowptr, const int32_t* __restrict__ col,
                                                          const int32_t* __restrict__ dst, const int32_t* d_n_dst,
                                                          int32_t n_fixed, int32_t n_cap, int32_t k, uint32_t key0,
                                                          uint32_t key1, uint32_t c3, int32_t* __restrict__ nbr_pad,
                                                          int32_t* __restrict__ src_global, int32_t* map,
                                                          int32_t insert_dst, int32_t* seeds_copy, int32_t* count_out,
                                                          int32_t n_vertices, int32_t* bad_id_flag, int32_t flag_value,
                                                          unsigned long long* scan_status, int32_t n_status,
                                                          int32_t* zero_extra, SideTasks side) {
    if (blockIdx.x >= side.first_block) { run_side_tasks(side); return; }
    // the tile status words of the scan that follows this launch start out empty
    for (int32_t t = (int32_t)(blockIdx.x * 256 + threadIdx.x); t < n_status; t += (int32_t)(side.first_block * 256)) scan_status[t] = 0ull;
    int32_t n_dst = d_n_dst ? *d_n_dst : n_fixed;
    if (n_dst > n_cap) n_dst = n_cap;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *count_out = n_dst;
        if (zero_extra) zero_extra[0] = zero_extra[1] = zero_extra[4] = 0;      // no cache: nothing computed, reused, refreshed
    }
    const int32_t i = (int32_t)(blockIdx.x * (256 / G) + threadIdx.x / G);
    const int32_t j = (int32_t)(threadIdx.x % G);
    const bool row_ok = i < n_dst;
    int32_t v = 0;
    int64_t begin = 0;
    uint32_t d = 0;
    if (row_ok) {
        v = dst[i];
        if (insert_dst && (uint32_t)v >= (uint32_t)n_vertices) {
            // a caller-supplied seed outside [0, V): stay inside the graph's arrays and report it
            v = 0;
            *bad_id_flag = flag_value;
        }
        begin = (int64_t)rowptr[v];
        d = (uint32_t)((int64_t)rowptr[v + 1] - begin);
        if (j == 0) {
            src_global[i] = v;
            if (insert_dst) map[v] = i;       // a plain store and the atomicMin below commute: i is the smaller value
            if (seeds_copy) seeds_copy[i] = v;
        }
    }
    const uint32_t pos = draw_position<G>(row_ok, v, d, k, j, key0, key1, c3);
    const int32_t cnt = d < (uint32_t)k ? (int32_t)d : k;
    if (row_ok && j < k) {
        const int32_t q = i * k + j;
        if (j < cnt) {
            int32_t u = col[begin + pos];
            nbr_pad[q] = u;
            atomicMin(&map[u], n_dst + q);   // integer min: order independent
        } else {
            nbr_pad[q] = -1;
        }
    }
}

// The draw alone, into the slots: for a bulk refresh, whose rows are aggregated straight from the slots and whose sources need no numbers (without
// the id map's atomics, the compaction and the side tasks behind it; 240 K rows, fanout 5, beside four steps: 74 us and 62 behind it -> 30; the super-batch 1229 -> 1164).
template <int G, typename RowT>
__global__ void __launch_bounds__(256) draw_rows_kernel(const RowT* __restrict__ rowptr, const int32_t* __restrict__ col, const int32_t* __restrict__ dst,
                                                        int32_t n, int32_t k, uint32_t key0, uint32_t key1, uint32_t c3, int32_t* __restrict__ nbr_pad,
                                                        int32_t* count_out) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *count_out = n;
    const int64_t i = (int64_t)blockIdx.x * (256 / G) + threadIdx.x / G;
    const int32_t j = (int32_t)(threadIdx.x % G);
    const bool row_ok = i < n;
    int32_t v = 0;
    int64_t begin = 0;
    uint32_t d = 0;
    if (row_ok) {
        v = dst[i];
        begin = (int64_t)rowptr[v];
        d = (uint32_t)((int64_t)rowptr[v + 1] - begin);
    }
    const uint32_t pos = draw_position<G>(row_ok, v, d, k, j, key0, key1, c3);
    if (row_ok && j < k) nbr_pad[i * k + j] = (uint32_t)j < d ? col[begin + pos] : -1;      // (a row of d <= k entries is taken whole)
}

template <typename RowT>
static void launch_draw(const RowT* rowptr, const int32_t* col, const int32_t* d_dst, int32_t n, int32_t k, uint32_t key0, uint32_t key1, uint32_t c3,
                        int32_t* nbr_pad, int32_t* count, hipStream_t st) {
    auto launch = [&](auto group) {
        constexpr int G = decltype(group)::value;
        hipLaunchKernelGGL((draw_rows_kernel<G, RowT>), dim3((unsigned)ceil_div(n, 256 / G)), dim3(256), 0, st, rowptr, col, d_dst, n, k, key0, key1, c3,
                           nbr_pad, count);
    };
    if (k <= 8) launch(std::integral_constant<int, 8>{});
    else if (k <= 16) launch(std::integral_constant<int, 16>{});
    else if (k <= 32) launch(std::integral_constant<int, 32>{});
    else launch(std::integral_constant<int, 64>{});
}

int32_t draw_rows(no_graph_s* g, const int32_t* d_dst, int32_t n, uint64_t stream_key, uint32_t domain, no_blocks_s* b, hipStream_t st) {
    HopBuffers& H = b->hop[0];
    const uint32_t key0 = (uint32_t)stream_key, key1 = (uint32_t)(stream_key >> 32), c3 = domain << 8;
    if (g->rowptr_bits == 64) launch_draw<int64_t>(g->rowptr64.p, g->col.p, d_dst, n, H.fanout, key0, key1, c3, H.nbr_pad.p, b->counts.p, st);
    else launch_draw<int32_t>(g->rowptr32.p, g->col.p, d_dst, n, H.fanout, key0, key1, c3, H.nbr_pad.p, b->counts.p, st);
    return launch_status("draw_rows");
}

// ---------------------------------------------------------------------------- 2./3. compaction and new ids

__device__ __forceinline__ int64_t slot_flags(const int32_t* __restrict__ nbr_pad, const int32_t* map, int64_t q,
                                              int32_t n_dst, int32_t* u_out) {
    const int32_t u = nbr_pad[q];
    *u_out = u;
    if (u < 0) return 0;
    return 1ll + ((map[u] == n_dst + (int32_t)q) ? (1ll << 32) : 0ll);    // low word: sampled; high word: first seen
}

// (the two-launch form: the tile sums pass marks the first occurrences in the padded array itself, -2 - id in place of id,
// so that the assignment pass reads its flags with the slots and does not wait for a second probe of the id map)
__device__ __forceinline__ int64_t slot_flags_marked(const int32_t* __restrict__ nbr_pad, int64_t q, int32_t* u_out) {
    const int32_t e = nbr_pad[q];
    *u_out = e <= -2 ? -2 - e : e;
    if (e == -1) return 0;
    return 1ll + (e <= -2 ? (1ll << 32) : 0ll);
}

__global__ void __launch_bounds__(ETHREADS) edge_tile_sums_kernel(int32_t* __restrict__ nbr_pad, const int32_t* map,
                                                                  const int32_t* d_n_dst, int32_t k, int64_t* tile_sums,
                                                                  int32_t* csc_cnt, int32_t n_zero, SideTasks side) {
    if (blockIdx.x >= side.first_block) { run_side_tasks(side); return; }
    for (int64_t t = (int64_t)blockIdx.x * ETHREADS + threadIdx.x; t < n_zero; t += (int64_t)side.first_block * ETHREADS) csc_cnt[t] = 0;
    const int32_t n_dst = *d_n_dst;
    const int64_t n_pad = (int64_t)n_dst * k;
    const int64_t base = (int64_t)blockIdx.x * ETILE;
    if (base >= n_pad) return;
    __shared__ int64_t smem[ETHREADS / 64];
    const int64_t q0 = base + (int64_t)threadIdx.x * EITEMS;
    int64_t s = 0;
#pragma unroll
    for (int t = 0; t < EITEMS; ++t) {
        int32_t u;
        if (q0 + t < n_pad) {
            const int64_t f = slot_flags(nbr_pad, map, q0 + t, n_dst, &u);
            if (f >> 32) nbr_pad[q0 + t] = -2 - u;
            s += f;
        }
    }
    s = block_sum<int64_t, ETHREADS>(s, smem);
    if (threadIdx.x == 0) tile_sums[blockIdx.x] = s;
}

// The sum of the first n tiles, to all threads of the block: added up here, or read where tile_offsets_kernel has done it.
__device__ __forceinline__ int64_t tiles_before(const int64_t* __restrict__ tile_sums, int64_t n, int32_t summed, int64_t* smem) {
    if (summed) return tile_sums[n];
    int64_t s = 0;
    for (int64_t t = threadIdx.x; t < n; t += ETHREADS) s += tile_sums[t];
    return block_sum<int64_t, ETHREADS>(s, smem);
}

// Sums of the tiles before each of them in place of their own, and behind them the sum of all, by one block. Without it every block adds up all tiles
// before its own, which grows with their square. Measured, without / with: bulk refresh of 14 K tiles 1.17 / 1.14 ms, of 81 K 6.79 / 5.43, of
// 271 K 32.4 / 17.4, of 1.08 M 313 / 30.8; sampling with room for 23 K tiles, of which a batch fills a part, 489 / 502 us.
constexpr int64_t OFFSETS_TILES = 24576;
__global__ void __launch_bounds__(1024) tile_offsets_kernel(const int32_t* d_n, int32_t k, int64_t* sums) {
    constexpr int PER = 8;
    __shared__ int64_t smem[1024 / 64 + 1];
    const int64_t n_tiles = ((int64_t)*d_n * k + ETILE - 1) / ETILE;
    int64_t v[PER], next[PER], carry = 0;
    auto request = [&](int64_t base) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int64_t t = base + (int64_t)threadIdx.x * PER + i;
            next[i] = t < n_tiles ? sums[t] : 0;
        }
    };
    request(0);
    for (int64_t base = 0; base < n_tiles; base += 1024 * PER) {
        int64_t s = 0, total;
#pragma unroll
        for (int i = 0; i < PER; ++i) s += v[i] = next[i];
        request(base + 1024 * PER);
        int64_t run = carry + block_exclusive_scan<int64_t, 1024>(s, &total, smem);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int64_t t = base + (int64_t)threadIdx.x * PER + i;
            if (t < n_tiles) sums[t] = run;
            run += v[i];
        }
        carry += total;
    }
    if (threadIdx.x == 0) sums[n_tiles] = carry;
}

__global__ void __launch_bounds__(ETHREADS) edge_assign_kernel(const int32_t* __restrict__ nbr_pad, int32_t* map,
                                                               const int32_t* d_n_dst, int32_t k, uint64_t k_magic,
                                                               const int64_t* __restrict__ tile_sums, int32_t summed,
                                                               int32_t* __restrict__ indptr, int32_t* __restrict__ nbr,
                                                               int32_t* __restrict__ edge_row, int32_t* __restrict__ src_global,
                                                               int32_t* counts /* [0]=n_dst (in), [1]=n_src, [2]=nnz */,
                                                               SideTasks side) {
    if (blockIdx.x >= side.first_block) { run_side_tasks(side); return; }
    __shared__ int64_t smem[ETHREADS / 64 + 1];
    const int32_t n_dst = *d_n_dst;
    const int64_t n_pad = (int64_t)n_dst * k;
    const int64_t n_tiles = (n_pad + ETILE - 1) / ETILE;
    if (blockIdx.x == 0) {
        const int64_t s = tiles_before(tile_sums, n_tiles, summed, smem);
        if (threadIdx.x == 0) {
            const int32_t nnz = (int32_t)(s & 0xffffffffll), n_new = (int32_t)(s >> 32);
            indptr[n_dst] = nnz;
            counts[1] = n_dst + n_new;
            counts[2] = nnz;
        }
    }
    const int64_t base = (int64_t)blockIdx.x * ETILE;
    if (base >= n_pad) return;
    const int64_t tile_off = tiles_before(tile_sums, blockIdx.x, summed, smem);
    const int64_t q0 = base + (int64_t)threadIdx.x * EITEMS;
    int64_t f[EITEMS];
    int32_t u[EITEMS];
    int64_t s = 0;
#pragma unroll
    for (int t = 0; t < EITEMS; ++t) {
        f[t] = 0;
        u[t] = -1;
        if (q0 + t < n_pad) f[t] = slot_flags_marked(nbr_pad, q0 + t, &u[t]);
        s += f[t];
    }
    int64_t total;
    int64_t run = block_exclusive_scan<int64_t, ETHREADS>(s, &total, smem) + tile_off;
#pragma unroll
    for (int t = 0; t < EITEMS; ++t) {
        const int64_t q = q0 + t;
        if (q < n_pad) {
            const int32_t e = (int32_t)(run & 0xffffffffll);
            const int32_t row = k == 1 ? (int32_t)q : (int32_t)__umul64hi((uint64_t)q, k_magic);   // q / k, exact
            if (q - (int64_t)row * k == 0) indptr[row] = e;
            if (f[t] & 1) {
                nbr[e] = u[t];
                edge_row[e] = row;
                if (f[t] >> 32) {
                    const int32_t local = n_dst + (int32_t)(run >> 32);
                    src_global[local] = u[t];
                    map[u[t]] = local;     // only the first occurrence writes; later readers never match n_dst + q
                }
            }
            run += f[t];
        }
    }
}

// One-launch form of the two kernels above (tile sums, then assignment), for scans of few tiles: a block publishes its
// tile's sum in a status word, adds up the words of the tiles before it and assigns. (Workgroups are handed out in index order, per
// die in turn: an earlier tile is done, running, or the next to start on its die, and a waiting block never holds
// the slot an earlier tile needs.) A word packs both 31-bit counts and a mark, so it is written and read by one
// 64-bit access at device scope and needs no fence; the words are emptied by the sampling launch before. The wait on
// an earlier tile is bounded: on expiry the block stores the call's id in `fail_flag` and goes on (wrong output, no hang;
// the host reports NO_ERR_TIMEOUT wherever it next reads the blocks' counts).
// ONE_LAUNCH_TILES, where the sampling has the chip to itself: the one-launch form saves a launch (2.3 us and a second read of the
// slots) and pays for the wait and for the count of finished tiles, each a release (a write-back of the die's L2), one after another,
// 10 to 20 ns each. Measured, one launch / two, us of a whole step: scans of 4 and 52 tiles and a split of 5 104.3 / 108.5; of 5, 47 and
// 411 tiles and a split of 48 174.7 / 179.4; sampling alone, scans of 15, 165 and 1005 tiles 87 (walk back in windows of 64) / 75,
// 74 with the first two in one launch. With stores past the L2 in place of the releases the first of these took 107.8.
// Beside a step's products the releases write back what those have in the L2: 210.3 us a step / 209.2, so there it is always two.
constexpr uint32_t ONE_LAUNCH_TILES = 256;
static_assert(ONE_LAUNCH_TILES <= ETHREADS, "a thread a word");
constexpr unsigned long long SCAN_SUM = 1ull;
__device__ __forceinline__ unsigned long long scan_pack(int64_t v) {
    return ((unsigned long long)(v & 0x7fffffffll)) | ((unsigned long long)((v >> 32) & 0x7fffffffll) << 31) | (SCAN_SUM << 62);
}
__device__ __forceinline__ int64_t scan_unpack(unsigned long long w) {
    return (int64_t)(w & 0x7fffffffull) | ((int64_t)((w >> 31) & 0x7fffffffull) << 32);
}

struct ScanWait { unsigned long long* status; int32_t* fail_flag; int32_t flag_value, spin_limit, withhold_first; };

// The sum of the tiles before `tile` (tile < ONE_LAUNCH_TILES, a thread a word), to all threads of the block; publishes this tile's word.
__device__ __forceinline__ int64_t scan_look_back(const ScanWait& w, uint32_t tile, int64_t total, int64_t* prefix_sh /* [ETHREADS / 64] */) {
    // (withhold_first: test aid; tile 0 keeps its word back, so the tile after it must give up its wait)
    if (threadIdx.x == 0 && !(w.withhold_first && tile == 0))
        __hip_atomic_store(&w.status[tile], scan_pack(total), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned long long word = 0ull;
    if (threadIdx.x < tile) {
        int spins = 0;
        while ((word = __hip_atomic_load(&w.status[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0ull) {
            if (++spins > w.spin_limit) {
                __hip_atomic_store(w.fail_flag, w.flag_value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
    }
    int64_t v = scan_unpack(word);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) prefix_sh[threadIdx.x >> 6] = v;
    __syncthreads();
    v = 0;
#pragma unroll
    for (int i = 0; i < ETHREADS / 64; ++i) v += prefix_sh[i];
    return v;
}

// Whether this block is the last of n_tiles to come here (the answer is for thread 0; every block calls once, all its threads). What the
// blocks stored before is then in memory, and load_shared reads it.
__device__ __forceinline__ bool last_tile(unsigned long long* done, uint32_t n_tiles) {
    __syncthreads();
    return threadIdx.x == 0 && __hip_atomic_fetch_add(done, 1ull, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT) == n_tiles - 1;
}
// Accesses past the dies' own caches, for words that the clean-up after an expired wait may write again from another die.
__device__ __forceinline__ void store_shared(int32_t* p, int32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ int32_t load_shared(const int32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

__global__ void __launch_bounds__(ETHREADS) edge_scan_kernel(const int32_t* __restrict__ nbr_pad, int32_t* map,
                                                             const int32_t* d_n_dst, int32_t k, uint64_t k_magic,
                                                             ScanWait wait, int32_t* __restrict__ indptr,
                                                             int32_t* __restrict__ nbr, int32_t* __restrict__ edge_row,
                                                             int32_t* __restrict__ src_global,
                                                             int32_t* counts /* [0]=n_dst (in), [1]=n_src, [2]=nnz */,
                                                             int32_t* csc_cnt, int32_t n_zero, unsigned long long* done,
                                                             SideTasks side) {
    if (blockIdx.x >= side.first_block) { run_side_tasks(side); return; }
    __shared__ int64_t smem[ETHREADS / 64 + 1];
    __shared__ int64_t prefix_sh[ETHREADS / 64];
    __shared__ int cleanup_sh;
    for (int64_t t = (int64_t)blockIdx.x * ETHREADS + threadIdx.x; t < n_zero; t += (int64_t)side.first_block * ETHREADS) csc_cnt[t] = 0;
    const int32_t n_dst = *d_n_dst;
    const int64_t n_pad = (int64_t)n_dst * k;
    if (n_pad == 0) {
        if (blockIdx.x == 0 && threadIdx.x == 0) { indptr[0] = 0; counts[1] = n_dst; counts[2] = 0; }
        return;
    }
    const int64_t base = (int64_t)blockIdx.x * ETILE;
    if (base >= n_pad) return;
    const int64_t q0 = base + (int64_t)threadIdx.x * EITEMS;
    int64_t f[EITEMS];
    int32_t u[EITEMS];
    int64_t s = 0;
#pragma unroll
    for (int t = 0; t < EITEMS; ++t) {
        f[t] = 0;
        u[t] = -1;
        if (q0 + t < n_pad) f[t] = slot_flags(nbr_pad, map, q0 + t, n_dst, &u[t]);
        s += f[t];
    }
    int64_t total;
    int64_t run = block_exclusive_scan<int64_t, ETHREADS>(s, &total, smem);
    const int64_t prefix = scan_look_back(wait, blockIdx.x, total, prefix_sh);
    run += prefix;
    if (threadIdx.x == 0 && base + ETILE >= n_pad) {      // the last tile holds the totals
        const int64_t all = prefix + total;
        const int32_t nnz = (int32_t)(all & 0xffffffffll), n_new = (int32_t)(all >> 32);
        indptr[n_dst] = nnz;
        counts[1] = n_dst + n_new;
        counts[2] = nnz;
    }
#pragma unroll
    for (int t = 0; t < EITEMS; ++t) {
        const int64_t q = q0 + t;
        if (q < n_pad) {
            const int32_t e = (int32_t)(run & 0xffffffffll);
            const int32_t row = k == 1 ? (int32_t)q : (int32_t)__umul64hi((uint64_t)q, k_magic);   // q / k, exact
            if (q - (int64_t)row * k == 0) indptr[row] = e;
            if (f[t] & 1) {
                nbr[e] = u[t];
                edge_row[e] = row;
                if (f[t] >> 32) {
                    const int32_t local = n_dst + (int32_t)(run >> 32);
                    src_global[local] = u[t];
                    map[u[t]] = local;     // only the first occurrence writes; later readers never match n_dst + q
                }
            }
            run += f[t];
        }
    }
    // A wait that expired leaves wrong prefixes behind, and kernels after this one would follow them out of their
    // arrays. The tile that finishes last therefore checks the flag and, if it is raised, turns the hop into a
    // consistent empty block: no edges, no new sources, and no entry of this hop left in the id map.
    const bool last = last_tile(done, (uint32_t)((n_pad + ETILE - 1) / ETILE));
    if (threadIdx.x == 0) cleanup_sh = last && load_shared(wait.fail_flag) == wait.flag_value;
    __syncthreads();
    if (cleanup_sh) {
        for (int64_t q = threadIdx.x; q < n_pad; q += ETHREADS) {
            const int32_t v = nbr_pad[q];
            if (v >= 0 && load_shared(&map[v]) >= n_dst) store_shared(&map[v], EMPTY);      // (entries below n_dst belong to the destinations)
        }
        for (int32_t r = (int32_t)threadIdx.x; r <= n_dst; r += ETHREADS) store_shared(&indptr[r], 0);
        if (threadIdx.x == 0) { store_shared(&counts[1], n_dst); store_shared(&counts[2], 0); }
    }
}

// ---------------------------------------------------------------------------- hot lookup on V^1

struct CacheProbe {
    const int32_t* v1;
    const int32_t* slot_of_vertex;
    const int32_t* version;
    int64_t step;
    int32_t staleness;
    // low word: 1 if the row must be computed; high word: 1 if it is computed AND hot (it will refresh its slot)
    __device__ __forceinline__ int64_t flags(int32_t slot, int32_t ver) const {
        if (slot < 0) return 1;
        const bool hit = ver >= 0 && step - (int64_t)ver <= (int64_t)staleness;
        return hit ? 0 : (1ll + (1ll << 32));
    }
};

// Blocks [0, v1_blocks) probe the cache for a tile of V^1; the remaining blocks write the local indices of
// the hop above (one edge per thread), which must be read out of the id map before the partition re-keys it:
// sharing the launch keeps that pass off the dependency chain of the sampling.
__global__ void __launch_bounds__(ETHREADS) v1_tile_sums_kernel(CacheProbe probe, const int32_t* d_n_v1, int64_t* tile_sums,
                                                                int32_t* __restrict__ probe_slot /* [n]: slot if served from the cache; -1 cold; -2 - slot if hot but to be computed */,
                                                                int32_t* __restrict__ probe_ver /* [n]: the version the probe read (hot vertices) */,
                                                                uint32_t v1_blocks, const int32_t* d_nnz,
                                                                const int32_t* __restrict__ nbr, const int32_t* map,
                                                                int32_t* __restrict__ indices, int32_t* csc_cnt, int32_t* csc_pos,
                                                                SideTasks side) {
    if (blockIdx.x >= side.first_block) { run_side_tasks(side); return; }
    if (blockIdx.x >= v1_blocks) {
        const int32_t e = (int32_t)((blockIdx.x - v1_blocks) * ETHREADS + threadIdx.x);
        if (e >= *d_nnz) return;
        const int32_t local = map[nbr[e]];
        indices[e] = local;
        if (csc_cnt) {      // integer count: order independent
            const int32_t pos = atomicAdd(&csc_cnt[local], 1);
            if (csc_pos) csc_pos[e] = pos;
        }
        return;
    }
    const int64_t n = *d_n_v1;
    const int64_t base = (int64_t)blockIdx.x * ETILE;
    if (base >= n) return;
    __shared__ int64_t smem[ETHREADS / 64];
    const int64_t i0 = base + (int64_t)threadIdx.x * EITEMS;
    // three dependent loads per vertex; each level is issued for all items before the next is needed
    int32_t v[EITEMS], slot[EITEMS], ver[EITEMS];
#pragma unroll
    for (int t = 0; t < EITEMS; ++t) v[t] = i0 + t < n ? probe.v1[i0 + t] : -1;
#pragma unroll
    for (int t = 0; t < EITEMS; ++t) slot[t] = v[t] >= 0 ? probe.slot_of_vertex[v[t]] : -1;
#pragma unroll
    for (int t = 0; t < EITEMS; ++t) ver[t] = slot[t] >= 0 ? probe.version[slot[t]] : -1;
    int64_t s = 0;
#pragma unroll
    for (int t = 0; t < EITEMS; ++t) {
        if (i0 + t < n) {
            const int64_t f = probe.flags(slot[t], ver[t]);
            probe_slot[i0 + t] = (f & 1) ? (slot[t] >= 0 ? -2 - slot[t] : -1) : slot[t];
            probe_ver[i0 + t] = ver[t];
            s += f;
        }
    }
    s = block_sum<int64_t, ETHREADS>(s, smem);
    if (threadIdx.x == 0) tile_sums[blockIdx.x] = s;
}

// Stable split of V^1 into rows to compute and rows served from the cache; re-keys the id map for
// the bottom hop (computed vertex -> its index in the compute list, reusable vertex -> no entry).
__global__ void __launch_bounds__(ETHREADS) v1_partition_kernel(const int32_t* __restrict__ v1, const int32_t* __restrict__ probe_slot,
                                                                const int32_t* __restrict__ probe_ver,
                                                                const int32_t* d_n_v1,
                                                                const int64_t* __restrict__ tile_sums, int32_t summed, int32_t* map,
                                                                int32_t* compute_list, int32_t* compute_pos, int32_t* compute_inv,
                                                                int32_t* refresh_slot, int32_t* hit_pos,
                                                                int32_t* hit_slot, int32_t* extra /* n_compute, n_hit, -, -, n_refresh */,
                                                                int32_t* version, int32_t stamp, int32_t* refresh_old, SideTasks side) {
    if (blockIdx.x >= side.first_block) { run_side_tasks(side); return; }
    // version != NULL: the slot of a hot vertex that will be recomputed is stamped with the step right here (the row
    // itself arrives with the step's layer-1 product), so that the split of the next batch depends on this split only
    // and not on that product; the version it replaces is kept, in case the batch is never trained on.
    __shared__ int64_t smem[ETHREADS / 64 + 1];
    const int64_t n = *d_n_v1;
    const int64_t n_tiles = (n + ETILE - 1) / ETILE;
    if (blockIdx.x == 0) {
        const int64_t s = tiles_before(tile_sums, n_tiles, summed, smem);
        if (threadIdx.x == 0) {
            const int32_t n_compute = (int32_t)(s & 0xffffffffll);
            extra[0] = n_compute;
            extra[1] = (int32_t)n - n_compute;
            extra[4] = (int32_t)(s >> 32);
        }
    }
    const int64_t base = (int64_t)blockIdx.x * ETILE;
    if (base >= n) return;
    const int64_t tile_off = tiles_before(tile_sums, blockIdx.x, summed, smem) & 0xffffffffll;
    const int64_t i0 = base + (int64_t)threadIdx.x * EITEMS;
    int32_t c[EITEMS], slot[EITEMS], vv[EITEMS], pv[EITEMS];
    int64_t s = 0;
#pragma unroll
    for (int t = 0; t < EITEMS; ++t) {
        c[t] = 0;
        slot[t] = -1;
        vv[t] = 0;
        pv[t] = -1;
        if (i0 + t < n) { slot[t] = probe_slot[i0 + t]; vv[t] = v1[i0 + t]; pv[t] = probe_ver[i0 + t]; c[t] = slot[t] < 0 ? 1 : 0; }
        s += c[t];
    }
    int64_t total;
    int64_t run = block_exclusive_scan<int64_t, ETHREADS>(s, &total, smem) + tile_off;
#pragma unroll
    for (int t = 0; t < EITEMS; ++t) {
        const int64_t i = i0 + t;
        if (i < n) {
            const int32_t v = vv[t];
            if (c[t]) {
                compute_pos[run] = (int32_t)i;
                compute_inv[i] = (int32_t)run;
                const int32_t rslot = slot[t] <= -2 ? -2 - slot[t] : -1;
                refresh_slot[run] = rslot;
                if (version && rslot >= 0) {
                    refresh_old[run] = pv[t];      // (what the probe read: nothing writes the versions in between)
                    version[rslot] = stamp;
                }
                compute_list[run] = v;
                map[v] = (int32_t)run;
            } else {
                const int64_t p = i - run;
                hit_pos[p] = (int32_t)i;
                compute_inv[i] = -1;
                hit_slot[p] = slot[t];
                map[v] = EMPTY;
            }
            run += c[t];
        }
    }
}

// One-launch form of the two kernels above (a single-pass scan like edge_scan_kernel, with the same status words,
// emptied by the sampling launch of the hop above, and the same bounded waits): a block probes the cache for its tile,
// publishes the tile's counts, adds up the tiles before it and writes its part of the split from the probe results it
// still holds in registers. The first idx_blocks blocks write the local indices of the hop above out of the id map;
// the split re-keys that map, so every tile block waits, before its map writes, until a counter says that all index
// blocks with work have read (they come first in index order and take two round trips, the probe takes four: the
// wait is there for correctness, not because it is ever long).
constexpr int IDX_ITEMS = 4;      // edges a thread: a quarter of the blocks that count themselves in one word, 10 ns apart
__global__ void __launch_bounds__(ETHREADS) v1_split_kernel(CacheProbe probe, const int32_t* d_n_v1, ScanWait wait,
                                                            uint32_t idx_blocks, const int32_t* d_nnz,
                                                            const int32_t* __restrict__ nbr, int32_t* map,
                                                            int32_t* __restrict__ indices, int32_t* csc_cnt, int32_t* csc_pos,
                                                            unsigned int* idx_done, int32_t* compute_list,
                                                            int32_t* compute_pos, int32_t* compute_inv, int32_t* refresh_slot,
                                                            int32_t* hit_pos, int32_t* hit_slot,
                                                            int32_t* extra /* n_compute, n_hit, -, -, n_refresh */,
                                                            int32_t* version, int32_t stamp, int32_t* refresh_old,
                                                            unsigned long long* done, int32_t csc_len,
                                                            int32_t* above_nnz, int32_t* above_indptr,
                                                            const int32_t* above_n_dst, SideTasks side) {
    if (blockIdx.x >= side.first_block) { run_side_tasks(side); return; }
    if (blockIdx.x < idx_blocks) {
        const int32_t nnz = *d_nnz;
        const int64_t e0 = (int64_t)blockIdx.x * (ETHREADS * IDX_ITEMS) + threadIdx.x;
        if (e0 - threadIdx.x >= nnz) return;      // (whole block: no work, no signal)
        int32_t local[IDX_ITEMS];
#pragma unroll
        for (int t = 0; t < IDX_ITEMS; ++t) local[t] = e0 + t * ETHREADS < nnz ? map[nbr[e0 + t * ETHREADS]] : 0;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // every map read of the block has returned
        __syncthreads();
        if (threadIdx.x == 0) __hip_atomic_fetch_add(idx_done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // (the range check only matters after an expired wait, when the split may have re-keyed the map already)
        int32_t pos[IDX_ITEMS];
        if (csc_cnt)
#pragma unroll
            for (int t = 0; t < IDX_ITEMS; ++t)              // integer count: order independent
                if (e0 + t * ETHREADS < nnz && (uint32_t)local[t] < (uint32_t)csc_len) pos[t] = atomicAdd(&csc_cnt[local[t]], 1);
#pragma unroll
        for (int t = 0; t < IDX_ITEMS; ++t)
            if (e0 + t * ETHREADS < nnz) {
                indices[e0 + t * ETHREADS] = local[t];
                if (csc_pos && (uint32_t)local[t] < (uint32_t)csc_len) csc_pos[e0 + t * ETHREADS] = pos[t];
            }
        return;
    }
    const uint32_t tile = blockIdx.x - idx_blocks;
    __shared__ int64_t smem[ETHREADS / 64 + 1];
    __shared__ int64_t prefix_sh[ETHREADS / 64];
    __shared__ int cleanup_sh;
    const int64_t n = *d_n_v1;
    const int64_t base = (int64_t)tile * ETILE;
    if (base >= n) return;
    const int64_t i0 = base + (int64_t)threadIdx.x * EITEMS;
    // three dependent loads per vertex; each level is issued for all items before the next is needed
    int32_t v[EITEMS], slot[EITEMS], ver[EITEMS];
#pragma unroll
    for (int t = 0; t < EITEMS; ++t) v[t] = i0 + t < n ? probe.v1[i0 + t] : -1;
#pragma unroll
    for (int t = 0; t < EITEMS; ++t) slot[t] = v[t] >= 0 ? probe.slot_of_vertex[v[t]] : -1;
#pragma unroll
    for (int t = 0; t < EITEMS; ++t) ver[t] = slot[t] >= 0 ? probe.version[slot[t]] : -1;
    int64_t f[EITEMS];
    int64_t s = 0;
#pragma unroll
    for (int t = 0; t < EITEMS; ++t) {
        f[t] = i0 + t < n ? probe.flags(slot[t], ver[t]) : 0;
        s += f[t];
    }
    int64_t total;
    int64_t run = block_exclusive_scan<int64_t, ETHREADS>(s, &total, smem);
    const int64_t prefix = scan_look_back(wait, tile, total, prefix_sh);
    if (threadIdx.x == 0) {
        if (base + ETILE >= n) {      // the last tile holds the totals
            const int64_t all = prefix + total;
            const int32_t n_compute = (int32_t)(all & 0xffffffffll);
            extra[0] = n_compute;
            extra[1] = (int32_t)n - n_compute;
            extra[4] = (int32_t)(all >> 32);
        }
        const unsigned int expected = (unsigned int)(((int64_t)*d_nnz + ETHREADS * IDX_ITEMS - 1) / (ETHREADS * IDX_ITEMS));
        int spins = 0;
        while (__hip_atomic_load(idx_done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < expected) {
            if (++spins > wait.spin_limit) { store_shared(wait.fail_flag, wait.flag_value); break; }
            __builtin_amdgcn_s_sleep(1);
        }
    }
    __syncthreads();
    run = (run & 0xffffffffll) + (prefix & 0xffffffffll);
#pragma unroll
    for (int t = 0; t < EITEMS; ++t) {
        const int64_t i = i0 + t;
        if (i < n) {
            const int32_t c = (int32_t)(f[t] & 1);
            if (c) {
                compute_pos[run] = (int32_t)i;
                compute_inv[i] = (int32_t)run;
                const int32_t rslot = slot[t] >= 0 ? slot[t] : -1;       // hot but to be computed
                refresh_slot[run] = rslot;
                if (version && rslot >= 0) {
                    refresh_old[run] = ver[t];
                    version[rslot] = stamp;
                }
                compute_list[run] = v[t];
                map[v[t]] = (int32_t)run;
            } else {
                const int64_t p = i - run;
                hit_pos[p] = (int32_t)i;
                compute_inv[i] = -1;
                hit_slot[p] = slot[t];
                map[v[t]] = EMPTY;
            }
            run += c;
        }
    }
    // After an expired wait the split (and possibly the local indices of the hop above, if the map was re-keyed under
    // their readers) cannot be trusted. The tile that finishes last then leaves a consistent state that no later
    // kernel can follow out of its arrays: nothing to compute, nothing reused, no edges in the hop above, and no
    // entry of V^1 left in the id map. (Versions already stamped stay stamped: the caller is told to invalidate.)
    const bool last = last_tile(done, (uint32_t)((n + ETILE - 1) / ETILE));
    if (threadIdx.x == 0) cleanup_sh = last && load_shared(wait.fail_flag) == wait.flag_value;
    __syncthreads();
    if (cleanup_sh) {
        for (int64_t i = threadIdx.x; i < n; i += ETHREADS) store_shared(&map[probe.v1[i]], EMPTY);
        const int32_t nd = *above_n_dst;
        for (int32_t r = (int32_t)threadIdx.x; r <= nd; r += ETHREADS) above_indptr[r] = 0;
        if (threadIdx.x == 0) { store_shared(&extra[0], 0); store_shared(&extra[1], 0); store_shared(&extra[4], 0); *above_nnz = 0; }
    }
}

__global__ void __launch_bounds__(SIDE_THREADS) side_tasks_kernel(SideTasks side) { run_side_tasks(side); }

// Takes back the stamps of a split whose batch is not trained on.
__global__ void unstamp_kernel(const int32_t* __restrict__ refresh_slot, const int32_t* __restrict__ refresh_old,
                               const int32_t* d_n_compute, int32_t n_cap, int32_t* version) {
    const int32_t n = min(*d_n_compute, n_cap);
    for (int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x); i < n; i += (int32_t)(gridDim.x * blockDim.x)) {
        const int32_t slot = refresh_slot[i];
        if (slot >= 0) version[slot] = refresh_old[i];
    }
}

// ---------------------------------------------------------------------------- host side

static inline int64_t edge_tiles(int64_t n_pad_cap) { int64_t t = ceil_div(n_pad_cap, ETILE); return t < 1 ? 1 : t; }
// words of one scan: a word a tile (status words, or the sums of the two-launch form), then the counter of finished tiles
static inline int64_t scan_words(int64_t n_pad_cap) { return edge_tiles(n_pad_cap) + 1; }
// scans with room for more than OFFSETS_TILES tiles have their sums added up by a launch between the two
static inline int32_t scan_summed(int64_t n_pad_cap, const int32_t* d_n, int32_t k, int64_t* tile_sums, hipStream_t st) {
    if (edge_tiles(n_pad_cap) <= OFFSETS_TILES) return 0;
    hipLaunchKernelGGL(tile_offsets_kernel, dim3(1), dim3(1024), 0, st, d_n, k, tile_sums);
    return 1;
}
static inline bool scan_one_launch(const no_blocks_s* b, int64_t n_pad_cap) { return !b->scan_two_pass && edge_tiles(n_pad_cap) <= ONE_LAUNCH_TILES; }
// does this hop count the edges that leave each source (for its transpose, or for the symmetric normalisation)?
static inline bool counts_sources(const no_blocks_s* b, const HopBuffers& H) { return H.has_csc || b->count_sources; }

// ---- side tasks: what is due, in the order it becomes so

static inline bool side_pending(const no_blocks_s* b) {
    for (int32_t h = 0; h < b->n_layers; ++h) if (b->side_next[h] >= 0) return true;
    return b->wipe_pending || b->rows_pending.table;
}

void side_take(no_blocks_s* b, uint32_t own_blocks, SideTasks* side) {
    side->first_block = own_blocks;
    side->n = 0;
    bool indices_left = false;
    for (int32_t h = 0; h < b->n_layers; ++h) indices_left = indices_left || b->side_next[h] == SIDE_INDICES;
    auto blocks_for = [](int64_t items) { return (uint32_t)std::min<int64_t>(std::max<int64_t>(ceil_div(items, SIDE_THREADS), 1), 8192); };
    for (int32_t h = 0; h < b->n_layers && side->n < MAX_SIDE_TASKS; ++h) {
        HopBuffers& H = b->hop[h];
        const int32_t* cnt = b->counts.p + 4 * h;
        if (b->side_next[h] < 0) continue;
        SideTask& t = side->t[side->n++];
        t = SideTask{};
        t.kind = b->side_next[h];
        t.d_n = cnt + 2;
        t.n_blocks = blocks_for(H.nnz_cap);
        switch (t.kind) {
            case SIDE_INDICES:
                t.in0 = H.nbr_global.p; t.in1 = b->map.p; t.out0 = H.indices.p;
                t.out1 = counts_sources(b, H) ? H.csc_cnt.p : nullptr;
                t.out2 = H.has_csc ? H.csc_dst.p : nullptr;      // (arrivals: the ranking, which writes csc_dst, is two tasks away)
                b->side_next[h] = !H.has_csc ? -1 : H.csc_tiles.p ? SIDE_TILE_SUMS : SIDE_SCAN;
                break;
            case SIDE_TILE_SUMS:
            case SIDE_SCAN:
                t.d_n = cnt + 1; t.d_nnz = cnt + 2; t.n_cap = H.n_src_cap;
                t.n_blocks = (uint32_t)std::max<int64_t>(ceil_div(H.n_src_cap, SIDE_SCAN_TILE), 1);
                t.in0 = H.csc_cnt.p; t.in1 = H.csc_tiles.p;
                t.out0 = t.kind == SIDE_SCAN ? H.csc_indptr.p : H.csc_tiles.p;
                b->side_next[h] = t.kind == SIDE_SCAN ? SIDE_FILL : SIDE_SCAN;
                break;
            case SIDE_FILL:
                t.in0 = H.indices.p; t.in1 = H.csc_indptr.p; t.in2 = H.csc_dst.p; t.out0 = H.csc_fill.p;
                b->side_next[h] = SIDE_RANK;
                break;
            default:
                t.in0 = H.indices.p; t.in1 = H.csc_indptr.p; t.in2 = H.csc_fill.p; t.in3 = H.edge_row.p;
                t.out0 = H.csc_eid.p; t.out1 = H.csc_dst.p;
                b->side_next[h] = -1;
                break;
        }
    }
    if (b->wipe_pending && !indices_left && side->n < MAX_SIDE_TASKS) {
        SideTask& t = side->t[side->n++];
        t = SideTask{};
        t.kind = SIDE_WIPE;
        const HopBuffers& last = b->hop[b->wipe_hop];
        t.d_n = b->counts.p + 4 * b->wipe_hop + 1; t.n_blocks = blocks_for(last.n_src_cap);
        t.in0 = last.src_global.p; t.out0 = b->map.p;
        b->wipe_pending = false;
    }
    if (b->rows_pending.table && side->n < MAX_SIDE_TASKS) {
        SideTask& t = side->t[side->n++];
        t = SideTask{};
        t.kind = SIDE_ROWS;
        const HopBuffers& last = b->hop[b->wipe_hop];
        const SideGather& g = b->rows_pending;
        t.d_n = b->counts.p + 4 * b->wipe_hop; t.n_cap = last.n_dst_cap; t.in0 = last.src_global.p;
        t.table = (const char*)g.table; t.rows_out = (char*)g.out; t.row_bytes = g.row_bytes;
        const uintptr_t mix = (uintptr_t)g.table | (uintptr_t)g.out | (uintptr_t)g.row_bytes;
        t.unit = (mix & 15) == 0 ? 16 : (mix & 7) == 0 ? 8 : (mix & 3) == 0 ? 4 : 2;
        // (8192 wavefronts: the chip's wave slots once)
        t.n_blocks = (uint32_t)std::min<int64_t>(std::max<int64_t>(ceil_div(last.n_dst_cap, SIDE_THREADS / 64), 1), 2048);
        b->rows_pending = SideGather{};
    }
}

int32_t blocks_finish(no_blocks_s* b, hipStream_t st, hipEvent_t done) {
    const hipEvent_t none = nullptr;
    bool recorded = false;
    while (side_pending(b)) {
        SideTasks side;
        side_take(b, 0, &side);
        const hipEvent_t last = side_pending(b) ? nullptr : done;
        NO_LAUNCH_TIMED(side_tasks_kernel, dim3(side.side_blocks()), dim3(SIDE_THREADS), st, none, last, side);
        recorded = last != nullptr;
    }
    if (done && !recorded) NO_HIP_CHECK(hipEventRecord(done, st));
    return launch_status("side tasks");
}

static ScanWait scan_wait(no_blocks_s* b, unsigned long long* status) {
    const ScanWaitDebug dbg = scan_wait_debug();
    return ScanWait{status, b->counts.p + 4 * b->n_layers + 6, b->call_id, dbg.spin_limit, dbg.withhold_first_tile};
}

template <typename RowT>
static int32_t sample_hop(const RowT* rowptr, const int32_t* col, no_blocks_s* b, int32_t h, const int32_t* d_dst,
                          const int32_t* d_n_dst_in, int32_t n_fixed, bool insert_dst, uint32_t key0, uint32_t key1,
                          uint32_t domain, hipStream_t st, int32_t* zero_extra, int32_t extra_status) {
    HopBuffers& H = b->hop[h];
    int32_t* cnt = b->counts.p + 4 * h;              // n_dst, n_src, nnz
    const int32_t k = H.fanout;
    H.d_dst = d_dst;
    H.d_n_dst = cnt;
    int64_t* tile_sums = (int64_t*)b->ws.p;
    const uint32_t c3 = (domain << 8) | (uint32_t)h;
    int32_t* seeds_copy = (h == 0) ? b->seeds.p : nullptr;
    hipEvent_t tev0 = nullptr, tev1 = nullptr;
    if (b->time_hop == h && b->time_ev0) { tev0 = b->time_ev0; tev1 = b->time_ev1; b->time_ev0 = b->time_ev1 = nullptr; b->time_hop = -1; }
    SideTasks side;
    if (tev0) NO_CHECK(blocks_finish(b, st));      // (the timed kernel does its own work only)
#define NO_LAUNCH_SAMPLE(G)                                                                                            \
    side_take(b, (uint32_t)ceil_div(H.n_dst_cap, 256 / G), &side);                                                       \
    NO_LAUNCH_TIMED((sample_rows_kernel<G, RowT>), dim3(side.first_block + side.side_blocks()), dim3(256), st, tev0, tev1, \
                       rowptr, col, d_dst, d_n_dst_in, n_fixed, H.n_dst_cap, k, key0, key1, c3, H.nbr_pad.p,               \
                       H.src_global.p, b->map.p, insert_dst ? 1 : 0, seeds_copy, cnt, (int32_t)b->n_vertices,               \
                       b->counts.p + 4 * b->n_layers + 5, b->call_id, (unsigned long long*)b->ws.p,                          \
                       (int32_t)scan_words(H.nnz_cap) + extra_status, zero_extra, side)
    if (k <= 8) { NO_LAUNCH_SAMPLE(8); }
    else if (k <= 16) { NO_LAUNCH_SAMPLE(16); }
    else if (k <= 32) { NO_LAUNCH_SAMPLE(32); }
    else { NO_LAUNCH_SAMPLE(64); }
#undef NO_LAUNCH_SAMPLE
    const unsigned tiles = (unsigned)edge_tiles(H.nnz_cap);
    const uint64_t k_magic = k > 1 ? (~0ull / (uint64_t)k) + 1ull : 0ull;     // ceil(2^64 / k)
    const int32_t n_zero = counts_sources(b, H) ? H.n_src_cap + 1 : 0;
    side_take(b, tiles, &side);
    if (!scan_one_launch(b, H.nnz_cap)) {
        hipLaunchKernelGGL(edge_tile_sums_kernel, dim3(tiles + side.side_blocks()), dim3(ETHREADS), 0, st, H.nbr_pad.p,
                           (const int32_t*)b->map.p, (const int32_t*)cnt, k, tile_sums, H.csc_cnt.p, n_zero, side);
        const int32_t summed = scan_summed(H.nnz_cap, cnt, k, tile_sums, st);
        side_take(b, tiles, &side);
        hipLaunchKernelGGL(edge_assign_kernel, dim3(tiles + side.side_blocks()), dim3(ETHREADS), 0, st, (const int32_t*)H.nbr_pad.p,
                           b->map.p, (const int32_t*)cnt, k, k_magic, (const int64_t*)tile_sums, summed, H.indptr.p, H.nbr_global.p,
                           H.edge_row.p, H.src_global.p, cnt, side);
    } else {
        hipLaunchKernelGGL(edge_scan_kernel, dim3(tiles + side.side_blocks()), dim3(ETHREADS), 0, st, (const int32_t*)H.nbr_pad.p,
                           b->map.p, (const int32_t*)cnt, k, k_magic, scan_wait(b, (unsigned long long*)b->ws.p), H.indptr.p, H.nbr_global.p,
                           H.edge_row.p, H.src_global.p, cnt, H.csc_cnt.p, n_zero, (unsigned long long*)b->ws.p + tiles, side);
    }
    b->side_next[h] = SIDE_INDICES;
    return launch_status("sample_hop");
}

int32_t sample_blocks_impl(no_graph_s* g, const int32_t* d_seeds, int32_t n_seeds, uint64_t stream_key, uint32_t domain,
                           int32_t n_hops, no_cache_s* cache, int64_t step, no_blocks_s* b, hipStream_t st, bool finish,
                           const SideGather* gather, bool stamp_refresh) {
    // a previous call that was never finished (an error behind it): its rows are nobody's, and its table may be gone
    b->rows_pending = SideGather{};
    NO_CHECK(blocks_finish(b, st));
    b->stamped_cache = nullptr;
    b->call_id = b->call_id % 0x3fffffff + 1;      // flag words written by this call's kernels carry this value
    const int32_t L = b->n_layers;
    int32_t* extra = b->counts.p + 4 * L;     // n_compute, n_hit, -, -, n_refresh
    const uint32_t key0 = (uint32_t)stream_key, key1 = (uint32_t)(stream_key >> 32);
    const int32_t* d_dst = d_seeds;
    const int32_t* d_n = nullptr;
    const bool use_cache = cache != nullptr && L >= 2 && n_hops == L && cache->n_hot > 0;
    b->last_used_cache = use_cache;
    for (int32_t h = 0; h < n_hops; ++h) {
        if (h == L - 1 && use_cache) {
            // split V^1 (= sources of hop L-2) into reusable rows and rows to compute; the same launch writes
            // hop L-2's local indices, which the re-keyed map could no longer give (the hops above have theirs: they went
            // with the sampling of the hop after)
            HopBuffers& P = b->hop[h - 1];
            b->side_next[h - 1] = -1;
            for (int32_t up = 0; up < h - 1; ++up)
                if (b->side_next[up] == SIDE_INDICES) { NO_CHECK(blocks_finish(b, st)); break; }
            SideTasks side;
            CacheProbe probe{d_dst, cache->slot_of_vertex.p, cache->version.p, step, cache->staleness};
            const unsigned tiles = (unsigned)edge_tiles(P.n_src_cap);
            const unsigned idx_blocks = (unsigned)ceil_div(P.nnz_cap, ETHREADS);
            int64_t* tile_sums = (int64_t*)b->ws.p;
            if (scan_one_launch(b, P.n_src_cap)) {
                // (its words, and behind them the counter of index blocks: emptied by the sampling launch of hop L-2, past its own)
                unsigned long long* v1_status = (unsigned long long*)b->ws.p + scan_words(P.nnz_cap);
                const unsigned idx_blocks = (unsigned)ceil_div(P.nnz_cap, ETHREADS * IDX_ITEMS);
                side_take(b, idx_blocks + tiles, &side);
                hipLaunchKernelGGL(v1_split_kernel, dim3(side.first_block + side.side_blocks()), dim3(ETHREADS), 0, st, probe, d_n,
                                   scan_wait(b, v1_status), idx_blocks, (const int32_t*)(b->counts.p + 4 * (h - 1) + 2), (const int32_t*)P.nbr_global.p,
                                   b->map.p, P.indices.p, counts_sources(b, P) ? P.csc_cnt.p : nullptr,
                                   P.has_csc ? P.csc_dst.p : nullptr, (unsigned int*)(v1_status + scan_words(P.n_src_cap)),
                                   b->compute_list.p, b->compute_pos.p, b->compute_inv.p, b->refresh_slot.p, b->hit_pos.p,
                                   b->hit_slot.p, extra, stamp_refresh ? cache->version.p : nullptr, (int32_t)step,
                                   b->refresh_old.p, v1_status + tiles, P.n_src_cap + 1,
                                   b->counts.p + 4 * (h - 1) + 2, P.indptr.p, (const int32_t*)(b->counts.p + 4 * (h - 1)), side);
            } else {
            side_take(b, tiles + idx_blocks, &side);
            hipLaunchKernelGGL(v1_tile_sums_kernel, dim3(side.first_block + side.side_blocks()), dim3(ETHREADS), 0, st, probe, d_n, tile_sums,
                               b->probe_slot.p, b->probe_ver.p, tiles, (const int32_t*)(b->counts.p + 4 * (h - 1) + 2),
                               (const int32_t*)P.nbr_global.p, (const int32_t*)b->map.p, P.indices.p,
                               counts_sources(b, P) ? P.csc_cnt.p : nullptr, P.has_csc ? P.csc_dst.p : nullptr, side);
            const int32_t summed = scan_summed(P.n_src_cap, d_n, 1, tile_sums, st);
            side_take(b, tiles, &side);
            hipLaunchKernelGGL(v1_partition_kernel, dim3(tiles + side.side_blocks()), dim3(ETHREADS), 0, st, d_dst,
                               (const int32_t*)b->probe_slot.p, (const int32_t*)b->probe_ver.p, d_n, (const int64_t*)tile_sums, summed, b->map.p, b->compute_list.p, b->compute_pos.p, b->compute_inv.p, b->refresh_slot.p, b->hit_pos.p,
                               b->hit_slot.p, extra, stamp_refresh ? cache->version.p : nullptr, (int32_t)step,
                               b->refresh_old.p, side);
            }
            if (P.has_csc) b->side_next[h - 1] = P.csc_tiles.p ? SIDE_TILE_SUMS : SIDE_SCAN;
            b->stamped_cache = stamp_refresh ? cache : nullptr;
            b->stamped_uid = cache->uid;
            b->stamped_contents = cache->contents;
            d_dst = b->compute_list.p;
            d_n = extra + 0;
        }
        int32_t* zero_extra = h == 0 && !use_cache ? extra : nullptr;
        // the hop above the bottom one also empties the status words of the V^1 split that follows it
        const int32_t extra_status = (use_cache && h == L - 2 && scan_one_launch(b, b->hop[h].n_src_cap))
                                         ? (int32_t)scan_words(b->hop[h].n_src_cap) + 1 : 0;
        if (g->rowptr_bits == 64)
            NO_CHECK(sample_hop<int64_t>(g->rowptr64.p, g->col.p, b, h, d_dst, d_n, n_seeds, h == 0, key0, key1, domain, st,
                                         zero_extra, extra_status));
        else
            NO_CHECK(sample_hop<int32_t>(g->rowptr32.p, g->col.p, b, h, d_dst, d_n, n_seeds, h == 0, key0, key1, domain, st,
                                         zero_extra, extra_status));
        d_dst = b->hop[h].src_global.p;
        d_n = b->counts.p + 4 * h + 1;
    }
    b->wipe_pending = true;
    b->wipe_hop = n_hops - 1;
    if (gather && gather->table) b->rows_pending = *gather;
    NO_CHECK(launch_status("sample_blocks"));
    return finish ? blocks_finish(b, st) : NO_OK;
}

int32_t blocks_unstamp(no_blocks_s* b, hipStream_t st) {
    if (!b->stamped_cache) return NO_OK;
    // nothing to restore when the cache was destroyed since (its address may already name another cache), or when all
    // its versions were replaced (refresh commit: the stamps sit in the copy that is now the pending one; invalidate)
    if (!cache_is_live(b->stamped_cache) || b->stamped_cache->uid != b->stamped_uid ||
        b->stamped_cache->contents != b->stamped_contents) {
        b->stamped_cache = nullptr;
        return NO_OK;
    }
    const int32_t L = b->n_layers;
    const int32_t cap = b->hop[L - 1].n_dst_cap;
    hipLaunchKernelGGL(unstamp_kernel, dim3((unsigned)std::min<int64_t>(ceil_div(cap, 256), 1024)), dim3(256), 0, st,
                       (const int32_t*)b->refresh_slot.p, (const int32_t*)b->refresh_old.p, (const int32_t*)(b->counts.p + 4 * L), cap,
                       b->stamped_cache->version.p);
    b->stamped_cache = nullptr;
    return launch_status("blocks_unstamp");
}

int32_t blocks_create_impl(no_graph_s* g, int32_t n_seeds_cap, const int32_t* fanouts, int32_t n_layers,
                           bool build_csc, no_blocks_s** out) {
    *out = nullptr;
    no_blocks_s* b = new no_blocks_s();
    struct Guard { no_blocks_s* b; ~Guard() { if (b) { b->release(); delete b; } } } guard{b};
    b->n_layers = n_layers;
    b->n_seeds_cap = n_seeds_cap;
    b->n_vertices = g->n_vertices;
    b->build_csc = build_csc;
    int64_t dst_cap = n_seeds_cap;
    int64_t max_pad = 1, max_src = 1;
    for (int32_t h = 0; h < n_layers; ++h) {
        HopBuffers& H = b->hop[h];
        // Different vertices are V at most, but seeds that are not different ones (several outside [0, V), all read as vertex 0) keep
        // their places among the sources of every hop. (Where 32 bits number no more slots than those of V destinations there is no
        // such room.)
        if (dst_cap > g->n_vertices && dst_cap * (fanouts[h] + 1) >= (1ll << 31) - 1) dst_cap = g->n_vertices;
        const int64_t nnz_cap = dst_cap * fanouts[h];
        const int64_t src_cap = std::min(dst_cap + nnz_cap, g->n_vertices + n_seeds_cap);
        NO_REQUIRE(nnz_cap + dst_cap < (1ll << 31) - 1, NO_ERR_OVERFLOW, "blocks: hop %d capacity exceeds int32", h);
        H.fanout = fanouts[h];
        H.n_dst_cap = (int32_t)dst_cap;
        H.nnz_cap = (int32_t)nnz_cap;
        H.n_src_cap = (int32_t)src_cap;
        H.has_csc = build_csc && h < n_layers - 1;
        NO_CHECK(H.src_global.alloc((size_t)src_cap));
        NO_CHECK(H.indptr.alloc((size_t)dst_cap + 1));
        NO_CHECK(H.nbr_pad.alloc((size_t)nnz_cap));
        NO_CHECK(H.nbr_global.alloc((size_t)nnz_cap));
        NO_CHECK(H.indices.alloc((size_t)nnz_cap));
        NO_CHECK(H.edge_row.alloc((size_t)nnz_cap));
        NO_CHECK(H.csc_cnt.alloc((size_t)src_cap + 1));       // (every hop: the bottom hop's counts serve the symmetric normalisation)
        if (H.has_csc) {
            NO_CHECK(H.csc_indptr.alloc((size_t)src_cap + 1));
            NO_CHECK(H.csc_dst.alloc((size_t)nnz_cap));
            NO_CHECK(H.csc_eid.alloc((size_t)nnz_cap));
            NO_CHECK(H.csc_fill.alloc((size_t)nnz_cap));
            if (src_cap > SIDE_SCAN_ONE_LAUNCH) NO_CHECK(H.csc_tiles.alloc((size_t)ceil_div(src_cap, SIDE_SCAN_TILE)));
        }
        if (nnz_cap > max_pad) max_pad = nnz_cap;
        if (src_cap > max_src) max_src = src_cap;
        dst_cap = src_cap;
    }
    NO_CHECK(b->counts.alloc((size_t)4 * n_layers + 8));
    NO_HIP_CHECK(hipMemset(b->counts.p, 0, ((size_t)4 * n_layers + 8) * 4));
    NO_CHECK(b->seeds.alloc((size_t)n_seeds_cap));
    NO_CHECK(b->map.alloc((size_t)g->n_vertices));
    NO_CHECK(fill_i32(b->map.p, EMPTY, g->n_vertices, nullptr));
    const int64_t max_items = max_pad > max_src ? max_pad : max_src;
    NO_CHECK(b->ws.alloc((size_t)(2 * scan_words(max_items + 1) + 8) * sizeof(int64_t)));      // the words of two scans, and a counter
    if (n_layers >= 2) {
        size_t v1_cap = (size_t)b->hop[n_layers - 2].n_src_cap;
        NO_CHECK(b->compute_list.alloc(v1_cap));
        NO_CHECK(b->compute_pos.alloc(v1_cap));
        NO_CHECK(b->compute_inv.alloc(v1_cap));
        NO_CHECK(b->refresh_slot.alloc(v1_cap));
        NO_CHECK(b->refresh_old.alloc(v1_cap));
        NO_CHECK(b->hit_pos.alloc(v1_cap));
        NO_CHECK(b->hit_slot.alloc(v1_cap));
        NO_CHECK(b->probe_slot.alloc(v1_cap));
        NO_CHECK(b->probe_ver.alloc(v1_cap));
    }
    NO_HIP_CHECK(hipDeviceSynchronize());
    guard.b = nullptr;
    *out = b;
    return NO_OK;
}

void fill_block_view(const no_blocks_s* b, int32_t h, no_block_view* v) {
    const HopBuffers& H = b->hop[h];
    const int32_t* cnt = b->counts.p + 4 * h;
    const int32_t* extra = b->counts.p + 4 * b->n_layers;
    v->n_dst_cap = H.n_dst_cap;
    v->n_src_cap = H.n_src_cap;
    v->nnz_cap = H.nnz_cap;
    v->d_n_dst = cnt;
    v->d_n_src = cnt + 1;
    v->d_nnz = cnt + 2;
    v->d_dst_global = H.src_global.p;     // the first n_dst sources are the destinations
    v->d_src_global = H.src_global.p;
    v->d_indptr = H.indptr.p;
    v->d_nbr_global = H.nbr_global.p;
    v->d_indices = H.indices.p;
    v->d_csc_indptr = H.has_csc ? H.csc_indptr.p : nullptr;
    v->d_csc_dst = H.has_csc ? H.csc_dst.p : nullptr;
    v->d_csc_eid = H.has_csc ? H.csc_eid.p : nullptr;
    const bool bottom_cached = (h == b->n_layers - 1) && b->last_used_cache;
    v->d_compute_pos = bottom_cached ? b->compute_pos.p : nullptr;
    v->d_hit_pos = bottom_cached ? b->hit_pos.p : nullptr;
    v->d_hit_slot = bottom_cached ? b->hit_slot.p : nullptr;
    v->d_n_compute = bottom_cached ? extra + 0 : nullptr;
    v->d_n_hit = bottom_cached ? extra + 1 : nullptr;
}

}  // namespace no

using namespace no;

static int32_t check_fanouts(const int32_t* f, int32_t n_layers, const char* who) {
    NO_REQUIRE(f != nullptr, NO_ERR_INVALID_ARG, "%s: fanouts is NULL", who);
    NO_REQUIRE(n_layers >= 1 && n_layers <= NO_MAX_LAYERS, NO_ERR_INVALID_ARG, "%s: n_layers must be in [1, %d]", who,
               NO_MAX_LAYERS);
    for (int32_t h = 0; h < n_layers; ++h)
        NO_REQUIRE(f[h] >= 1 && f[h] <= NO_MAX_FANOUT, NO_ERR_INVALID_ARG, "%s: fanout[%d] must be in [1, %d]", who, h,
                   NO_MAX_FANOUT);
    return NO_OK;
}

extern "C" int32_t no_blocks_create(no_graph_t g, int32_t n_seeds_cap, const int32_t* h_fanouts, int32_t n_layers,
                                    no_blocks_t* out) {
    clear_error();
    NO_REQUIRE(out != nullptr, NO_ERR_INVALID_ARG, "no_blocks_create: out is NULL");
    *out = nullptr;
    NO_REQUIRE(g != nullptr, NO_ERR_INVALID_ARG, "no_blocks_create: graph is NULL");
    NO_REQUIRE(n_seeds_cap >= 1, NO_ERR_INVALID_ARG, "no_blocks_create: n_seeds_cap must be positive");
    NO_REQUIRE(n_seeds_cap <= g->n_vertices, NO_ERR_INVALID_ARG, "no_blocks_create: more seeds than vertices");
    NO_CHECK(check_fanouts(h_fanouts, n_layers, "no_blocks_create"));
    NO_CHECK(blocks_create_impl(g, n_seeds_cap, h_fanouts, n_layers, true, out));
    handle_created();
    return NO_OK;
}

extern "C" int32_t no_sample_blocks(no_graph_t g, const int32_t* d_seeds, int32_t n_seeds, uint64_t seed, int64_t step,
                                    no_cache_t cache, no_blocks_t blocks, void* stream) {
    clear_error();
    NO_REQUIRE(g && blocks && d_seeds, NO_ERR_INVALID_ARG, "no_sample_blocks: NULL argument");
    NO_REQUIRE(n_seeds >= 1, NO_ERR_INVALID_ARG, "no_sample_blocks: n_seeds must be positive");
    NO_REQUIRE(n_seeds <= blocks->n_seeds_cap, NO_ERR_CAPACITY, "no_sample_blocks: %d seeds exceed the capacity %d",
               n_seeds, blocks->n_seeds_cap);
    NO_REQUIRE(blocks->n_vertices == g->n_vertices, NO_ERR_INVALID_ARG, "no_sample_blocks: blocks belong to another graph");
    NO_REQUIRE(step >= 0, NO_ERR_INVALID_ARG, "no_sample_blocks: step must be >= 0");
    NO_REQUIRE(!cache || cache->n_vertices == g->n_vertices, NO_ERR_INVALID_ARG,
               "no_sample_blocks: cache belongs to another graph");
    return sample_blocks_impl(g, d_seeds, n_seeds, seed + (uint64_t)step, 0u, blocks->n_layers, cache, step, blocks,
                              (hipStream_t)stream);
}

extern "C" int32_t no_blocks_view(no_blocks_t blocks, int32_t hop, no_block_view* out) {
    clear_error();
    NO_REQUIRE(blocks && out, NO_ERR_INVALID_ARG, "no_blocks_view: NULL argument");
    NO_REQUIRE(hop >= 0 && hop < blocks->n_layers, NO_ERR_INVALID_ARG, "no_blocks_view: hop out of range");
    fill_block_view(blocks, hop, out);
    // the capacities for unique seeds (the arrays have room for others: blocks_create_impl)
    const int32_t V = (int32_t)blocks->n_vertices;
    if (out->n_dst_cap > V) {
        out->nnz_cap = V * blocks->hop[hop].fanout;
        out->n_dst_cap = V;
    }
    out->n_src_cap = std::min(out->n_src_cap, V);
    return NO_OK;
}

extern "C" int32_t no_blocks_sizes(no_blocks_t blocks, void* stream, int32_t* h_sizes) {
    clear_error();
    NO_REQUIRE(blocks && h_sizes, NO_ERR_INVALID_ARG, "no_blocks_sizes: NULL argument");
    const int32_t L = blocks->n_layers;
    int32_t tmp[4 * NO_MAX_LAYERS + 8];
    NO_HIP_CHECK(hipMemcpyAsync(tmp, blocks->counts.p, ((size_t)4 * L + 8) * 4, hipMemcpyDeviceToHost, (hipStream_t)stream));
    NO_HIP_CHECK(hipStreamSynchronize((hipStream_t)stream));
    for (int32_t h = 0; h < L; ++h) {
        h_sizes[4 * h + 0] = tmp[4 * h + 0];
        h_sizes[4 * h + 1] = tmp[4 * h + 1];
        h_sizes[4 * h + 2] = tmp[4 * h + 2];
        h_sizes[4 * h + 3] = (h == L - 1 && blocks->last_used_cache) ? tmp[4 * L + 1] : 0;
    }
    const int32_t id = blocks->call_id;
    NO_REQUIRE(id == 0 || tmp[4 * L + 6] != id, NO_ERR_TIMEOUT,
               "no_blocks_sizes: a scan of the last sampling call gave up waiting for an earlier tile; the blocks are invalid");
    NO_REQUIRE(id == 0 || tmp[4 * L + 5] != id, NO_ERR_OUT_OF_RANGE,
               "no_blocks_sizes: the last sampling call met a seed id outside [0, V) (read as vertex 0)");
    return NO_OK;
}

namespace no {
static ScanWaitDebug g_scan_wait_debug{1 << 20, 0};
ScanWaitDebug scan_wait_debug() { return g_scan_wait_debug; }
}  // namespace no

extern "C" int32_t no_debug_scan_wait(int32_t spin_limit, int32_t withhold_first_tile) {
    clear_error();
    NO_REQUIRE(spin_limit >= 0, NO_ERR_INVALID_ARG, "no_debug_scan_wait: spin_limit must be >= 0");
    g_scan_wait_debug.spin_limit = spin_limit > 0 ? spin_limit : (1 << 20);
    g_scan_wait_debug.withhold_first_tile = withhold_first_tile ? 1 : 0;
    return NO_OK;
}

extern "C" int32_t no_blocks_destroy(no_blocks_t blocks) {
    clear_error();
    if (!blocks) return NO_OK;
    blocks->release();
    delete blocks;
    handle_destroyed();
    return NO_OK;
}
