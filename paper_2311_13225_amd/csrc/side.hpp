// Side tasks of a sampling call: the parts of it that no later hop waits for. They are the local indices of a hop, its transpose
// and, at the end, the wipe of the id map and the dense copy of the bottom destinations' rows. They run as extra blocks
// at the end of the grids of the launches that follow, the next hop's sampling and compaction first, then the layer
// aggregations, each in a launch after the one it depends on.
//
// Why not on a stream of their own: a wait for another stream's event costs the enqueuing thread 11-12 us (a launch 3 us),
// and a step had up to seven of them, more than its small kernels take on the GPU. Extra blocks cost nothing to enqueue and
// fill compute units that a hop's own kernels, bound by a few dependent memory round trips, leave idle.
#pragma once
#include "primitives.hpp"

namespace no {

enum SideKind : int32_t {
    SIDE_INDICES = 0,     // indices[e] = map[nbr[e]]; counts per source and the edge's arrival among its source's edges
    SIDE_TILE_SUMS,       // (large hops only) tile sums of the per-source counts
    SIDE_SCAN,            // exclusive scan of the counts: column pointers of the transpose
    SIDE_FILL,            // every edge into its column, in order of arrival
    SIDE_RANK,            // columns into ascending edge order
    SIDE_WIPE,            // empty the id map again
    SIDE_ROWS,            // dense copy of table rows
};

struct SideTask {
    int32_t kind = 0;
    uint32_t n_blocks = 0;
    const int32_t* d_n = nullptr;         // items (edges, sources, rows)
    const int32_t* d_nnz = nullptr;       // scans: edges of the hop (0 after a failed scan: the columns are empty)
    int32_t n_cap = 0;
    const int32_t* in0 = nullptr; const int32_t* in1 = nullptr; const int32_t* in2 = nullptr; const int32_t* in3 = nullptr;
    int32_t* out0 = nullptr; int32_t* out1 = nullptr; int32_t* out2 = nullptr;
    const char* table = nullptr; char* rows_out = nullptr; int32_t row_bytes = 0; int32_t unit = 0;      // SIDE_ROWS
};

// By value in a kernel's arguments. first_block = blocks of the launch's own work (kernels use it in place of gridDim.x).
constexpr int MAX_SIDE_TASKS = 4;
struct SideTasks {
    uint32_t first_block = 0;
    int32_t n = 0;
    SideTask t[MAX_SIDE_TASKS];
    uint32_t side_blocks() const { uint32_t b = 0; for (int i = 0; i < n; ++i) b += t[i].n_blocks; return b; }
};

// In its place for kernels whose register budget has no room for the tasks' code: launches without any.
struct NoSideTasks { uint32_t first_block = 0; };
__device__ __forceinline__ void run_side_tasks(const NoSideTasks&) {}

constexpr int SIDE_THREADS = 256;
constexpr int SIDE_SCAN_ITEMS = 8, SIDE_SCAN_TILE = SIDE_THREADS * SIDE_SCAN_ITEMS;
// Up to this many sources (by capacity: the hop's chain of tasks is laid down before any count is known) a scan block adds up
// all counts before its tile by itself (at most 8 round trips of eight 16-byte loads a thread, 4 us for the last block); above, a
// launch of tile sums goes first.
constexpr int32_t SIDE_SCAN_ONE_LAUNCH = 65536;

__device__ __forceinline__ int32_t sum4(const int4& v) { return (v.x + v.y) + (v.z + v.w); }

__device__ __forceinline__ void side_scan(const SideTask& t, uint32_t block) {
    __shared__ int32_t smem[SIDE_THREADS / 64 + 1];
    const int32_t n = min(*t.d_n, t.n_cap);
    const bool empty = *t.d_nnz == 0;
    const int32_t* cnt = t.in0;
    const int32_t base = (int32_t)block * SIDE_SCAN_TILE;
    if (n == 0 && block == 0 && threadIdx.x == 0) t.out0[0] = 0;
    if (base >= n) return;
    int32_t before = 0;
    if (!empty) {
        if (t.in1) {
            for (int32_t i = (int32_t)threadIdx.x; i < (int32_t)block; i += SIDE_THREADS) before += t.in1[i];
        } else {
            const int4* c4 = reinterpret_cast<const int4*>(cnt);      // (a tile is 512 vectors: whole rounds of two)
            int32_t i = (int32_t)threadIdx.x;
            const int32_t n4 = base / 4;
            for (; i + 7 * SIDE_THREADS < n4; i += 8 * SIDE_THREADS) {
                int4 v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = c4[i + j * SIDE_THREADS];
#pragma unroll
                for (int j = 0; j < 8; ++j) before += sum4(v[j]);
            }
            for (; i < n4; i += SIDE_THREADS) before += sum4(c4[i]);
        }
    }
    const int32_t i0 = base + (int32_t)threadIdx.x * SIDE_SCAN_ITEMS;
    int32_t v[SIDE_SCAN_ITEMS], s = 0;
#pragma unroll
    for (int k = 0; k < SIDE_SCAN_ITEMS; ++k) {
        v[k] = !empty && i0 + k < n ? cnt[i0 + k] : 0;
        s += v[k];
    }
    before = block_sum<int32_t, SIDE_THREADS>(before, smem);
    int32_t total;
    int32_t run = block_exclusive_scan<int32_t, SIDE_THREADS>(s, &total, smem) + before;
#pragma unroll
    for (int k = 0; k < SIDE_SCAN_ITEMS; ++k) {
        if (i0 + k < n) t.out0[i0 + k] = run;
        run += v[k];
        if (i0 + k == n - 1) t.out0[n] = run;
    }
}

__device__ __forceinline__ void side_tile_sums(const SideTask& t, uint32_t block) {
    __shared__ int32_t smem[SIDE_THREADS / 64];
    const int32_t n = min(*t.d_n, t.n_cap), base = (int32_t)block * SIDE_SCAN_TILE;
    if (base >= n) return;
    const int32_t i0 = base + (int32_t)threadIdx.x * SIDE_SCAN_ITEMS;
    int32_t s = 0;
#pragma unroll
    for (int k = 0; k < SIDE_SCAN_ITEMS; ++k)
        if (i0 + k < n) s += t.in0[i0 + k];
    s = block_sum<int32_t, SIDE_THREADS>(s, smem);
    if (threadIdx.x == 0) t.out0[block] = s;
}

// Every edge finds its rank among the edges of its column; columns are short (a source is sampled by
// few destinations), so the quadratic work is small and needs no sort network or shared memory.
__device__ __forceinline__ void side_rank(const SideTask& t, int32_t e) {
    const int32_t u = t.in0[e], row = t.in3[e];
    const int32_t b = t.in1[u], len = t.in1[u + 1] - b;
    int32_t r = 0;
    if (len > 1) {
        const int32_t* col = t.in2 + b;
        int32_t i = 0;
        for (; i + 8 <= len; i += 8) {       // independent loads: eight compares in flight
            const int32_t x0 = col[i], x1 = col[i + 1], x2 = col[i + 2], x3 = col[i + 3];
            const int32_t x4 = col[i + 4], x5 = col[i + 5], x6 = col[i + 6], x7 = col[i + 7];
            r += (x0 < e) + (x1 < e) + (x2 < e) + (x3 < e) + (x4 < e) + (x5 < e) + (x6 < e) + (x7 < e);
        }
        for (; i < len; ++i) r += col[i] < e ? 1 : 0;
    }
    t.out0[b + r] = e;
    t.out1[b + r] = row;
}

template <typename V>
__device__ __forceinline__ void side_rows(const SideTask& t, uint32_t block) {
    const int32_t n = min(*t.d_n, t.n_cap), units = t.row_bytes / (int32_t)sizeof(V), lane = lane_id();
    const int32_t n_waves = (int32_t)t.n_blocks * (SIDE_THREADS / 64);
    for (int32_t r = (int32_t)(block * (SIDE_THREADS / 64) + threadIdx.x / 64); r < n; r += n_waves) {
        const V* src = reinterpret_cast<const V*>(t.table + (int64_t)t.in0[r] * t.row_bytes);
        V* dst = reinterpret_cast<V*>(t.rows_out + (int64_t)r * t.row_bytes);
        for (int32_t ub = lane; ub < units; ub += 4 * 64) {      // (past the end: the last unit again, not stored)
            const int32_t u1 = ub + 64, u2 = ub + 128, u3 = ub + 192, last = units - 1;
            const V v0 = src[ub], v1 = src[min(u1, last)], v2 = src[min(u2, last)], v3 = src[min(u3, last)];
            dst[ub] = v0;
            if (u1 < units) dst[u1] = v1;
            if (u2 < units) dst[u2] = v2;
            if (u3 < units) dst[u3] = v3;
        }
    }
}

// The work of a block of the launch's tail (blockIdx.x >= side.first_block); blocks of SIDE_THREADS threads.
__device__ __forceinline__ void run_side_tasks(const SideTasks& side) {
    uint32_t block = blockIdx.x - side.first_block;
    int i = 0;
    while (i < side.n - 1 && block >= side.t[i].n_blocks) block -= side.t[i++].n_blocks;
    const SideTask& t = side.t[i];
    const int32_t first = (int32_t)(block * SIDE_THREADS + threadIdx.x), stride = (int32_t)(t.n_blocks * SIDE_THREADS);
    switch (t.kind) {
        case SIDE_INDICES: {
            const int32_t n = *t.d_n;
            for (int32_t e = first; e < n; e += stride) {
                const int32_t local = t.in1[t.in0[e]];
                t.out0[e] = local;
                if (t.out1) {      // integer count: order independent
                    const int32_t pos = atomicAdd(&t.out1[local], 1);
                    if (t.out2) t.out2[e] = pos;
                }
            }
            break;
        }
        case SIDE_TILE_SUMS: side_tile_sums(t, block); break;
        case SIDE_SCAN: side_scan(t, block); break;
        case SIDE_FILL: {
            const int32_t n = *t.d_n;
            for (int32_t e = first; e < n; e += stride) t.out0[t.in1[t.in0[e]] + t.in2[e]] = e;
            break;
        }
        case SIDE_RANK: {
            const int32_t n = *t.d_n;
            for (int32_t e = first; e < n; e += stride) side_rank(t, e);
            break;
        }
        case SIDE_WIPE: {
            const int32_t n = *t.d_n;
            for (int32_t s = first; s < n; s += stride) t.out0[t.in0[s]] = EMPTY;
            break;
        }
        case SIDE_ROWS:
            if (t.unit == 16) side_rows<uint4>(t, block);
            else if (t.unit == 8) side_rows<uint2>(t, block);
            else if (t.unit == 4) side_rows<uint32_t>(t, block);
            else side_rows<uint16_t>(t, block);
            break;
        default: break;
    }
}

}  // namespace no
