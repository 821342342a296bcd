// no_build_csr: COO -> in-neighbour CSR on the device (input G(V,E) of Algorithm 1; rows are
// the N_in(v) of Eq. 1). A stable radix sort by (dst, src) gives rows ascending by
// src with duplicates kept; the row pointers are looked up in the sorted destinations.
#include <algorithm>
#include "primitives.hpp"
#include "radix.hpp"
#include "handles.hpp"

namespace no {

// The caller's edge list as the first pass of the sort reads it: the pair of edge i is (src, dst), and with both directions
// asked for (i >= n_in) edge i - n_in the other way round. Its counting launch also checks both ends of every edge.
template <typename IdT>
struct EdgeSource {
    const IdT* src; const IdT* dst; int64_t n_in, n_vertices; int32_t* bad;
    __device__ __forceinline__ uint32_t key(int64_t i) const { return (uint32_t)(i < n_in ? src[i] : dst[i - n_in]); }
    __device__ __forceinline__ uint32_t val(int64_t i) const { return (uint32_t)(i < n_in ? dst[i] : src[i - n_in]); }
    __device__ __forceinline__ void keys_checked(int64_t i, int here, uint32_t (&k)[RS_ITEMS]) const {
        if (i + here <= n_in) {
            IdT s[RS_ITEMS], d[RS_ITEMS];
            load_run(src, i, here, s);
            load_run(dst, i, here, d);
            bool wrong = false;
#pragma unroll
            for (int q = 0; q < RS_ITEMS; ++q) {      // (past `here` the ids read as 0)
                wrong |= s[q] < 0 || (int64_t)s[q] >= n_vertices || d[q] < 0 || (int64_t)d[q] >= n_vertices;
                k[q] = (uint32_t)s[q];
            }
            if (wrong) *bad = 1;
        } else if (i >= n_in) {                       // the other direction: already checked
            IdT d[RS_ITEMS];
            load_run(dst, i - n_in, here, d);
#pragma unroll
            for (int q = 0; q < RS_ITEMS; ++q) k[q] = (uint32_t)d[q];
        } else {
            for (int q = 0; q < RS_ITEMS; ++q) {
                k[q] = q < here ? key(i + q) : 0u;
                if (i + q < n_in && q < here) {
                    const IdT s = src[i + q], d = dst[i + q];
                    if (s < 0 || (int64_t)s >= n_vertices || d < 0 || (int64_t)d >= n_vertices) *bad = 1;
                }
            }
        }
    }
};

// The passes over the number (destination, source), `bits` bits each half. Their count is the least for the whole number:
// an odd one has a digit that lies across both halves (22 bits each, 124 M pairs: 5 passes of 9 bits in 2.9 ms instead of
// twice 3 of 8 bits in 3.7 ms; the digit across costs its pass 0.15 ms, since the counts and the order need both words).
struct SortPlan {
    int bits, passes, width;
    bool across;
    explicit SortPlan(int bits_) : bits(std::max(1, bits_)) {
        passes = std::max(2, radix_passes(2 * bits));       // (the first one reads sources only)
        across = passes % 2 != 0;
        width = radix_digit_bits(across ? 2 * bits : bits);
    }
};

// rowptr[v] = number of entries of the sorted list below v, v in [0, V]. A block looks up the two ends of its 256 vertices
// (a wavefront each, 64 probes a step: 5 dependent reads for 10^8 entries instead of 27) and every thread searches between
// them: the reads of a block stay within a few lines, and nothing is counted edge by edge (one atomic per edge took 6.7 ms
// on 124 M edges: popular vertices queue up on one word).
template <typename RowT>
__global__ void __launch_bounds__(256) rowptr_kernel(const uint32_t* __restrict__ sorted_dst, int64_t n, int64_t n_vertices,
                                                     RowT* __restrict__ rowptr) {
    __shared__ int64_t ends[2];
    const int64_t v0 = (int64_t)blockIdx.x * 256, v = v0 + threadIdx.x;
    const int wave = (int)(threadIdx.x >> 6), lane = lane_id();
    if (wave < 2) {
        const int64_t x = v0 + 256 * (int64_t)wave;
        int64_t lo = 0, hi = n;                        // the answer lies in [lo, hi]
        while (lo < hi) {
            const int64_t step = (hi - lo + 63) / 64, at = lo + step * (lane + 1) - 1;      // lane l probes the last entry of its part
            const uint64_t m = __ballot(at < hi ? (int64_t)sorted_dst[at] < x : false);
            const int parts = __popcll(m);                              // parts that lie wholly below x
            lo = min(hi, lo + step * parts);
            hi = min(hi, lo + step - 1);                                // the next part's last entry is not below x (or is not there)
        }
        if (lane == 0) ends[wave] = lo;
    }
    __syncthreads();
    if (v > n_vertices) return;
    int64_t lo = ends[0], hi = ends[1];
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo) / 2;
        if ((int64_t)sorted_dst[mid] < v) lo = mid + 1; else hi = mid;
    }
    rowptr[v] = (RowT)lo;
}

// NO_CSR_DEDUP: entry i of the (dst, src)-sorted edge list is kept iff it differs from entry i - 1
__global__ void mark_first_of_run_kernel(const uint32_t* dst, const uint32_t* src, int64_t n, int32_t* keep) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) keep[i] = (i == 0 || dst[i] != dst[i - 1] || src[i] != src[i - 1]) ? 1 : 0;
}

__global__ void compact_edges_kernel(const uint32_t* dst, const uint32_t* src, const int32_t* keep, const int32_t* pos,
                                     int64_t n, int32_t* col_out, uint32_t* dst_out) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride)
        if (keep[i]) {
            col_out[pos[i]] = (int32_t)src[i];
            dst_out[pos[i]] = dst[i];
        }
}

}  // namespace no

using namespace no;

extern "C" int32_t no_build_csr(const void* src, const void* dst, int64_t n_edges_in, int64_t n_vertices,
                                int32_t rowptr_bits, uint32_t flags, void* stream, no_graph_t* out) {
    clear_error();
    NO_REQUIRE(out != nullptr, NO_ERR_INVALID_ARG, "no_build_csr: out is NULL");
    *out = nullptr;
    NO_REQUIRE(n_vertices > 0 && n_edges_in >= 0, NO_ERR_INVALID_ARG, "no_build_csr: need n_vertices > 0, n_edges >= 0");
    NO_REQUIRE(n_edges_in == 0 || (src && dst), NO_ERR_INVALID_ARG, "no_build_csr: src/dst is NULL");
    NO_REQUIRE(rowptr_bits == 32 || rowptr_bits == 64, NO_ERR_INVALID_ARG, "no_build_csr: rowptr_bits must be 32 or 64");
    NO_REQUIRE((flags & ~(uint32_t)(NO_CSR_INPUT_ON_DEVICE | NO_CSR_IDS_64 | NO_CSR_SYMMETRISE | NO_CSR_DEDUP)) == 0,
               NO_ERR_INVALID_ARG, "no_build_csr: unknown flag");
    NO_REQUIRE(n_vertices < (1ll << 31), NO_ERR_OVERFLOW, "no_build_csr: vertex ids are int32 inside the library, V must be < 2^31");
    const bool symmetrise = (flags & NO_CSR_SYMMETRISE) != 0, dedup = (flags & NO_CSR_DEDUP) != 0, ids64 = (flags & NO_CSR_IDS_64) != 0;
    const int64_t n_edges = symmetrise ? 2 * n_edges_in : n_edges_in;       // before duplicates are dropped
    NO_REQUIRE(rowptr_bits == 64 || n_edges < (1ll << 31), NO_ERR_OVERFLOW,
               "no_build_csr: 32-bit row pointers need fewer than 2^31 edges");
    NO_REQUIRE(n_edges < (1ll << 32) - 1, NO_ERR_UNSUPPORTED, "no_build_csr: at most 2^32-2 edges");
    NO_REQUIRE(!dedup || n_edges < (1ll << 31), NO_ERR_UNSUPPORTED, "no_build_csr: NO_CSR_DEDUP takes fewer than 2^31 edges");
    hipStream_t st = (hipStream_t)stream;

    no_graph_s* g = new no_graph_s();
    g->n_vertices = n_vertices;
    g->n_edges = n_edges;
    g->rowptr_bits = rowptr_bits;
    struct Guard { no_graph_s* g; ~Guard() { if (g) { g->release(); delete g; } } } guard{g};

    // One allocation for the temporaries: two sets of pair arrays that the passes alternate between, a fifth array where
    // duplicates are dropped, and the passes' scratch.
    const size_t ne = (size_t)n_edges, stride = (ne + 64) & ~(size_t)63;      // (room for one word more than the edges)
    const SortPlan sort(ilog2_ceil((uint64_t)n_vertices));
    const RadixPlan plan(n_edges);
    const size_t ws_words = std::max(plan.ws_words(), (scan_ws_bytes(n_edges) + 3) / 4);
    DevBuf<uint32_t> arena;
    DevBuf<int32_t> bad;
    DevBuf<char> staged;
    struct Tmp { DevBuf<uint32_t>* a; DevBuf<int32_t>* b; DevBuf<char>* s; ~Tmp() { ReleaseScope scope; a->release(); b->release(); s->release(); } } tmp{&arena, &bad, &staged};
    NO_CHECK(arena.alloc((dedup ? 5 : 4) * stride + ws_words));
    NO_CHECK(bad.alloc(1));
    NO_CHECK(g->col.alloc(ne));
    NO_CHECK(fill_i32(bad.p, 0, 1, st));
    uint32_t* keys[2] = {arena.p, arena.p + 2 * stride};
    uint32_t* vals[2] = {arena.p + stride, arena.p + 3 * stride};
    void* ws = arena.p + (dedup ? 5 : 4) * stride;
    const uint32_t* sorted_dst = keys[0];

    if (n_edges > 0) {
        // a host list is copied to the device: 32-bit ids into the arrays that the first pass does not write
        const size_t id_bytes = ids64 ? 8 : 4, list_bytes = (size_t)n_edges_in * id_bytes;
        if (!(flags & NO_CSR_INPUT_ON_DEVICE)) {
            char* at[2] = {(char*)keys[1], (char*)vals[1]};
            if (ids64) {
                NO_CHECK(staged.alloc(2 * list_bytes));
                at[0] = staged.p;
                at[1] = staged.p + list_bytes;
            }
            NO_HIP_CHECK(hipMemcpyAsync(at[0], src, list_bytes, hipMemcpyHostToDevice, st));
            NO_HIP_CHECK(hipMemcpyAsync(at[1], dst, list_bytes, hipMemcpyHostToDevice, st));
            src = at[0];
            dst = at[1];
        }
        // stable passes over the 2 * bits wide (destination, source): rows ascending by source
        int to = 0;
        if (ids64)
            NO_CHECK(radix_pass(EdgeSource<int64_t>{(const int64_t*)src, (const int64_t*)dst, n_edges_in, n_vertices, bad.p}, plan, 0, sort.width,
                                vals[to], keys[to], ws, st));
        else
            NO_CHECK(radix_pass(EdgeSource<int32_t>{(const int32_t*)src, (const int32_t*)dst, n_edges_in, n_vertices, bad.p}, plan, 0, sort.width,
                                vals[to], keys[to], ws, st));
        // (a pass leaves the destinations in keys[to], the sources in vals[to]; the last one the sources in the graph)
        PairArrays in{vals[to], keys[to]};              // the key is the source, then the destination
        bool by_dst = false;
        for (int p = 1, at = sort.width; p < sort.passes; ++p, to ^= 1) {
            if (at >= sort.bits && !by_dst) {
                by_dst = true;
                in = PairArrays{in.vals, in.keys};
                at = sort.across ? at - sort.bits : 0;
            }
            uint32_t* dsts = keys[to ^ 1];
            uint32_t* srcs = p + 1 == sort.passes && !dedup ? (uint32_t*)g->col.p : vals[to ^ 1];
            const int here = std::min(sort.width, sort.bits - at);
            if (by_dst) {
                NO_CHECK(radix_pass(in, plan, at, here, dsts, srcs, ws, st));
                in = PairArrays{dsts, srcs};
            } else {
                if (sort.across && here < sort.width) NO_CHECK(radix_pass_across(in, plan, at, sort.width, sort.bits, srcs, dsts, ws, st));
                else NO_CHECK(radix_pass(in, plan, at, here, srcs, dsts, ws, st));
                in = PairArrays{srcs, dsts};
            }
            at += sort.width;
        }
        sorted_dst = keys[to];
        if (dedup) {
            // keep the first of every run of equal pairs
            auto grid_for = [](int64_t n) { int64_t b = ceil_div(n, 256 * 4); if (b > 65536) b = 65536; return dim3((unsigned)b); };
            int32_t* keep = (int32_t*)keys[to ^ 1];
            int32_t* pos = (int32_t*)vals[to ^ 1];
            uint32_t* kept_dst = arena.p + 4 * stride;
            hipLaunchKernelGGL(mark_first_of_run_kernel, grid_for(n_edges), dim3(256), 0, st, sorted_dst, (const uint32_t*)vals[to],
                               n_edges, keep);
            NO_CHECK(exclusive_scan_i32(keep, nullptr, n_edges, pos, nullptr, ws, st));
            hipLaunchKernelGGL(compact_edges_kernel, grid_for(n_edges), dim3(256), 0, st, sorted_dst, (const uint32_t*)vals[to],
                               (const int32_t*)keep, (const int32_t*)pos, n_edges, g->col.p, kept_dst);
            NO_CHECK(launch_status("csr dedup"));
            int32_t kept = 0;
            NO_HIP_CHECK(hipMemcpyAsync(&kept, pos + n_edges, 4, hipMemcpyDeviceToHost, st));
            NO_HIP_CHECK(hipStreamSynchronize(st));
            g->n_edges = kept;
            sorted_dst = kept_dst;
        }
    }
    const dim3 rows((unsigned)ceil_div(n_vertices + 1, 256));
    if (rowptr_bits == 64) {
        NO_CHECK(g->rowptr64.alloc((size_t)n_vertices + 1));
        hipLaunchKernelGGL((rowptr_kernel<int64_t>), rows, dim3(256), 0, st, sorted_dst, g->n_edges, n_vertices, g->rowptr64.p);
    } else {
        NO_CHECK(g->rowptr32.alloc((size_t)n_vertices + 1));
        hipLaunchKernelGGL((rowptr_kernel<int32_t>), rows, dim3(256), 0, st, sorted_dst, g->n_edges, n_vertices, g->rowptr32.p);
    }
    NO_CHECK(launch_status("rowptr"));
    int32_t h_bad = 0;
    NO_HIP_CHECK(hipMemcpyAsync(&h_bad, bad.p, 4, hipMemcpyDeviceToHost, st));
    NO_HIP_CHECK(hipStreamSynchronize(st));
    NO_REQUIRE(h_bad == 0, NO_ERR_OUT_OF_RANGE, "no_build_csr: an edge endpoint lies outside [0, V)");
    guard.g = nullptr;
    handle_created();
    *out = g;
    return NO_OK;
}

extern "C" int32_t no_graph_view(no_graph_t g, int64_t* n_vertices, int64_t* n_edges, int32_t* rowptr_bits,
                                 const void** d_rowptr, const int32_t** d_col) {
    clear_error();
    NO_REQUIRE(g != nullptr, NO_ERR_INVALID_ARG, "no_graph_view: graph is NULL");
    if (n_vertices) *n_vertices = g->n_vertices;
    if (n_edges) *n_edges = g->n_edges;
    if (rowptr_bits) *rowptr_bits = g->rowptr_bits;
    if (d_rowptr) *d_rowptr = g->rowptr_bits == 64 ? (const void*)g->rowptr64.p : (const void*)g->rowptr32.p;
    if (d_col) *d_col = g->col.p;
    return NO_OK;
}

extern "C" int32_t no_graph_destroy(no_graph_t g) {
    clear_error();
    if (!g) return NO_OK;
    g->release();
    delete g;
    handle_destroyed();
    return NO_OK;
}
