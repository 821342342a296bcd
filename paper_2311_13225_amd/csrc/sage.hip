// no_sage_layer_fwd / no_sage_layer_bwd: one GraphSAGE-mean layer over a sampled block.
// Forward: mean over each destination's sampled row (Eq. 1, AGGREGATE = average), then the dense
// UPDATE of Eq. 2 on the matrix cores. Backward: the matching weight gradients and, for layers
// above the bottom one, the input gradient through the transposed block (segment sums in a fixed
// order, no float atomics). The bottom layer needs only the saved mean and the new embedding.
#include "layers.hpp"
#include "handles.hpp"
#include "gemm_tile.hpp"
#include "riders.hpp"

#include <stdlib.h>
#include <algorithm>
#include <mutex>
#include <type_traits>

namespace no {

// ------------------------------------------------------------------------ row segment reduce

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

template <typename T, int VEC> struct RowVec;
template <> struct RowVec<float, 4> {
    static __device__ __forceinline__ void add(float (&acc)[4], const float* p) {
        float4 v = *reinterpret_cast<const float4*>(p);
        acc[0] += v.x; acc[1] += v.y; acc[2] += v.z; acc[3] += v.w;
    }
};
template <> struct RowVec<float, 2> {
    static __device__ __forceinline__ void add(float (&acc)[2], const float* p) {
        float2 v = *reinterpret_cast<const float2*>(p);
        acc[0] += v.x; acc[1] += v.y;
    }
};
template <> struct RowVec<float, 1> {
    static __device__ __forceinline__ void add(float (&acc)[1], const float* p) { acc[0] += p[0]; }
};
template <> struct RowVec<uint16_t, 8> {
    static __device__ __forceinline__ void add(float (&acc)[8], const uint16_t* p) {
        uint4 v = *reinterpret_cast<const uint4*>(p);
        uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc[2 * i] += __uint_as_float(w[i] << 16);
            acc[2 * i + 1] += __uint_as_float(w[i] & 0xffff0000u);
        }
    }
};
template <> struct RowVec<uint16_t, 2> {
    static __device__ __forceinline__ void add(float (&acc)[2], const uint16_t* p) {
        uint32_t w = *reinterpret_cast<const uint32_t*>(p);
        acc[0] += __uint_as_float(w << 16);
        acc[1] += __uint_as_float(w & 0xffff0000u);
    }
};
template <> struct RowVec<uint16_t, 1> {
    static __device__ __forceinline__ void add(float (&acc)[1], const uint16_t* p) { acc[0] += bf16_to_f32(p[0]); }
};

// Per-source weights of the symmetric normalisation (Table 1: the adjacency matrix after symmetric normalisation, here
// of the sampled block with self loops): s_u = (c_u + [u < n_self])^-1/2, c_u = number of the block's edges that leave u.
__device__ __forceinline__ float source_weight(const SourceWeights& sw, int32_t u, int32_t n_self) {
    const int32_t c = (sw.is_ptr ? sw.cnt[u + 1] - sw.cnt[u] : sw.cnt[u]) + (u < n_self ? 1 : 0);
    return c > 0 ? 1.f / sqrtf((float)c) : 0.f;
}

// A vector unit as it comes from memory, and its accumulation in fp32 (the two halves of RowVec::add, for kernels that
// keep many units in flight in their memory form: 4 registers per bf16 unit of 8 instead of 8)
template <typename T, int VEC> struct RawUnit;
template <> struct RawUnit<float, 4> { using type = float4; };
template <> struct RawUnit<float, 2> { using type = float2; };
template <> struct RawUnit<float, 1> { using type = float; };
template <> struct RawUnit<uint16_t, 8> { using type = uint4; };
template <> struct RawUnit<uint16_t, 2> { using type = uint32_t; };
template <> struct RawUnit<uint16_t, 1> { using type = uint16_t; };
__device__ __forceinline__ void accum_unit(float (&acc)[4], const float4& v) { acc[0] += v.x; acc[1] += v.y; acc[2] += v.z; acc[3] += v.w; }
__device__ __forceinline__ void accum_unit(float (&acc)[2], const float2& v) { acc[0] += v.x; acc[1] += v.y; }
__device__ __forceinline__ void accum_unit(float (&acc)[1], const float& v) { acc[0] += v; }
__device__ __forceinline__ void accum_unit(float (&acc)[8], const uint4& v) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        acc[2 * i] += __uint_as_float(w[i] << 16);
        acc[2 * i + 1] += __uint_as_float(w[i] & 0xffff0000u);
    }
}
__device__ __forceinline__ void accum_unit(float (&acc)[2], const uint32_t& w) {
    acc[0] += __uint_as_float(w << 16);
    acc[1] += __uint_as_float(w & 0xffff0000u);
}
__device__ __forceinline__ void accum_unit(float (&acc)[1], const uint16_t& b) { acc[0] += bf16_to_f32(b); }

// out[row, :] = init + scale * sum_{p in [seg[row], seg[row+1])} w_p * src[idx[p], :]
//   MEAN: init = 0 and, by agg_mode: AGG_NEIGH_MEAN scale = 1/len (0 for an empty segment): forward aggregate of the
//         GraphSAGE-mean layer. The other modes add the row's own source row first (Eq. 1 over N_in(v) U {v}):
//         AGG_SELF_MEAN scale = 1/(len + 1); AGG_SELF_SUM scale = 1; AGG_SELF_SYM scale = (len + 1)^-1/2 and every term
//         (the self row included) is weighed by its source's s_u (WEIGHTED).
//   else: scale = 1, w = 1, init = out[row,:] for row < *d_n_init, else 0 (backward through the transpose); WEIGHTED: the
//         result is multiplied by s_row (the adjoint of the forward weights, row = source).
// A group of G = 2^g_log2 lanes owns one work item = (row, chunk of G vector units); a lane owns one
// vector unit of it. Rows wider than 64 units are split into several items handled by different
// wavefronts, so a wide row keeps many short independent load chains in flight instead of one long one;
// the items of a row are consecutive, which keeps the reads of a source row next to each other in time.
// Up to eight source rows are loaded before the first add; the adds stay in segment order.
// MASKED: the result goes to masked_out (backward inside a step), a variant of its own because the registers it holds cost the plain
// form 3 us of the 84 of a layer's forward and backward pass (3.4 K rows, 256 x 256). MASK_BITS: the ReLU decisions from the bytes that the layer
// below's product left, a sixteenth of its output's size (steps, us: 4096 seeds, 256 columns 675.5 -> 670.8, bf16 209.5 -> 206.3, dense 198.3 -> 197.1).
// Side: SideTasks where the launch carries some, else NoSideTasks (the tasks' code costs the widest forms 2 to 34 registers).
enum { MASK_NONE = 0, MASK_H, MASK_BITS };
template <typename T, int VEC, bool MEAN, bool WEIGHTED, int MASK, typename Side>
__global__ void __launch_bounds__(256, MEAN ? 1 : WEIGHTED ? 4 : 5) segment_rows_kernel(RowCopyJob job, const T* __restrict__ src, int64_t ld_src,
                                                           const int32_t* __restrict__ seg, const int32_t* __restrict__ idx,
                                                           const int32_t* d_n_rows, int32_t n_rows_cap,
                                                           const int32_t* d_n_init, float* __restrict__ out, int64_t ld_out,
                                                           int32_t units, int32_t g_log2, int32_t n_chunks,
                                                           const int32_t* __restrict__ self_idx, int32_t agg_mode,
                                                           const void* __restrict__ mask, const int32_t* __restrict__ out_rows,
                                                           float* __restrict__ masked_out, SourceWeights sw, Side side) {
    constexpr bool MASKED = MASK != MASK_NONE;
    using Decision = std::conditional_t<MASK == MASK_BITS, uint8_t, typename RawUnit<float, MASKED ? VEC : 1>::type>;
    if (blockIdx.x >= side.first_block) { run_side_tasks(side); return; }
    if (job.dst && blockIdx.x >= job.first_block) {
        // extra blocks of the launch: dst[dst_rows[i], :] = src[src_rows[i], :], one wavefront per row (rows that are
        // ready before this kernel's own output is, e.g. the cached layer-1 rows of the reused vertices)
        const int32_t nj = *job.d_n;
        const int64_t w0 = (((int64_t)(blockIdx.x - job.first_block)) * blockDim.x + threadIdx.x) >> 6;
        const int64_t nw = ((int64_t)(side.first_block - job.first_block) * blockDim.x) >> 6;
        const int ln = (int)(threadIdx.x & 63);
        for (int64_t i = w0; i < nj; i += nw) {
            const float* s_ = job.src + (int64_t)job.src_rows[i] * job.dim;
            float* d_ = job.dst + (int64_t)job.dst_rows[i] * job.dim;
            for (int c = ln; c < job.dim; c += 64) d_[c] = s_[c];
        }
        return;
    }
    int32_t n = *d_n_rows;
    if (n > n_rows_cap) n = n_rows_cap;
    const int32_t n_init = (!MEAN && d_n_init) ? *d_n_init : 0;
    const int32_t lane = (int32_t)(threadIdx.x & 63);
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t n_waves = ((int64_t)(job.dst ? job.first_block : side.first_block) * blockDim.x) >> 6;
    const int32_t items_per_pass = 64 >> g_log2;
    const int32_t sub = lane >> g_log2, u0 = lane & ((1 << g_log2) - 1);
    const int64_t n_items = (int64_t)n * n_chunks;
    const bool with_self = MEAN && agg_mode != AGG_NEIGH_MEAN;
    for (int64_t item = wave * items_per_pass + sub; item < n_items; item += n_waves * items_per_pass) {
        const int64_t row = item / n_chunks;
        const int32_t u = (int32_t)(item - row * n_chunks) * (1 << g_log2) + u0;
        if (u >= units) continue;
        const int32_t b = seg[row], e = seg[row + 1];
        float scale = MEAN ? (e > b ? 1.f / (float)(e - b) : 0.f) : 1.f;
        const T* col = src + (int64_t)u * VEC;
        // Backward, the consumer is the layer below: its ReLU decision (its output h, row `row`) is applied and the row placed where
        // that layer's gradient rows live (out_rows[row], -1 = the row takes no gradient, and nothing of it is read). Both
        // are asked for before the segment: the kernel is bound by its chain of dependent round trips, which they would make two
        // longer at the end (step of 4096 seeds, 256 columns: 774 -> 752 us; super-batch with most rows served by the cache: 1477 -> 1437).
        int64_t masked_row = row;
        Decision decision{};
        if constexpr (MASKED) {
            if (out_rows) masked_row = out_rows[row];
            if (masked_row < 0) continue;
            decision = static_cast<const Decision*>(mask)[row * units + u];      // (rows of ld_out = units * VEC columns)
        }
        float acc[VEC];
#pragma unroll
        for (int c = 0; c < VEC; ++c) acc[c] = 0.f;
        if (with_self) {
            // Eq. 1 over N_in(v) U {v}: the destination's own row (row `row` of src, or self_idx[row]) joins the aggregate
            RowVec<T, VEC>::add(acc, col + (int64_t)(self_idx ? self_idx[row] : (int32_t)row) * ld_src);
            if (WEIGHTED) {
                const float ws = source_weight(sw, (int32_t)row, n);
#pragma unroll
                for (int c = 0; c < VEC; ++c) acc[c] *= ws;
            }
            scale = agg_mode == AGG_SELF_MEAN ? 1.f / (float)(e - b + 1)
                  : agg_mode == AGG_SELF_SUM  ? 1.f : 1.f / sqrtf((float)(e - b + 1));
        }
        float* o = out + row * ld_out + (int64_t)u * VEC;
        if (!MEAN && row < n_init) {
#pragma unroll
            for (int c = 0; c < VEC; ++c) acc[c] = o[c];
        }
        int32_t p = b;
        if (!MEAN && g_log2 == 6 && (units & 63) == 0) {      // (every lane of the wavefront is at work on this row)
            // Backward through the transpose, one wavefront per source row: a popular source has hundreds of entries, and
            // eight rows per round trip (each behind a round trip for its indices) would make that one row the kernel's
            // critical path. The wavefront reads 64 indices with one load and keeps 16 rows in flight; segments shorter
            // than 16 (nearly all of them) fall through to the rounds of 8, 4 and 1-3 below.
            for (; p + 16 <= e;) {
                const int32_t n = min(64, e - p);
                const int32_t mine = lane < n ? idx[p + lane] : 0;
                int32_t t = 0;
                for (; t + 16 <= n; t += 16) {
                    float a[16][VEC];
#pragma unroll
                    for (int j = 0; j < 16; ++j) {
                        const int32_t ix = __shfl(mine, t + j, 64);
#pragma unroll
                        for (int c = 0; c < VEC; ++c) a[j][c] = 0.f;
                        RowVec<T, VEC>::add(a[j], col + (int64_t)ix * ld_src);
                    }
#pragma unroll
                    for (int j = 0; j < 16; ++j)
#pragma unroll
                        for (int c = 0; c < VEC; ++c) acc[c] += a[j][c];
                }
                p += t;
            }
        }
        for (; p + 8 <= e; p += 8) {
            int32_t ix[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) ix[j] = idx[p + j];
            float wt[8];
            if (MEAN && WEIGHTED) {
#pragma unroll
                for (int j = 0; j < 8; ++j) wt[j] = source_weight(sw, sw.local ? sw.local[p + j] : ix[j], n);
            }
            float a[8][VEC];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
#pragma unroll
                for (int c = 0; c < VEC; ++c) a[j][c] = 0.f;
                RowVec<T, VEC>::add(a[j], col + (int64_t)ix[j] * ld_src);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int c = 0; c < VEC; ++c) acc[c] += (MEAN && WEIGHTED) ? wt[j] * a[j][c] : a[j][c];
        }
        if (p + 4 <= e) {
            int32_t ix[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) ix[j] = idx[p + j];
            float wt[4];
            if (MEAN && WEIGHTED) {
#pragma unroll
                for (int j = 0; j < 4; ++j) wt[j] = source_weight(sw, sw.local ? sw.local[p + j] : ix[j], n);
            }
            float a[4][VEC];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
#pragma unroll
                for (int c = 0; c < VEC; ++c) a[j][c] = 0.f;
                RowVec<T, VEC>::add(a[j], col + (int64_t)ix[j] * ld_src);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int c = 0; c < VEC; ++c) acc[c] += (MEAN && WEIGHTED) ? wt[j] * a[j][c] : a[j][c];
            p += 4;
        }
        if (p < e) {        // one to three rows left
            const int32_t i0 = idx[p], i1 = p + 1 < e ? idx[p + 1] : i0, i2 = p + 2 < e ? idx[p + 2] : i0;
            float w0 = 1.f, w1 = 1.f, w2 = 1.f;
            if (MEAN && WEIGHTED) {
                w0 = source_weight(sw, sw.local ? sw.local[p] : i0, n);
                w1 = p + 1 < e ? source_weight(sw, sw.local ? sw.local[p + 1] : i1, n) : 0.f;
                w2 = p + 2 < e ? source_weight(sw, sw.local ? sw.local[p + 2] : i2, n) : 0.f;
            }
            float a[3][VEC];
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int c = 0; c < VEC; ++c) a[j][c] = 0.f;
            RowVec<T, VEC>::add(a[0], col + (int64_t)i0 * ld_src);
            if (p + 1 < e) RowVec<T, VEC>::add(a[1], col + (int64_t)i1 * ld_src);
            if (p + 2 < e) RowVec<T, VEC>::add(a[2], col + (int64_t)i2 * ld_src);
#pragma unroll
            for (int c = 0; c < VEC; ++c)
                acc[c] = (MEAN && WEIGHTED) ? ((acc[c] + w0 * a[0][c]) + w1 * a[1][c]) + w2 * a[2][c]
                                            : ((acc[c] + a[0][c]) + a[1][c]) + a[2][c];
        }
        if (!MEAN && WEIGHTED) {
            const float ws = source_weight(sw, (int32_t)row, n_init);
#pragma unroll
            for (int c = 0; c < VEC; ++c) acc[c] *= ws;
        }
        if constexpr (MASKED) {
            float hm[VEC];
            if constexpr (MASK == MASK_H) {
                __builtin_memcpy(hm, &decision, sizeof(hm));
            } else {
#pragma unroll
                for (int c = 0; c < VEC; ++c) hm[c] = (uint32_t)decision >> c & 1u ? 1.f : 0.f;
            }
            float* mo = masked_out + masked_row * ld_out + (int64_t)u * VEC;
#pragma unroll
            for (int c = 0; c < VEC; ++c) mo[c] = hm[c] > 0.f ? acc[c] : 0.f;
            continue;
        }
#pragma unroll
        for (int c = 0; c < VEC; ++c) o[c] = acc[c] * scale;
    }
}

template <typename T, int VEC, bool MEAN>
static void launch_segment(const T* src, int64_t ld_src, const int32_t* seg, const int32_t* idx, const int32_t* d_n,
                           int32_t n_cap, const int32_t* d_n_init, float* out, int64_t ld_out, int32_t dim, hipStream_t st,
                           const int32_t* self_idx = nullptr, int32_t agg_mode = AGG_NEIGH_MEAN, const float* mask_h = nullptr,
                           const int32_t* out_rows = nullptr, float* masked_out = nullptr, const RowCopyJob* copy = nullptr,
                           hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr, const SourceWeights* weights = nullptr, no_blocks_s* side_of = nullptr,
                           const CutJobs* cut = nullptr, const ReduceArgs* reduce = nullptr, const uint8_t* mask_bits = nullptr) {
    const int32_t units = dim / VEC;
    int g_log2 = 0;
    while ((1 << g_log2) < units && g_log2 < 6) ++g_log2;
    const int32_t n_chunks = (int32_t)ceil_div(units, 1 << g_log2);
    int64_t waves = ceil_div((int64_t)n_cap * n_chunks, 64 >> g_log2);
    int64_t blocks = ceil_div(waves, 4);
    if (blocks > 256 * 64) blocks = 256 * 64;
    if (blocks < 1) blocks = 1;
    RowCopyJob job = copy ? *copy : RowCopyJob{};
    int64_t copy_blocks = 0;
    if (job.dst) {
        job.first_block = (uint32_t)blocks;
        copy_blocks = ceil_div(job.n_cap, 4);
        if (copy_blocks > 1024) copy_blocks = 1024;
        if (copy_blocks < 1) copy_blocks = 1;
    }
    const SourceWeights sw = weights ? *weights : SourceWeights{};
    const uint32_t own = (uint32_t)(blocks + copy_blocks);
    auto launch_as = [&](auto weighted, auto masked, const auto& side, uint32_t grid) {
        using Side = std::decay_t<decltype(side)>;
        const void* mask = decltype(masked)::value == MASK_BITS ? (const void*)mask_bits : (const void*)mask_h;
        NO_LAUNCH_TIMED((segment_rows_kernel<T, VEC, MEAN, decltype(weighted)::value, decltype(masked)::value, Side>), dim3(grid), dim3(256), st, ev0, ev1, job, src,
                        ld_src, seg, idx, d_n, n_cap, d_n_init, out, ld_out, units, g_log2, n_chunks, self_idx, agg_mode, mask, out_rows,
                        masked_out, sw, side);
    };
    auto launch = [&](auto weighted, const auto& side, uint32_t grid) {
        if constexpr (!MEAN) {
            if constexpr (VEC == 4) {
                if (masked_out && mask_bits) { launch_as(weighted, std::integral_constant<int, MASK_BITS>{}, side, grid); return; }
            }
            if (masked_out) { launch_as(weighted, std::integral_constant<int, MASK_H>{}, side, grid); return; }
        }
        launch_as(weighted, std::integral_constant<int, MASK_NONE>{}, side, grid);
    };
    if constexpr (MEAN) {
        launch_with_riders(cut, side_of, own, [&](const auto& side, uint32_t grid) {
            if (sw.cnt) launch(std::true_type{}, side, grid);
            else launch(std::false_type{}, side, grid);
        });
        return;
    } else if (reduce) {
        ReduceSide side{own, (uint32_t)reduce_blocks(*reduce), *reduce};
        const uint32_t grid = own + side.blocks * (uint32_t)reduce->n_problems;
        if (sw.cnt) launch_as(std::true_type{}, std::integral_constant<int, MASK_NONE>{}, side, grid);
        else launch_as(std::false_type{}, std::integral_constant<int, MASK_NONE>{}, side, grid);
        return;
    }
    NoSideTasks none;
    none.first_block = own;
    if (sw.cnt) launch(std::true_type{}, none, own);
    else launch(std::false_type{}, none, own);
}

// The layer-1 aggregate straight from the sampler's fixed-stride slot array: row r's sampled neighbours are the
// entries pad[r*k .. r*k + k) in slot order (the order of the compacted row), -1 from the first unused slot on, and a
// first occurrence may carry the relabelling's mark (-2 - id in place of id). Reading the slots needs neither the row
// pointers nor the compacted index array, so a work item's chain of dependent memory round trips is "row count -> slots
// -> rows -> store" instead of "row count -> row pointers -> indices -> rows -> store": the kernel is bound by that chain
// (every wave handles one or two items), not by bytes in flight. NS (8 or 16) slots and their rows are in flight at a time. Same sums in the same order as segment_rows_kernel<MEAN>.
// agg_mode as there (no per-source weights here).
template <typename T, int VEC, int NS, typename Side>
__global__ void __launch_bounds__(256) padded_rows_kernel(RowCopyJob job, const T* __restrict__ src, int64_t ld_src,
                                                          const int32_t* __restrict__ pad, int32_t k,
                                                          const int32_t* d_n_rows, int32_t n_rows_cap,
                                                          float* __restrict__ out, int64_t ld_out, int32_t units,
                                                          int32_t g_log2, int32_t n_chunks,
                                                          const int32_t* __restrict__ self_idx, int32_t agg_mode, Side side) {
    if (blockIdx.x >= side.first_block) { run_side_tasks(side); return; }
    if (job.dst && blockIdx.x >= job.first_block) {
        const int32_t nj = *job.d_n;
        const int64_t w0 = (((int64_t)(blockIdx.x - job.first_block)) * blockDim.x + threadIdx.x) >> 6;
        const int64_t nw = ((int64_t)(side.first_block - job.first_block) * blockDim.x) >> 6;
        const int ln = (int)(threadIdx.x & 63);
        for (int64_t i = w0; i < nj; i += nw) {
            const float* s_ = job.src + (int64_t)job.src_rows[i] * job.dim;
            float* d_ = job.dst + (int64_t)job.dst_rows[i] * job.dim;
            for (int c = ln; c < job.dim; c += 64) d_[c] = s_[c];
        }
        return;
    }
    using Raw = typename RawUnit<T, VEC>::type;
    int32_t n = *d_n_rows;
    if (n > n_rows_cap) n = n_rows_cap;
    const int32_t lane = (int32_t)(threadIdx.x & 63);
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t n_waves = ((int64_t)(job.dst ? job.first_block : side.first_block) * blockDim.x) >> 6;
    const int32_t items_per_pass = 64 >> g_log2;
    const int32_t sub = lane >> g_log2, u0 = lane & ((1 << g_log2) - 1);
    const int64_t n_items = (int64_t)n * n_chunks;
    const bool with_self = agg_mode != AGG_NEIGH_MEAN;
    for (int64_t item = wave * items_per_pass + sub; item < n_items; item += n_waves * items_per_pass) {
        const int64_t row = item / n_chunks;
        const int32_t u = (int32_t)(item - row * n_chunks) * (1 << g_log2) + u0;
        if (u >= units) continue;
        const int32_t* slots = pad + row * k;
        int32_t e[NS];
#pragma unroll
        for (int j = 0; j < NS; ++j) e[j] = j < k ? slots[j] : -1;
        int32_t self_row = (int32_t)row;
        if (with_self && self_idx) self_row = self_idx[row];
        const T* col = src + (int64_t)u * VEC;
        float acc[VEC];
#pragma unroll
        for (int c = 0; c < VEC; ++c) acc[c] = 0.f;
        if (with_self) RowVec<T, VEC>::add(acc, col + (int64_t)self_row * ld_src);
        int32_t len = 0;
        for (int32_t j0 = 0;;) {
            Raw raw[NS];
#pragma unroll
            for (int j = 0; j < NS; ++j)
                if (e[j] != -1) raw[j] = *reinterpret_cast<const Raw*>(col + (int64_t)(e[j] <= -2 ? -2 - e[j] : e[j]) * ld_src);
#pragma unroll
            for (int j = 0; j < NS; ++j)
                if (e[j] != -1) {
                    accum_unit(acc, raw[j]);
                    ++len;
                }
            j0 += NS;
            if (j0 >= k || e[NS - 1] == -1) break;          // unused slots are at the end of a row
#pragma unroll
            for (int j = 0; j < NS; ++j) e[j] = j0 + j < k ? slots[j0 + j] : -1;
        }
        const float scale = agg_mode == AGG_NEIGH_MEAN ? (len > 0 ? 1.f / (float)len : 0.f)
                          : agg_mode == AGG_SELF_MEAN  ? 1.f / (float)(len + 1) : 1.f;
        float* o = out + row * ld_out + (int64_t)u * VEC;
#pragma unroll
        for (int c = 0; c < VEC; ++c) o[c] = acc[c] * scale;
    }
}

template <typename T, int VEC>
static void launch_padded(const T* src, int64_t ld_src, const int32_t* pad, int32_t k, const int32_t* d_n, int32_t n_cap,
                          float* out, int64_t ld_out, int32_t dim, hipStream_t st, const int32_t* self_idx, int32_t agg_mode,
                          const RowCopyJob* copy, hipEvent_t ev0, hipEvent_t ev1, no_blocks_s* side_of, const CutJobs* cut) {
    const int32_t units = dim / VEC;
    int g_log2 = 0;
    while ((1 << g_log2) < units && g_log2 < 6) ++g_log2;
    const int32_t n_chunks = (int32_t)ceil_div(units, 1 << g_log2);
    int64_t waves = ceil_div((int64_t)n_cap * n_chunks, 64 >> g_log2);
    int64_t blocks = ceil_div(waves, 4);
    if (blocks > 256 * 64) blocks = 256 * 64;
    if (blocks < 1) blocks = 1;
    RowCopyJob job = copy ? *copy : RowCopyJob{};
    int64_t copy_blocks = 0;
    if (job.dst) {
        job.first_block = (uint32_t)blocks;
        copy_blocks = ceil_div(job.n_cap, 4);
        if (copy_blocks > 1024) copy_blocks = 1024;
        if (copy_blocks < 1) copy_blocks = 1;
    }
    const uint32_t own = (uint32_t)(blocks + copy_blocks);
    auto launch = [&](auto slots, const auto& side, uint32_t grid) {
        using Side = std::decay_t<decltype(side)>;
        NO_LAUNCH_TIMED((padded_rows_kernel<T, VEC, decltype(slots)::value, Side>), dim3(grid), dim3(256), st, ev0, ev1, job, src, ld_src,
                        pad, k, d_n, n_cap, out, ld_out, units, g_log2, n_chunks, self_idx, agg_mode, side);
    };
    using Few = std::integral_constant<int, 8>;
    using Many = std::integral_constant<int, 16>;
    launch_with_riders(cut, side_of, own, [&](const auto& side, uint32_t grid) {
        if (k <= 8) launch(Few{}, side, grid);
        else launch(Many{}, side, grid);
    });
}

int32_t mean_aggregate(const void* x_src, no_dtype dt, int32_t dim, const int32_t* indptr, const int32_t* indices,
                       const int32_t* d_n_dst, int32_t n_dst_cap, float* mean, hipStream_t st, int32_t agg_mode,
                       const int32_t* self_idx, const RowCopyJob* copy, hipEvent_t ev0, hipEvent_t ev1,
                       const SourceWeights* weights, const PaddedSlots* padded, no_blocks_s* side_of, const CutJobs* cut) {
    if (n_dst_cap <= 0) return NO_OK;
    if (padded && padded->pad && !(weights && weights->cnt)) {
        // the rows are addressed through the sampler's slot array (global ids): two memory round trips fewer per item
        const int32_t* pad = padded->pad;
        const int32_t k = padded->k;
#define NO_PAD_FWD(T, V, ptr) \
    launch_padded<T, V>(ptr, dim, pad, k, d_n_dst, n_dst_cap, mean, dim, dim, st, self_idx, agg_mode, copy, ev0, ev1, side_of, cut)
        if (dt == NO_F32) {
            const float* x = (const float*)x_src;
            const bool a16 = (((uintptr_t)x | (uintptr_t)mean) & 15) == 0, a8 = (((uintptr_t)x | (uintptr_t)mean) & 7) == 0;
            if (dim % 4 == 0 && a16) NO_PAD_FWD(float, 4, x);
            else if (dim % 2 == 0 && a8) NO_PAD_FWD(float, 2, x);
            else NO_PAD_FWD(float, 1, x);
        } else {
            const uint16_t* x = (const uint16_t*)x_src;
            if (dim % 8 == 0 && ((uintptr_t)x & 15) == 0 && ((uintptr_t)mean & 15) == 0) NO_PAD_FWD(uint16_t, 8, x);
            else if (dim % 2 == 0 && ((uintptr_t)x & 3) == 0) NO_PAD_FWD(uint16_t, 2, x);
            else NO_PAD_FWD(uint16_t, 1, x);
        }
#undef NO_PAD_FWD
        return launch_status("mean_aggregate (slot array)");
    }
#define NO_SEG_FWD(T, V, ptr) \
    launch_segment<T, V, true>(ptr, dim, indptr, indices, d_n_dst, n_dst_cap, nullptr, mean, dim, dim, st, self_idx, agg_mode, \
                               nullptr, nullptr, nullptr, copy, ev0, ev1, weights, side_of, cut)
    if (dt == NO_F32) {
        const float* x = (const float*)x_src;
        const bool a16 = (((uintptr_t)x | (uintptr_t)mean) & 15) == 0, a8 = (((uintptr_t)x | (uintptr_t)mean) & 7) == 0;
        if (dim % 4 == 0 && a16) NO_SEG_FWD(float, 4, x);
        else if (dim % 2 == 0 && a8) NO_SEG_FWD(float, 2, x);
        else NO_SEG_FWD(float, 1, x);
    } else {
        const uint16_t* x = (const uint16_t*)x_src;
        if (dim % 8 == 0 && ((uintptr_t)x & 15) == 0 && ((uintptr_t)mean & 15) == 0) NO_SEG_FWD(uint16_t, 8, x);
        else if (dim % 2 == 0 && ((uintptr_t)x & 3) == 0) NO_SEG_FWD(uint16_t, 2, x);
        else NO_SEG_FWD(uint16_t, 1, x);
    }
#undef NO_SEG_FWD
    return launch_status("mean_aggregate");
}

// grad_x[u,:] = s_u * ((u < n_dst ? grad_x[u,:] : 0) + sum over transposed entries of u of gmean_scaled[csc_dst[p],:]),
// s_u = 1 unless source weights are given
int32_t transpose_aggregate(const float* gmean_scaled, int32_t dim, const int32_t* csc_indptr, const int32_t* csc_dst,
                            const int32_t* d_n_src, int32_t n_src_cap, const int32_t* d_n_dst, float* grad_x,
                            hipStream_t st, const float* mask_h, const int32_t* out_rows, float* masked_out,
                            const SourceWeights* weights, const ReduceArgs* reduce, const uint8_t* mask_bits) {
    if (n_src_cap <= 0) return NO_OK;
    const uintptr_t al = (uintptr_t)gmean_scaled | (uintptr_t)grad_x | (uintptr_t)mask_h | (uintptr_t)masked_out;
    const bool a16 = (al & 15) == 0, a8 = (al & 7) == 0;
#define NO_SEG_BWD(V) \
    launch_segment<float, V, false>(gmean_scaled, dim, csc_indptr, csc_dst, d_n_src, n_src_cap, d_n_dst, grad_x, dim, dim, st, \
                                    nullptr, AGG_NEIGH_MEAN, mask_h, out_rows, masked_out, nullptr, nullptr, nullptr, weights, nullptr, nullptr, reduce, mask_bits)
    if (dim % 4 == 0 && a16) NO_SEG_BWD(4);
    else if (dim % 2 == 0 && a8) NO_SEG_BWD(2);
    else NO_SEG_BWD(1);
#undef NO_SEG_BWD
    return launch_status("transpose_aggregate");
}

// ------------------------------------------------------------------------ small elementwise kernels

// gz[r,:] = grad_h[rows ? rows[r] : r, :] masked by [h[r,:] > 0] when relu: selects the rows that take a gradient
// (the computed vertices when hot rows were reused) and applies the activation's derivative in one pass.
__global__ void mask_rows_kernel(const float* __restrict__ grad_h, const int32_t* __restrict__ rows,
                                 const float* __restrict__ h, const int32_t* d_n, int32_t n_cap, int32_t dim, int32_t relu,
                                 float* __restrict__ gz, uint32_t own_blocks, CutJobs cut) {
    if (blockIdx.x >= own_blocks) { run_cut_jobs(cut, blockIdx.x - own_blocks); return; }
    int32_t n = *d_n;
    if (n > n_cap) n = n_cap;
    const int64_t total = (int64_t)n * dim;
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)own_blocks * blockDim.x;
    if (!rows && (((uintptr_t)grad_h | (uintptr_t)h | (uintptr_t)gz) & 15) == 0) {      // (relu: without rows and without it there is no launch)
        const int64_t quads = total / 4;
        for (int64_t q = i; q < quads; q += stride) {
            const float4 g = reinterpret_cast<const float4*>(grad_h)[q], v = reinterpret_cast<const float4*>(h)[q];
            reinterpret_cast<float4*>(gz)[q] = make_float4(v.x > 0.f ? g.x : 0.f, v.y > 0.f ? g.y : 0.f, v.z > 0.f ? g.z : 0.f, v.w > 0.f ? g.w : 0.f);
        }
        i += quads * 4;
    }
    for (; i < total; i += stride) {
        const int64_t r = i / dim, c = i - r * dim;
        const float g = rows ? grad_h[(int64_t)rows[r] * dim + c] : grad_h[i];
        gz[i] = (!relu || h[i] > 0.f) ? g : 0.f;
    }
}

__global__ void bf16_rows_to_f32_kernel(const uint16_t* __restrict__ x, const int32_t* d_n, int32_t n_cap, int32_t dim,
                                        float* __restrict__ out) {
    int32_t n = *d_n;
    if (n > n_cap) n = n_cap;
    const int64_t total = (int64_t)n * dim;
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < total; i += stride) out[i] = bf16_to_f32(x[i]);
}

static inline unsigned ew_blocks(int64_t total) {
    int64_t b = ceil_div(total, 256 * 4);
    if (b > 256 * 16) b = 256 * 16;
    if (b < 1) b = 1;
    return (unsigned)b;
}

static int32_t bf16_rows_to_f32(const uint16_t* x, const int32_t* d_n, int32_t n_cap, int32_t dim, float* out, hipStream_t st) {
    if (n_cap <= 0 || dim <= 0) return NO_OK;
    hipLaunchKernelGGL(bf16_rows_to_f32_kernel, dim3(ew_blocks((int64_t)n_cap * dim)), dim3(256), 0, st, x, d_n, n_cap, dim, out);
    return launch_status("bf16_rows_to_f32");
}

// ------------------------------------------------------------------------ workspace layout

// Number of row slices of the weight-gradient product: enough 64x64 output tiles x slices to give every
// compute unit several blocks, bounded so that a slice keeps at least 64 rows of the capacity.
int32_t layer_splits(int32_t n_dst_cap, int32_t d_in, int32_t d_out) {
    const int64_t tiles = 2 * ceil_div(d_in + 1, 64) * ceil_div(d_out, 64);
    const int64_t target = 1600;      // blocks of the split product (measured: flat from 960 to 1600, slower beyond)
    int64_t s = ceil_div(target, tiles);
    const int64_t by_rows = ceil_div(n_dst_cap, 64);
    if (s > by_rows) s = by_rows;
    if (s > 64) s = 64;
    if (s < 1) s = 1;
    return (int32_t)s;
}

static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// in_step: a step's workspace is its model's own, with room for as many slices as fill the chip with large tiles (tn_plan). It is laid out for two
// products; one alone (GCN-style layers) takes both halves: step_splits.
LayerWorkspace carve_workspace(void* ws, int32_t n_dst_cap, int32_t d_in, int32_t d_out, bool in_step) {
    LayerWorkspace w;
    w.splits = layer_splits(n_dst_cap, d_in, d_out);
    if (in_step) {
        const int64_t fill = TN_SLOTS / (2 * ceil_div(d_in, 128) * ceil_div(d_out, 128)), by_rows = ceil_div(n_dst_cap, TN_LEAST_ROWS);
        w.splits = (int32_t)std::max<int64_t>(w.splits, std::min<int64_t>(std::min(fill, by_rows), 128));
    }
    size_t off = 0;
    char* base = (char*)ws;
    w.gz = (float*)(base + off);        off += align256((size_t)n_dst_cap * d_out * 4);
    w.gmean = (float*)(base + off);     off += align256((size_t)n_dst_cap * d_in * 4);
    w.x_dst_f32 = (float*)(base + off); off += align256((size_t)n_dst_cap * d_in * 4);
    w.partials = (float*)(base + off);  off += align256((size_t)2 * w.splits * (d_in + 1) * d_out * 4);
    w.planes_bytes = (size_t)(base + off - (char*)w.x_dst_f32);
    w.fwd_planes = w.gz;
    w.fwd_planes_bytes = (size_t)((char*)w.x_dst_f32 - (char*)w.gz);
    w.bytes = off;
    return w;
}

// The most slices of a step's weight gradients. One product alone takes both halves of the partials' room (less one slice, in whose place the word of
// tn_used_word stands), unless the step reuses rows: the next batch's aggregation then waits for this one's layer 1 and runs beside the weight
// gradients, in the places that a block a compute unit leaves. Measured, GCN-style steps prepared ahead, 602 x 256, us in one half / in both: 1024 seeds without
// reuse 175.4 / 170.2, 2048 255.7 / 248.8, 4096 386.6 / 375.4, 25 K rows of a uniform graph 341 / 315 (the product alone 70.5 / 57.1); with reuse 147.6 / 151.4,
// 197.5 / 203.6, 327.3 / 320.7.
static int32_t step_splits(const LayerWorkspace& w, int32_t n_problems, bool reuses_rows) { return n_problems == 1 && !reuses_rows ? 2 * w.splits - 1 : w.splits; }

// ------------------------------------------------------------------------ layer forward / backward

int32_t sage_forward(const no_block_view& blk, const void* x_src, no_dtype dt, int32_t d_in, const float* w_self,
                     const float* w_neigh, const float* bias, int32_t d_out, int32_t relu, float* mean, float* h,
                     const LayerWorkspace& w, hipStream_t st, StageProfiler* prof, int agg_stage, int gemm_stage,
                     const void* agg_table, int32_t arch, const Layer1Reuse* reuse,
                     bool aggregate_done, const SourceWeights* weights, const PaddedSlots* padded,
                     const Bf16Products* bf, no_blocks_s* side_of, uint16_t* const* cut_fwd, bool cut_done, hipEvent_t product_done, uint8_t* positive) {
    // aggregate_done: `mean` (and the reused rows of H^1) were already written by an earlier launch of the same
    // aggregation (a batch prepared ahead); only the product runs
    // reuse: the output rows are scattered into H^1, recomputed hot rows also refresh the cache, and the reused
    // rows are copied in from the cache by extra blocks of the aggregation launch (they do not depend on this layer)
    const RowCopyJob* hits = (reuse && reuse->hits.dst) ? &reuse->hits : nullptr;
    auto scatter = [&](GemmNNArgs& a) {
        if (!reuse) return;
        a.c_rows = reuse->compute_pos;
        a.c_keep = reuse->emb; a.c_keep_rows = reuse->refresh_slot; a.c_keep_stamp = reuse->version; a.stamp = reuse->step;      // version == NULL: stamped by the split already
    };
    auto product = [&](auto launch) -> int32_t {
        hipEvent_t p0 = nullptr, p1 = nullptr;
        if (prof && gemm_stage >= 0) prof->kernel_pair(gemm_stage, &p0, &p1);
        if (p0 || !product_done) {
            NO_CHECK(launch(p0, p1));
            if (product_done) NO_HIP_CHECK(hipEventRecord(product_done, st));
            return NO_OK;
        }
        return launch(nullptr, product_done);
    };
    // The weights of a product on planes are cut beside the aggregation, which does not read them.
    const bool gcn = arch_is_gcn(arch);
    CutJobs cut;
    uint16_t* own_planes[2];
    const size_t each = cut_weights_elements(d_in, d_out, true);
    auto takes_planes = agg_table ? forward_takes_planes : layer_takes_planes;
    if (!cut_fwd && !bf && takes_planes(blk.n_dst_cap, d_in, d_out, gcn ? 1 : 2) && (gcn ? 1 : 2) * each * 2 <= w.fwd_planes_bytes) {
        own_planes[0] = (uint16_t*)w.fwd_planes;
        own_planes[1] = own_planes[0] + each;
        cut_fwd = own_planes;
    }
    if (cut_fwd && !cut_done) {
        cut.add(w_self, d_in, d_out, cut_fwd[0], true);
        if (!gcn) cut.add(w_neigh, d_in, d_out, cut_fwd[1], true);
    }
    if (gcn) {
        // Eq. 1 over N_in(v) U {v} (the destination's own row joins the aggregate: average, sum, or symmetric
        // normalisation with per-source weights), Eq. 2 with one matrix
        hipEvent_t e0 = nullptr, e1 = nullptr;
        if (prof && agg_stage >= 0 && !aggregate_done) prof->kernel_pair(agg_stage, &e0, &e1);
        if (arch == NO_ARCH_GCN_SYM && !(weights && weights->cnt)) {
            set_error("GCN-style layer with symmetric normalisation: the block has no per-source edge counts");
            return NO_ERR_INVALID_ARG;
        }
        if (!aggregate_done)
            NO_CHECK(mean_aggregate(agg_table ? agg_table : x_src, dt, d_in, blk.d_indptr, blk.d_indices, blk.d_n_dst,
                                blk.n_dst_cap, mean, st, aggregate_mode(arch), agg_table ? blk.d_src_global : nullptr, hits, e0, e1,
                                arch == NO_ARCH_GCN_SYM ? weights : nullptr, agg_table ? padded : nullptr, side_of, &cut));
        GemmNNArgs a{};
        a.A[0] = mean; a.lda[0] = d_in;
        a.B[0] = w_self; a.ldb[0] = d_out;
        a.K[0] = d_in;
        a.C[0] = h; a.ldc[0] = d_out;
        a.n_problems = 1; a.accumulate = 1;
        a.d_M = blk.d_n_dst; a.M_cap = blk.n_dst_cap; a.N = d_out;
        a.bias = bias; a.relu = relu;
        scatter(a);
        a.positive = positive;
        a.cut_B[0] = cut_fwd ? cut_fwd[0] : nullptr;
        return product([&](hipEvent_t p0, hipEvent_t p1) { return gemm_nn_forward(a, st, p0, p1); });
    }
    // agg_table != NULL: the rows to average are rows of that table addressed by blk.d_indices (global ids),
    // while x_src holds only the destination rows (fused gather + aggregate of the bottom layer). An fp32
    // table also feeds the self product directly, row m = table row src_global[m], so the forward pass
    // does not need the dense copy of the destination rows at all.
    const bool direct_self = agg_table && dt == NO_F32 && blk.d_src_global;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (prof && agg_stage >= 0 && !aggregate_done) prof->kernel_pair(agg_stage, &e0, &e1);
    if (!aggregate_done)
        NO_CHECK(mean_aggregate(agg_table ? agg_table : x_src, dt, d_in, blk.d_indptr, blk.d_indices, blk.d_n_dst,
                                blk.n_dst_cap, mean, st, AGG_NEIGH_MEAN, nullptr, hits, e0, e1, nullptr,
                                agg_table ? padded : nullptr, side_of, &cut));
    if (bf) {
        // bf16 operands on the matrix cores: the destinations' rows straight from the table (bf16 as stored), the mean
        // rounded on load, the weights from their bf16 copies
        GemmBf16NNArgs a{};
        a.X = bf->x_table; a.ldx = bf->ldx; a.x_rows = bf->x_rows;
        a.Mn = mean; a.ldm = d_in;
        a.Wt[0] = bf->wt_self; a.Wt[1] = bf->wt_neigh; a.Kpad = bf->Kpad;
        a.K = d_in; a.N = d_out;
        a.C = h; a.ldc = d_out;
        a.d_M = blk.d_n_dst; a.M_cap = blk.n_dst_cap;
        a.bias = bias; a.relu = relu;
        if (reuse) { a.c_rows = reuse->compute_pos; a.c_keep = reuse->emb; a.c_keep_rows = reuse->refresh_slot; }
        a.positive = positive;
        return product([&](hipEvent_t p0, hipEvent_t p1) { return gemm_bf16_nn(a, st, p0, p1); });
    }
    const float* x_dst = direct_self ? (const float*)agg_table : (const float*)x_src;
    if (dt == NO_BF16) {
        NO_CHECK(bf16_rows_to_f32((const uint16_t*)x_src, blk.d_n_dst, blk.n_dst_cap, d_in, w.x_dst_f32, st));
        x_dst = w.x_dst_f32;
    }
    GemmNNArgs a{};
    a.A[0] = x_dst; a.lda[0] = d_in;
    a.a_rows[0] = direct_self ? blk.d_src_global : nullptr;
    a.A[1] = mean;  a.lda[1] = d_in;
    a.B[0] = w_self;  a.ldb[0] = d_out;
    a.B[1] = w_neigh; a.ldb[1] = d_out;
    a.K[0] = a.K[1] = d_in;
    a.C[0] = h; a.ldc[0] = d_out;
    a.n_problems = 2; a.accumulate = 1;
    a.d_M = blk.d_n_dst; a.M_cap = blk.n_dst_cap; a.N = d_out;
    a.bias = bias; a.relu = relu;
    scatter(a);
    a.positive = positive;
    a.cut_B[0] = cut_fwd ? cut_fwd[0] : nullptr;
    a.cut_B[1] = cut_fwd ? cut_fwd[1] : nullptr;
    return product([&](hipEvent_t p0, hipEvent_t p1) { return gemm_nn_forward(a, st, p0, p1); });
}

int32_t sage_backward(const no_block_view& blk, const void* x_src, no_dtype dt, int32_t d_in, const float* mean,
                      const float* h, const float* grad_h, const float* w_self, const float* w_neigh, int32_t d_out,
                      int32_t relu, float* gw_self, float* gw_neigh, float* gbias, float* grad_x_src,
                      const LayerWorkspace& w, hipStream_t st, StageProfiler* prof, int prep_stage, int dw_stage,
                      int reduce_stage, int dx_stage, const int32_t* grad_rows, float lr, float* w_self_rw,
                      float* w_neigh_rw, float* bias_rw, int32_t arch, const StatsJob* stats_job, const float* gz_in,
                      const BelowLayer* below, GradJobs* pending, bool defer, const SourceWeights* weights,
                      const Bf16Products* bf, uint16_t* const* cut_bwd, bool input_products_done) {
    const bool gcn = arch_is_gcn(arch);
    if (arch == NO_ARCH_GCN_SYM && grad_x_src && !(weights && weights->cnt)) {
        set_error("GCN-style layer with symmetric normalisation: the block has no per-source edge counts");
        return NO_ERR_INVALID_ARG;
    }
    const int32_t n_cap = blk.n_dst_cap;
    if (prof && prep_stage >= 0) prof->begin(prep_stage);
    // gz_in: the layer above already applied this layer's ReLU decision and row selection while it wrote the gradient
    const float* gz = gz_in ? gz_in : grad_h;
    uint16_t* own_planes[2];
    if (!gz_in && (relu || grad_rows)) {
        // The weights of a large input gradient are cut beside the masking (a launch of their own: 3 us of the 80 of a layer of 3.4 K
        // rows, 256 x 256).
        CutJobs cut;
        const size_t plane = cut_weights_elements(d_in, d_out);
        if (grad_x_src && !cut_bwd && input_grad_takes_planes(n_cap, d_out, d_in, 2) && (gcn ? 1 : 2) * plane * 2 <= w.planes_bytes) {
            own_planes[0] = w.planes();
            own_planes[1] = own_planes[0] + plane;
            cut.add(w_self, d_in, d_out, own_planes[0]);
            if (!gcn) cut.add(w_neigh, d_in, d_out, own_planes[1]);
            cut_bwd = own_planes;
        }
        const uint32_t own = ew_blocks((int64_t)n_cap * d_out);
        hipLaunchKernelGGL(mask_rows_kernel, dim3(own + cut.blocks()), dim3(256), 0, st, grad_h, grad_rows, h, blk.d_n_dst, n_cap, d_out,
                           relu, w.gz, own, cut);
        gz = w.gz;
    }
    if (prof && prep_stage >= 0) prof->end();
    // weight gradients x_dst^T gz, mean^T gz and the bias gradient (column sums of gz), split over rows and summed in split order
    const float* x_dst = dt == NO_BF16 && !gcn && !bf ? w.x_dst_f32 : (const float*)x_src;
    GemmTNArgs t{};
    t.A[0] = x_dst; t.lda[0] = d_in;
    t.A[1] = mean;  t.lda[1] = d_in;
    if (gcn) { t.A[0] = mean; t.n_problems = 1; }
    t.G = gz; t.ldg = d_out;
    t.P = w.partials; t.Kp = d_in; t.N = d_out;
    t.d_R = blk.d_n_dst; t.R_cap = n_cap; t.splits = pending ? step_splits(w, t.n_problems, pending->reuses_rows) : w.splits; t.plain_splits = layer_splits(n_cap, d_in, d_out);
    t.small_up_to = pending ? 0 : n_cap;      // (a step's batch fills 15 to 45 % of the capacity; a caller's block is its own size)
    // Batches that fill a fraction of the capacity use fewer slices than the capacity-sized bound: a slice keeps at least
    // this many rows. Measured on a batch of 24 K rows (bound: 64 slices): the product takes the same time from 64 down
    // to 93 slices' worth of rows (256 per slice) and 10 % longer at 384 and above (too few blocks), while the reduction
    // after it reads fewer partial tiles.
    // Few rows of a layer with few tiles are cut finer, until there are 256 blocks of small tiles or 64 rows a slice (backward pass, us: 1 K rows,
    // 100 x 47: 25.5 -> 20.1, 128 x 256: 26.1 -> 24.0; 2 K rows, 64 x 64: 24.0 -> 20.4; 5 K rows: 28.9 -> 26.3).
    t.rows_per_split = 256;
    t.few_splits = (int32_t)(256 / (ceil_div(d_in, 64) * ceil_div(d_out, 64) * t.n_problems));
    ReduceArgs r{w.partials, t.splits, d_in, d_out, gw_self, gw_neigh, gbias, lr, w_self_rw, w_neigh_rw, bias_rw, gcn ? 1 : 2};
    if (bf) { r.wt_self = bf->wt_self; r.wt_neigh = bf->wt_neigh; r.Kpad = bf->Kpad; }
    // In a layer call the weight gradients may go with the launch of the input gradient, unless the weights' planes stand where the partials
    // go or the fp32 rows are still to be made.
    const bool together = !pending && !(dt == NO_BF16 && !gcn) &&
                          (gcn ? 1 : 2) * cut_weights_elements(d_in, d_out) * 2 <= (size_t)((char*)w.partials - (char*)w.x_dst_f32);
    bool tn_done = false;
    if (grad_x_src) {
        // uses the pre-update weights, so it runs before the reduce that may apply the SGD step:
        // gz W_self^T -> rows [0, n_dst) of grad_x; (gz W_neigh^T) / len(row) -> gmean; then the transpose adds
        if (prof && dx_stage >= 0) prof->begin(dx_stage);
        GemmNNArgs a{};
        a.A[0] = a.A[1] = gz; a.lda[0] = a.lda[1] = d_out;
        a.B[0] = w_self;  a.ldb[0] = d_out;
        a.B[1] = w_neigh; a.ldb[1] = d_out;
        a.K[0] = a.K[1] = d_out;
        a.C[0] = grad_x_src; a.ldc[0] = d_in;
        a.C[1] = w.gmean;    a.ldc[1] = d_in;
        a.row_scale_indptr[1] = blk.d_indptr;
        if (gcn) {
            // one matrix: gz W^T / (len + 1) is both the destination's own share (rows [0, n_dst) of grad_x) and
            // what the transpose spreads over the sampled sources
            // (sum: no factor; symmetric normalisation: (len + 1)^-1/2 here, the source's own factor after the transpose)
            a.B[1] = w_self;
            a.row_scale_indptr[0] = blk.d_indptr;
            a.row_scale_plus = 1;
            a.row_scale_rsqrt = arch == NO_ARCH_GCN_SYM ? 1 : 0;
            if (arch == NO_ARCH_GCN_SUM) a.row_scale_indptr[0] = a.row_scale_indptr[1] = nullptr;
        }
        a.n_problems = 2; a.accumulate = 0;
        a.cut_B[0] = cut_bwd ? cut_bwd[0] : nullptr;
        a.cut_B[1] = cut_bwd ? cut_bwd[gcn ? 0 : 1] : nullptr;
        a.cut_scratch = w.planes();
        a.cut_scratch_bytes = w.planes_bytes;
        a.d_M = blk.d_n_dst; a.M_cap = n_cap; a.N = d_in;
        if (!input_products_done) NO_CHECK(gemm_nn_input_grad(a, st, together ? &t : nullptr, &tn_done));
        NO_CHECK(transpose_aggregate(w.gmean, d_in, blk.d_csc_indptr, blk.d_csc_dst, blk.d_n_src, blk.n_src_cap,
                                     blk.d_n_dst, grad_x_src, st, below ? below->h : nullptr, below ? below->out_rows : nullptr,
                                     below ? below->gz_out : nullptr, arch == NO_ARCH_GCN_SYM ? weights : nullptr, tn_done ? &r : nullptr, below ? below->positive : nullptr));
        if (prof && dx_stage >= 0) prof->end();
    }
    if (dt == NO_BF16 && !gcn && !bf) NO_CHECK(bf16_rows_to_f32((const uint16_t*)x_src, blk.d_n_dst, n_cap, d_in, w.x_dst_f32, st));
    if (pending && defer) {
        // an upper layer inside a step: its product and reduction ride on the bottom layer's launches
        if (pending->n >= NO_MAX_LAYERS) { set_error("sage_backward: too many deferred layers"); return NO_ERR_CAPACITY; }
        pending->tn[pending->n] = t;
        pending->red[pending->n] = r;
        ++pending->n;
        return launch_status("sage_backward");
    }
    GemmTNArgs tj[NO_MAX_LAYERS];
    ReduceArgs rj[NO_MAX_LAYERS];
    int32_t n_jobs = 0, n_tn = 0;
    rj[n_jobs++] = r;
    if (bf) t.A16 = bf->x_dense;      // this layer's two products take bf16 operands
    tj[n_tn++] = t;
    for (int32_t i = 0; pending && i < pending->n && n_jobs < NO_MAX_LAYERS; ++i) { tj[n_tn++] = pending->tn[i]; rj[n_jobs++] = pending->red[i]; }
    if (pending) pending->n = 0;
    if (tn_done) return launch_status("sage_backward");      // (the reduction went with the transposed sum)
    {
        hipEvent_t e0 = nullptr, e1 = nullptr;
        if (prof && dw_stage >= 0) prof->kernel_pair(dw_stage, &e0, &e1);
        NO_CHECK(gemm_tn_partials(tj, n_tn, st, e0, e1));
    }
    if (prof && reduce_stage >= 0) prof->begin(reduce_stage);
    NO_CHECK(reduce_grads(rj, n_jobs, st, stats_job));
    if (prof && reduce_stage >= 0) prof->end();
    return launch_status("sage_backward");
}

}  // namespace no

using namespace no;

static int32_t check_layer_args(const no_block_view* blk, const void* x, no_dtype dt, int32_t d_in, int32_t d_out,
                                const char* who) {
    NO_REQUIRE(blk && x, NO_ERR_INVALID_ARG, "%s: NULL argument", who);
    NO_REQUIRE(dt == NO_F32 || dt == NO_BF16, NO_ERR_INVALID_ARG, "%s: unknown dtype", who);
    NO_REQUIRE(d_in >= 1 && d_out >= 1, NO_ERR_INVALID_ARG, "%s: dimensions must be positive", who);
    NO_REQUIRE(blk->n_dst_cap >= 1 && blk->n_src_cap >= blk->n_dst_cap, NO_ERR_INVALID_ARG, "%s: bad block capacities", who);
    NO_REQUIRE(blk->d_n_dst && blk->d_indptr && blk->d_indices, NO_ERR_INVALID_ARG, "%s: block view lacks CSR arrays", who);
    return NO_OK;
}

extern "C" size_t no_sage_layer_ws_bytes(int32_t n_dst_cap, int32_t n_src_cap, int32_t d_in, int32_t d_out) {
    (void)n_src_cap;
    if (n_dst_cap < 1 || d_in < 1 || d_out < 1) return 0;
    return carve_workspace(nullptr, n_dst_cap, d_in, d_out).bytes;
}

extern "C" int32_t no_sage_layer_fwd(const no_block_view* blk, const void* d_x_src, no_dtype dt_x, int32_t d_in,
                                     const float* d_w_self, const float* d_w_neigh, const float* d_bias, int32_t d_out,
                                     int32_t relu, float* d_mean, float* d_h, void* d_ws, size_t ws_bytes, void* stream) {
    clear_error();
    NO_CHECK(check_layer_args(blk, d_x_src, dt_x, d_in, d_out, "no_sage_layer_fwd"));
    NO_REQUIRE(d_w_self && d_w_neigh && d_bias && d_mean && d_h, NO_ERR_INVALID_ARG, "no_sage_layer_fwd: NULL argument");
    LayerWorkspace w = carve_workspace(d_ws, blk->n_dst_cap, d_in, d_out);
    NO_REQUIRE(d_ws != nullptr && ws_bytes >= w.bytes, NO_ERR_CAPACITY, "no_sage_layer_fwd: workspace too small (%zu < %zu)",
               ws_bytes, w.bytes);
    return sage_forward(*blk, d_x_src, dt_x, d_in, d_w_self, d_w_neigh, d_bias, d_out, relu, d_mean, d_h, w,
                        (hipStream_t)stream);
}

extern "C" int32_t no_sage_layer_bwd(const no_block_view* blk, const void* d_x_src, no_dtype dt_x, int32_t d_in,
                                     const float* d_mean, const float* d_h, const float* d_grad_h, const float* d_w_self,
                                     const float* d_w_neigh, int32_t d_out, int32_t relu, float* d_gw_self,
                                     float* d_gw_neigh, float* d_gbias, float* d_grad_x_src, void* d_ws, size_t ws_bytes,
                                     void* stream) {
    clear_error();
    NO_CHECK(check_layer_args(blk, d_x_src, dt_x, d_in, d_out, "no_sage_layer_bwd"));
    NO_REQUIRE(d_mean && d_h && d_grad_h && d_w_self && d_w_neigh && d_gw_self && d_gw_neigh && d_gbias, NO_ERR_INVALID_ARG,
               "no_sage_layer_bwd: NULL argument");
    NO_REQUIRE(!d_grad_x_src || (blk->d_csc_indptr && blk->d_csc_dst && blk->d_n_src), NO_ERR_INVALID_ARG,
               "no_sage_layer_bwd: input gradient requested but the block has no transpose");
    LayerWorkspace w = carve_workspace(d_ws, blk->n_dst_cap, d_in, d_out);
    NO_REQUIRE(d_ws != nullptr && ws_bytes >= w.bytes, NO_ERR_CAPACITY, "no_sage_layer_bwd: workspace too small (%zu < %zu)",
               ws_bytes, w.bytes);
    return sage_backward(*blk, d_x_src, dt_x, d_in, d_mean, d_h, d_grad_h, d_w_self, d_w_neigh, d_out, relu, d_gw_self,
                         d_gw_neigh, d_gbias, d_grad_x_src, w, (hipStream_t)stream);
}

// ------------------------------------------------------------------------ backward without any allocation
//
// The workspace of no_sage_layer_bwd (masked gradient, mean gradient, fp32 copy of bf16 rows, split partial products)
// held in a file-scope device array instead of a caller's buffer, for callers that cannot allocate or pass one.
constexpr size_t kStaticWsBytes = NO_LAYER_STATIC_WS_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticWsBytes];

namespace {
constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static void* g_scratch_ptr[kMaxDevices] = {nullptr};

// The address of this device's copy of `scratch` (every GPU holds its own copy at its own address; the array's name
// is only a host-side handle for the lookup and is never passed to a kernel or a memory call).
static int32_t static_workspace(void** out) {
    int dev = -1;
    NO_HIP_CHECK(hipGetDevice(&dev));
    NO_REQUIRE(dev >= 0 && dev < kMaxDevices, NO_ERR_UNSUPPORTED, "static workspace: device index %d not supported", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        NO_HIP_CHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        NO_REQUIRE(p != nullptr, NO_ERR_HIP, "static workspace: no device address for the scratch array");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return NO_OK;
}
}  // namespace

extern "C" int32_t no_sage_layer_bwd_static(const no_block_view* blk, const void* d_x_src, no_dtype dt_x, int32_t d_in,
                                            const float* d_mean, const float* d_h, const float* d_grad_h,
                                            const float* d_w_self, const float* d_w_neigh, int32_t d_out, int32_t relu,
                                            float* d_gw_self, float* d_gw_neigh, float* d_gbias, float* d_grad_x_src,
                                            void* stream) {
    clear_error();
    NO_CHECK(check_layer_args(blk, d_x_src, dt_x, d_in, d_out, "no_sage_layer_bwd_static"));
    NO_REQUIRE(d_mean && d_h && d_grad_h && d_w_self && d_w_neigh && d_gw_self && d_gw_neigh && d_gbias, NO_ERR_INVALID_ARG,
               "no_sage_layer_bwd_static: NULL argument");
    NO_REQUIRE(!d_grad_x_src || (blk->d_csc_indptr && blk->d_csc_dst && blk->d_n_src), NO_ERR_INVALID_ARG,
               "no_sage_layer_bwd_static: input gradient requested but the block has no transpose");
    const size_t need = carve_workspace(nullptr, blk->n_dst_cap, d_in, d_out).bytes;
    NO_REQUIRE(need <= kStaticWsBytes, NO_ERR_CAPACITY,
               "no_sage_layer_bwd_static: the layer needs %zu bytes of workspace, the static one holds %zu", need,
               kStaticWsBytes);
    void* ws = nullptr;
    NO_CHECK(static_workspace(&ws));
    // (every part of the workspace is written by this call's kernels before it is read: nothing has to start at zero)
    LayerWorkspace w = carve_workspace(ws, blk->n_dst_cap, d_in, d_out);
    return sage_backward(*blk, d_x_src, dt_x, d_in, d_mean, d_h, d_grad_h, d_w_self, d_w_neigh, d_out, relu, d_gw_self,
                         d_gw_neigh, d_gbias, d_grad_x_src, w, (hipStream_t)stream);
}

static int32_t check_gcn_form(const no_block_view* blk, no_arch form, SourceWeights* sw, const char* who) {
    NO_REQUIRE(form == NO_ARCH_GCN || form == NO_ARCH_GCN_SUM || form == NO_ARCH_GCN_SYM, NO_ERR_INVALID_ARG,
               "%s: form must be one of the GCN-style layer forms", who);
    *sw = SourceWeights{};
    if (form == NO_ARCH_GCN_SYM) {
        // the column sums of the block's adjacency are the lengths of the transpose's columns
        NO_REQUIRE(blk->d_csc_indptr != nullptr, NO_ERR_INVALID_ARG,
                   "%s: symmetric normalisation needs the block's transpose (its column lengths)", who);
        sw->cnt = blk->d_csc_indptr;
        sw->is_ptr = 1;
    }
    return NO_OK;
}

extern "C" int32_t no_gcn_layer_fwd(const no_block_view* blk, no_arch form, const void* d_x_src, no_dtype dt_x, int32_t d_in,
                                    const float* d_w, const float* d_bias, int32_t d_out, int32_t relu, float* d_agg,
                                    float* d_h, void* d_ws, size_t ws_bytes, void* stream) {
    clear_error();
    NO_CHECK(check_layer_args(blk, d_x_src, dt_x, d_in, d_out, "no_gcn_layer_fwd"));
    SourceWeights sw;
    NO_CHECK(check_gcn_form(blk, form, &sw, "no_gcn_layer_fwd"));
    NO_REQUIRE(d_w && d_bias && d_agg && d_h, NO_ERR_INVALID_ARG, "no_gcn_layer_fwd: NULL argument");
    LayerWorkspace w = carve_workspace(d_ws, blk->n_dst_cap, d_in, d_out);
    NO_REQUIRE(d_ws != nullptr && ws_bytes >= w.bytes, NO_ERR_CAPACITY, "no_gcn_layer_fwd: workspace too small (%zu < %zu)",
               ws_bytes, w.bytes);
    return sage_forward(*blk, d_x_src, dt_x, d_in, d_w, nullptr, d_bias, d_out, relu, d_agg, d_h, w, (hipStream_t)stream,
                        nullptr, -1, -1, nullptr, form, nullptr, false, &sw);
}

extern "C" int32_t no_gcn_layer_bwd(const no_block_view* blk, no_arch form, int32_t d_in, const float* d_agg, const float* d_h,
                                    const float* d_grad_h, const float* d_w, int32_t d_out, int32_t relu, float* d_gw,
                                    float* d_gbias, float* d_grad_x_src, void* d_ws, size_t ws_bytes, void* stream) {
    clear_error();
    NO_CHECK(check_layer_args(blk, d_agg, NO_F32, d_in, d_out, "no_gcn_layer_bwd"));
    SourceWeights sw;
    NO_CHECK(check_gcn_form(blk, d_grad_x_src ? form : (form == NO_ARCH_GCN_SYM ? NO_ARCH_GCN : form), &sw, "no_gcn_layer_bwd"));
    NO_REQUIRE(d_h && d_grad_h && d_w && d_gw && d_gbias, NO_ERR_INVALID_ARG, "no_gcn_layer_bwd: NULL argument");
    NO_REQUIRE(!d_grad_x_src || (blk->d_csc_indptr && blk->d_csc_dst && blk->d_n_src), NO_ERR_INVALID_ARG,
               "no_gcn_layer_bwd: input gradient requested but the block has no transpose");
    LayerWorkspace w = carve_workspace(d_ws, blk->n_dst_cap, d_in, d_out);
    NO_REQUIRE(d_ws != nullptr && ws_bytes >= w.bytes, NO_ERR_CAPACITY, "no_gcn_layer_bwd: workspace too small (%zu < %zu)",
               ws_bytes, w.bytes);
    return sage_backward(*blk, d_agg, NO_F32, d_in, d_agg, d_h, d_grad_h, d_w, nullptr, d_out, relu, d_gw, nullptr, d_gbias,
                         d_grad_x_src, w, (hipStream_t)stream, nullptr, -1, -1, -1, -1, nullptr, 0.f, nullptr, nullptr, nullptr,
                         form, nullptr, nullptr, nullptr, nullptr, false, &sw);
}
