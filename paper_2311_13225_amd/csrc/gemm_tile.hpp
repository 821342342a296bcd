// What the matrix-product kernels share: 4-byte-aligned 16-byte loads, rounding to bf16, the accumulator's
// layout and the dealing of tiles to the dies.
#pragma once
#include "gemm.hpp"

namespace no {

typedef float floatx16 __attribute__((ext_vector_type(16)));

// 16-byte load from a 4-byte aligned address (rows of 602 floats start on 8-byte boundaries only).
typedef float float4_a4 __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ float4 load4_fast(const float* p) {
    float4_a4 v = *reinterpret_cast<const float4_a4*>(p);
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ float4 load4_guarded(const float* p, int valid) {
    if (valid >= 4) return load4_fast(p);      // only the lanes that straddle an edge go element by element
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (valid > 0) v.x = p[0];
    if (valid > 1) v.y = p[1];
    if (valid > 2) v.z = p[2];
    return v;
}

// Two values rounded to bf16, nearest-even, one instruction.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
    const f32x2_t f = {a, b};
    const bf16x2_t r = __builtin_convertvector(f, bf16x2_t);
    uint32_t u;
    __builtin_memcpy(&u, &r, 4);
    return u;
}

// Operands are cut at 2^24 times their size, and the sums brought back (exactly) by 2^-48: the last bit of the smallest fp32 number,
// 2^-149, is then no smaller than the smallest normal bf16 number, so that no piece of any finite operand is lost below the range.
// (An operand from 2^104 or a sum from 2^79 on leaves it at the top: gemm_cut.hip sums those outputs on the fp32 instruction.)
constexpr float CUT_SCALE = 16777216.f, CUT_UNSCALE = 1.f / (CUT_SCALE * CUT_SCALE);

// The partial products of one pair of fragments, smallest first, and the accumulator each goes to.
constexpr int CUT_TERMS = 6;
struct CutTerm { int a, b, acc; };
__device__ constexpr CutTerm CUT_TERM[CUT_TERMS] = {{2, 0, 0}, {0, 2, 0}, {1, 1, 0}, {1, 0, 0}, {0, 1, 0}, {0, 0, 1}};

// Eight values, each cut into three bf16 values (gemm_cut.hip): the three planes (packed in pairs)
__device__ __forceinline__ void cut8(const float (&f)[8], uint4 (&p)[3]) {
    uint32_t h[4], m[4], l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float a = f[2 * i] * CUT_SCALE, b = f[2 * i + 1] * CUT_SCALE;
        h[i] = bf16_pair(a, b);
        a -= __uint_as_float(h[i] << 16);
        b -= __uint_as_float(h[i] & 0xffff0000u);
        m[i] = bf16_pair(a, b);
        a -= __uint_as_float(m[i] << 16);
        b -= __uint_as_float(m[i] & 0xffff0000u);
        l[i] = bf16_pair(a, b);
    }
    p[0] = make_uint4(h[0], h[1], h[2], h[3]);
    p[1] = make_uint4(m[0], m[1], m[2], m[3]);
    p[2] = make_uint4(l[0], l[1], l[2], l[3]);
}

// One unit of a matrix's planes (see cut_weights; i < cut_weights_elements / 24): eight reduction indices of one row of the matrix, or
// (forward) of one column.
__device__ __forceinline__ void cut_weights_unit(const float* w, int32_t K, int32_t N, bool forward, uint16_t* out, int64_t i) {
    const int32_t X = forward ? N : K, R = forward ? K : N;      // the product reduces over R
    const int64_t plane = (int64_t)cut_pad(R) * X;
    const int32_t rb = (int32_t)(i / X), x = (int32_t)(i - (int64_t)rb * X);
    float f[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int32_t r = rb * 8 + j;
        f[j] = r < R ? (forward ? w[(int64_t)r * N + x] : w[(int64_t)x * N + r]) : 0.f;
    }
    uint4 p[3];
    cut8(f, p);
#pragma unroll
    for (int q = 0; q < 3; ++q) *reinterpret_cast<uint4*>(out + i * 8 + q * plane) = p[q];
}

// Block `block` of the extra blocks that carry these jobs (256 threads).
__device__ __forceinline__ void run_cut_jobs(const CutJobs& cut, uint32_t block) {
    int j = 0;
    while (block >= cut.end_block[j]) ++j;
    if (j > 0) block -= cut.end_block[j - 1];
    const int64_t i = (int64_t)block * 256 + threadIdx.x;
    const bool forward = cut.forward >> j & 1;
    if (i < (int64_t)cut_weights_elements(cut.K[j], cut.N[j], forward) / 24) cut_weights_unit(cut.w[j], cut.K[j], cut.N[j], forward, cut.out[j], i);
}

// Which of four neighbouring outputs are positive (GemmNNArgs::positive).
__device__ __forceinline__ uint8_t positive_of(float a, float b, float c, float d) {
    return (uint8_t)((a > 0.f ? 1 : 0) | (b > 0.f ? 2 : 0) | (c > 0.f ? 4 : 0) | (d > 0.f ? 8 : 0));
}

// Accumulator element r of lane: row = 8*(r/4) + 4*(lane/32) + r%4, column = lane%32 of the 32x32 tile.
__device__ __forceinline__ int acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// Eight consecutive reduction indices of one row of A, on their way from memory to LDS.
struct RowUnit {
    float f[8];
    // indices [k, k + 8) of a row of K >= 8 values. Always two loads and no branch around them (the wait before the values are
    // used then counts exactly the loads behind them): a unit that sticks out is read where it ends with the row, or, wholly
    // outside, at the row's start, and put right by trim().
    __device__ __forceinline__ void request(const float* row, int k, int K) {
        const float* p = row + (k + 8 <= K ? k : (k < K ? K - 8 : 0));
        const float4 a = load4_fast(p), b = load4_fast(p + 4);
        f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w; f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
    }
    __device__ __forceinline__ void trim(int k, int K) {
        const int sh = k + 8 <= K ? 0 : (k < K ? k + 8 - K : 8);      // values to shift out
#pragma unroll
        for (int b = 4; b >= 1; b >>= 1)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float from = j + b < 8 ? f[j + b < 8 ? j + b : 0] : 0.f;
                f[j] = (sh & b) ? from : f[j];
            }
#pragma unroll
        for (int j = 0; j < 8; ++j) f[j] = sh >= 8 ? 0.f : f[j];
    }
};

// A block of 256 threads of the reduction of a layer's split products, q = 0 or 1: sums the split partial products in split order: g_self = rows
// [0,Kp) of product 0, g_bias = row Kp of product 0, g_neigh = rows [0,Kp) of product 1. With lr != 0 the parameters take their SGD step in the
// same pass (W <- W - lr * g), after every kernel that read them.
inline int64_t reduce_blocks(const ReduceArgs& a) { return ceil_div((int64_t)(a.Kp + 1) * a.N, 256); }
__device__ __forceinline__ void reduce_block(const ReduceArgs& a, uint32_t block, int q) {
    const int32_t Kp = a.Kp, N = a.N;
    const int32_t splits = *tn_used_word(a.P, a.splits, Kp, N);
    const int64_t per = (int64_t)(Kp + 1) * N;
    const int64_t i = (int64_t)block * 256 + threadIdx.x;
    if (i >= per || q >= a.n_problems) return;
    const bool bias_row = i >= (int64_t)Kp * N;
    if (q == 1 && bias_row) return;
    const float* p = a.P + (int64_t)q * a.splits * per + i;
    // eight partials are requested before the first add; the adds stay in split order
    float s = 0.f;
    int32_t k = 0;
    for (; k + 8 <= splits; k += 8) {
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = p[(int64_t)(k + j) * per];
#pragma unroll
        for (int j = 0; j < 8; ++j) s += v[j];
    }
    for (; k < splits; ++k) s += p[(int64_t)k * per];
    float* gout = bias_row ? a.g_bias + (i - (int64_t)Kp * N) : (q == 0 ? a.g_self + i : a.g_neigh + i);
    *gout = s;
    float* w = a.w_self ? (bias_row ? a.w_bias + (i - (int64_t)Kp * N) : (q == 0 ? a.w_self + i : a.w_neigh + i)) : nullptr;
    if (a.lr != 0.f && w) *w -= a.lr * s;
    if (a.wt_self && w && !bias_row) {
        // the parameter's bf16 copy for the next step's products (transposed: [N][Kpad]), round-to-nearest-even
        const uint32_t u = __float_as_uint(*w);
        const int32_t k = (int32_t)(i / N), n = (int32_t)(i - (int64_t)k * N);
        (q == 0 ? a.wt_self : a.wt_neigh)[(int64_t)n * a.Kpad + k] = (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
    }
}

// Workgroups are handed to the 8 accelerator dies (XCDs, each with its own L2) round-robin by linear
// id. The tiles that share an operand panel (all column tiles of one row tile; all tiles of one
// reduction slice) get consecutive *logical* ids, and logical ids are dealt out in chunks per XCD, so
// a panel is fetched into one L2 once instead of into several.
constexpr int N_XCD = 8;
__device__ __forceinline__ int64_t xcd_logical_id(int64_t total_padded) {
    const int64_t id = blockIdx.x;
    return (id % N_XCD) * (total_padded / N_XCD) + id / N_XCD;
}
static inline unsigned xcd_padded(int64_t total) { return (unsigned)(ceil_div(total, N_XCD) * N_XCD); }

}  // namespace no
