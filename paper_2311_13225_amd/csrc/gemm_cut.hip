// The gradients' fp32 matrix products on the bf16 matrix cores (v_mfma_f32_32x32x16_bf16, 16 times the rate of the fp32
// instruction).
//
// Every fp32 operand value is cut into three bf16 values, high + middle + low, each the nearest bf16 of what the ones
// before it left over: 3 x 8 significand bits hold all 24 of an fp32 number, so nothing of a finite input is lost (at the ends of the
// range either: CUT_SCALE). A product of two such sums is nine partial products, each exact in fp32; the six largest are accumulated
// in fp32 (high x high, high x middle, middle x high, middle x middle, high x low, low x high). With |middle| <= 2^-8 and |low| <= 2^-17
// of a value, the three left out are at most 2^-24.0 of the product together, what one fp32 rounding may be off (2^-27.5 in the
// root mean square over random significands). The largest partial product has an accumulator of its own, which is therefore
// rounded once per 16 terms (the fp32 instruction: 8 times).
// Measured against fp64 on random operands, relative 2-norm error of a weight gradient over 25 K rows / an input gradient over
// 256 columns: fp32 instruction 3.0e-7 / 2.1e-7, this 1.9e-7 / 1.0e-7 (with one accumulator for all six 3.8e-7 / 2.4e-7).
//
// Outputs that do not come out finite (an infinite or NaN operand, one that left the range when it was scaled or rounded to its high
// piece, or a sum that did) are summed again on the fp32 instruction from the uncut operands, by the wavefront that owns them
// and in the same launch: such an output is what the fp32 instruction makes of it, whatever it is. (Backward pass of a layer of
// 3.4 K rows, 256 x 256: 40 us; with NaN everywhere 87, with one NaN in the gradient 73. Summed one by one: 2594 and 632.)
//
// Bound: 6 bf16 products per term are 416 TFLOP/s of fp32 products against the fp32 instruction's 157; next to them stand
// the vector instructions that cut the operands (5.5 an element). So an element is cut as few times as possible: weights
// once per step (or call), into the order in which the matrix cores take them; rows once per 128 output columns.
// Measured, fp32 instruction -> this: input gradient of 60 K x 256 rows by two 256 x 256 matrices 176 -> 108 us, 5.5 K rows 21 -> 16;
// weight gradients of 25 K rows, 2 x 100 x 256: 47 -> 35 us, of 60 K rows, 2 x 256 x 256: 194 -> 130.
// (Forward products: gemm_fwd.hip.)
#include <algorithm>

#include "gemm_tile.hpp"

namespace no {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

constexpr int SK = 32;              // reduction indices per step
constexpr int SPITCH = SK + 8;      // bf16 elements per LDS row: rows start 20 banks apart

__device__ __forceinline__ bf16x8_t cut_fragment(const uint16_t* p) {
    bf16x8_t v;
    __builtin_memcpy(&v, __builtin_assume_aligned(p, 16), 16);
    return v;
}

__device__ __forceinline__ bool finite(float v) { return fabsf(v) < INFINITY; }
// z stays 0 while every value that was added is finite, and is NaN from then on (one instruction a value, no lane mask)
__device__ __forceinline__ void note_not_finite(float& z, float v) { z = fmaf(v, 0.f, z); }

// ------------------------------------------------------------------------------------------ weights

// The transposes of both matrices of a layer ([K][N] fp32, row-major) cut into planes: out[matrix][plane][N/8][K][8], eight indices of the
// reduction (over the columns) together, zeros from N to the next multiple of 32. forward: the matrices themselves, out[..][K/8][N][8].
__global__ void __launch_bounds__(256) cut_weights_kernel(const float* __restrict__ w0, const float* __restrict__ w1, int32_t K, int32_t N,
                                                          int32_t forward, uint16_t* __restrict__ out, int64_t matrix_stride) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < matrix_stride / 24) cut_weights_unit(blockIdx.y ? w1 : w0, K, N, forward != 0, out + blockIdx.y * matrix_stride, i);
}

int32_t cut_weights(const float* w0, const float* w1, int32_t K, int32_t N, bool forward, uint16_t* out, hipStream_t st) {
    const int64_t stride = (int64_t)cut_weights_elements(K, N, forward), units = stride / 24;
    hipLaunchKernelGGL(cut_weights_kernel, dim3((unsigned)ceil_div(units, 256), w1 ? 2u : 1u), dim3(256), 0, st, w0, w1, K, N, forward ? 1 : 0, out, stride);
    return launch_status("cut_weights");
}

__global__ void __launch_bounds__(256) cut_all_kernel(CutJobs cut) { run_cut_jobs(cut, blockIdx.x); }

int32_t cut_all(const CutJobs& cut, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
    if (cut.n == 0) return NO_OK;
    NO_LAUNCH_TIMED(cut_all_kernel, dim3(cut.blocks()), dim3(256), st, ev0, ev1, cut);
    return launch_status("cut_all");
}

// ------------------------------------------------------------------------------------------ NN

// Block: WM x WN wavefronts (WM * WN = 4), each 32 MI rows x 32 NJ columns. Rows of A are cut once per block, into one of two
// LDS copies while the other is multiplied (one barrier per 32 indices), two steps ahead in registers; fragments of B come
// straight from their planes (a lane's eight indices are 16 contiguous bytes, the 32 lanes of a fragment 512: L2 reads, one
// step ahead). What is left at 60 K rows is memory next to the products: without the loads of B the launch takes 81 of 101 us,
// without either operand's 70.
template <int MI, int NJ, int WN>
struct NNTile {
    static constexpr int BM = 32 * MI * (4 / WN), BN = 32 * NJ * WN, COPY = 3 * BM * SPITCH, CPITCH = 32 * NJ + 4;
    static constexpr int BYTES = 2 * COPY * 2 > 4 * 32 * CPITCH * 4 ? 2 * COPY * 2 : 4 * 32 * CPITCH * 4;
};
template <int MI, int NJ, int WN>
__device__ __forceinline__ void cut_nn_tile(const GemmNNArgs& g, unsigned char* smem /* [BYTES] */, float* scale_sh /* [BM] */) {
    using Tile = NNTile<MI, NJ, WN>;
    constexpr int BM = Tile::BM, BN = Tile::BN, PLANE = BM * SPITCH, COPY = Tile::COPY;
    constexpr int UNITS = BM >= 64 ? BM / 64 : 1, CW = 32 * NJ, CPITCH = Tile::CPITCH;
    uint16_t* As = reinterpret_cast<uint16_t*>(smem);
    int M = *g.d_M;
    if (M > g.M_cap) M = g.M_cap;
    // the grid covers the row capacity; only the tiles of the actual M rows are dealt out to the XCDs
    const int gx = (g.N + BN - 1) / BN, gy = (M + BM - 1) / BM, gz = g.n_problems;
    const int64_t total = (int64_t)gx * gy * gz, padded = (total + N_XCD - 1) / N_XCD * N_XCD;
    if ((int64_t)blockIdx.x >= padded) return;
    const int64_t lid = xcd_logical_id(padded);
    if (lid >= total) return;
    const int bx = (int)(lid % gx), by = (int)((lid / gx) % gy), bz = (int)(lid / ((int64_t)gx * gy));
    const int m0 = by * BM, prob = bz;
    const int tid = (int)threadIdx.x, wave = tid >> 6, wm = wave / WN, wn = wave % WN;
    const int lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int c0 = bx * BN + wn * CW;                  // this wavefront's columns
    const bool wave_on = c0 < g.N;                     // (one without columns multiplies the last ones again and stores nothing)
    floatx16 acc[2][MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[0][i][j][r] = acc[1][i][j][r] = 0.f;
    // this thread's rows of A (rows past the operand repeat the last one and are never stored)
    const bool loads = BM >= 64 || tid < BM * 4;
    const int kq = (tid & 3) * 8;
    const float* arow[UNITS];
#pragma unroll
    for (int i = 0; i < UNITS; ++i) arow[i] = g.A[prob] + (int64_t)min(m0 + ((tid + 256 * i) >> 2) % BM, M - 1) * g.lda[prob];
    if (tid < BM) {
        const int row = min(m0 + tid, M - 1);
        const int32_t* sp = g.row_scale_indptr[prob];
        float s = 1.f;
        if (sp) {
            const int len = sp[row + 1] - sp[row] + g.row_scale_plus;
            s = len > 0 ? (g.row_scale_rsqrt ? 1.f / sqrtf((float)len) : 1.f / (float)len) : 0.f;
        }
        scale_sh[tid] = s * CUT_UNSCALE;
    }
    const int K = g.K[prob], N = g.N, steps = cut_pad(K) / SK;
    RowUnit ta[2][UNITS];
    auto request_a = [&](RowUnit (&t)[UNITS], int s) {      // (past the last step: that one again, not used)
#pragma unroll
        for (int i = 0; i < UNITS; ++i) t[i].request(arow[i], min(s, steps - 1) * SK + kq, K);
    };
    auto store_a = [&](RowUnit (&t)[UNITS], int s, uint16_t* S) {
        const int k0 = s * SK;
        if (k0 + SK > K) {
#pragma unroll
            for (int i = 0; i < UNITS; ++i) t[i].trim(k0 + kq, K);
        }
        if (loads) {
#pragma unroll
            for (int i = 0; i < UNITS; ++i) {
                uint4 p[3];
                cut8(t[i].f, p);
                uint16_t* at = S + ((tid + 256 * i) >> 2) * SPITCH + kq;
#pragma unroll
                for (int q = 0; q < 3; ++q) *reinterpret_cast<uint4*>(at + q * PLANE) = p[q];
            }
        }
    };
    // Fragments of B for step s (two halves of 16 indices): uniform base, this lane's offset within two blocks of eight.
    uint32_t boff[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) boff[j] = (uint32_t)(half * N + min(c0 + j * 32 + l32, N - 1)) * 16u;
    const char* const B = reinterpret_cast<const char*>(g.cut_B[prob]);
    const int64_t plane = (int64_t)cut_pad(K) * N * 2;
    auto request_b = [&](bf16x8_t (&b)[2][NJ][3], int s) {
        const char* base = B + (int64_t)min(s, steps - 1) * N * 64;
#pragma unroll
        for (int p = 0; p < 3; ++p, base += plane)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int j = 0; j < NJ; ++j) b[h][j][p] = cut_fragment(reinterpret_cast<const uint16_t*>(base + (int64_t)h * N * 32 + boff[j]));
    };
    auto multiply = [&](const uint16_t* S, const bf16x8_t (&b)[NJ][3], int ks) {
        bf16x8_t a[MI][3];
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int p = 0; p < 3; ++p) a[i][p] = cut_fragment(S + p * PLANE + ((wm * MI + i) * 32 + l32) * SPITCH + ks * 16 + half * 8);
#pragma unroll
        for (int t = 0; t < CUT_TERMS; ++t)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    acc[CUT_TERM[t].acc][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][CUT_TERM[t].a], b[j][CUT_TERM[t].b],
                                                                                          acc[CUT_TERM[t].acc][i][j], 0, 0, 0);
    };
    bf16x8_t b0[2][NJ][3], b1[2][NJ][3];
    request_a(ta[0], 0);
    request_a(ta[1], 1);
    request_b(b0, 0);
    store_a(ta[0], 0, As);
    request_a(ta[0], 2);
    __syncthreads();
    auto step = [&](int s, uint16_t* cur, uint16_t* nxt, RowUnit (&t)[UNITS], bf16x8_t (&b)[2][NJ][3], bf16x8_t (&next_b)[2][NJ][3]) {
        request_b(next_b, s + 1);
        multiply(cur, b[0], 0);
        if (s + 1 < steps) store_a(t, s + 1, nxt);
        request_a(t, s + 3);
        multiply(cur, b[1], 1);
        __syncthreads();
    };
    for (int s = 0; s < steps; s += 2) {
        step(s, As, As + COPY, ta[1], b0, b1);
        if (s + 1 < steps) step(s + 1, As + COPY, As, ta[0], b1, b0);
    }
    // Epilogue: a wavefront's 32 x 64 tiles go through LDS (its own part, over the operand copies) so that a lane stores 16
    // contiguous bytes of an output row: whole 256-byte row segments per 16 lanes.
    float* Ct = reinterpret_cast<float*>(smem) + wave * 32 * CPITCH;
    float* C = g.C[prob];
    const int64_t ldc = g.ldc[prob];
    constexpr int QL = CW / 4, RL = 64 / QL;             // lanes to a row, rows to an instruction
    const int c4 = lane % QL * 4, col = c0 + c4;
    const bool vec = (ldc % 4 == 0) && ((reinterpret_cast<uintptr_t>(C) & 15) == 0) && col + 4 <= N;
    float bad = 0.f;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        if (wave_on) {
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) Ct[acc_row(r, lane) * CPITCH + j * 32 + l32] = acc[1][i][j][r] + acc[0][i][j][r];
        }
        __syncthreads();
        if (wave_on) {
#pragma unroll
            for (int q = 0; q < 32 / RL; ++q) {
                const int lr = q * RL + lane / QL, row = (wm * MI + i) * 32 + lr;
                if (m0 + row >= M || col >= N) continue;
                float4 t = *reinterpret_cast<const float4*>(Ct + lr * CPITCH + c4);
                note_not_finite(bad, t.x); note_not_finite(bad, t.y); note_not_finite(bad, t.z); note_not_finite(bad, t.w);
                const float s = scale_sh[row];
                t.x *= s; t.y *= s; t.z *= s; t.w *= s;
                float* dst = C + (int64_t)(m0 + row) * ldc + col;
                if (vec) {
                    *reinterpret_cast<float4*>(dst) = t;
                } else {
                    const float v[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (col + e < N) dst[e] = v[e];
                }
            }
        }
        if (i + 1 < MI) __syncthreads();
    }
    if (!__any(bad != 0.f)) return;      // (a loop of its own: beside the stores it would cost every call 1 to 3 %)
    __threadfence_block();        // (the lanes read each other's stores)
    // Some output of this wavefront is not finite: its products once more on the fp32 instruction, from memory (a lane brings four
    // consecutive indices of a row of A and of a column of B, lanes 0-31 the first four of eight, as in gemm_nn_small_kernel).
    const float *pa[MI], *pb[NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i) pa[i] = g.A[prob] + (int64_t)min(m0 + (wm * MI + i) * 32 + l32, M - 1) * g.lda[prob];
#pragma unroll
    for (int j = 0; j < NJ; ++j) pb[j] = g.B[prob] + (int64_t)min(c0 + j * 32 + l32, N - 1) * g.ldb[prob];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[0][i][j][r] = 0.f;
    auto add = [&](const float4 (&a)[MI], const float4 (&b)[NJ]) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                acc[0][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i].x, b[j].x, acc[0][i][j], 0, 0, 0);
                acc[0][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i].y, b[j].y, acc[0][i][j], 0, 0, 0);
                acc[0][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i].z, b[j].z, acc[0][i][j], 0, 0, 0);
                acc[0][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i].w, b[j].w, acc[0][i][j], 0, 0, 0);
            }
    };
    constexpr int U = 4;      // loads of so many groups of eight indices in flight
    int k = half * 4;
    for (; k - half * 4 + 8 * U <= K; k += 8 * U) {
        float4 a[U][MI], b[U][NJ];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int i = 0; i < MI; ++i) a[u][i] = load4_fast(pa[i] + k + 8 * u);
#pragma unroll
            for (int j = 0; j < NJ; ++j) b[u][j] = load4_fast(pb[j] + k + 8 * u);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) add(a[u], b[u]);
    }
    for (; k - half * 4 < K; k += 8) {
        float4 a[MI], b[NJ];
#pragma unroll
        for (int i = 0; i < MI; ++i) a[i] = load4_guarded(pa[i] + k, K - k);
#pragma unroll
        for (int j = 0; j < NJ; ++j) b[j] = load4_guarded(pb[j] + k, K - k);
        add(a, b);
    }
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = (wm * MI + i) * 32 + acc_row(r, lane), n = c0 + j * 32 + l32;
                if (m0 + row >= M || n >= N) continue;
                float* dst = C + (int64_t)(m0 + row) * ldc + n;
                if (!finite(*dst)) *dst = acc[0][i][j][r] * (scale_sh[row] * (1.f / CUT_UNSCALE));
            }
}

template <int MI, int NJ, int WN>
__global__ void __launch_bounds__(256, 2) cut_nn_kernel(GemmNNArgs g) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[NNTile<MI, NJ, WN>::BYTES];
    __shared__ float scale_sh[NNTile<MI, NJ, WN>::BM];
    cut_nn_tile<MI, NJ, WN>(g, smem, scale_sh);
}

// ------------------------------------------------------------------------------------------ TN

// W neighbouring columns (2 or 4) of eight consecutive rows, on their way from memory to LDS: eight loads of 4 W bytes, turned in
// registers into W units of eight reduction indices.
template <int W>
struct ColumnUnit {
    typedef float vec __attribute__((ext_vector_type(W)));
    typedef float vec_a4 __attribute__((ext_vector_type(W), aligned(4)));
    vec f[8];
    __device__ __forceinline__ void request(const float* p, int64_t ld) {
#pragma unroll
        for (int j = 0; j < 8; ++j) f[j] = *reinterpret_cast<const vec_a4*>(p + (int64_t)j * ld);
    }
    __device__ __forceinline__ void request_short(const float* p, int64_t ld, int rows, int cols) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int c = 0; c < W; ++c) f[j][c] = j < rows && c < cols ? p[(int64_t)j * ld + c] : 0.f;
    }
    // Columns of a bf16 operand: two to a float's place until spread() is called, which waits for them.
    typedef uint32_t raw __attribute__((ext_vector_type(W / 2)));
    typedef uint32_t raw_a2 __attribute__((ext_vector_type(W / 2), aligned(2)));
    __device__ __forceinline__ void request(const uint16_t* p, int64_t ld) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const raw v = *reinterpret_cast<const raw_a2*>(p + (int64_t)j * ld);
#pragma unroll
            for (int c = 0; c < W / 2; ++c) f[j][c] = __uint_as_float(v[c]);
        }
    }
    __device__ __forceinline__ void request_short(const uint16_t* p, int64_t ld, int rows, int cols) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            uint32_t v[W];
#pragma unroll
            for (int c = 0; c < W; ++c) v[c] = j < rows && c < cols ? p[(int64_t)j * ld + c] : 0u;
#pragma unroll
            for (int c = 0; c < W / 2; ++c) f[j][c] = __uint_as_float(v[2 * c] | (v[2 * c + 1] << 16));
        }
    }
    __device__ __forceinline__ void spread() {
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int c = W / 2 - 1; c >= 0; --c) {
                const uint32_t v = __float_as_uint(f[j][c]);
                f[j][2 * c + 1] = __uint_as_float(v & 0xffff0000u);
                f[j][2 * c] = __uint_as_float(v << 16);
            }
    }
};

// The jobs of one launch (by value in the kernel arguments): job j owns the linear block ids [end_block[j-1], end_block[j]).
struct CutTNLaunch { GemmTNArgs job[NO_MAX_LAYERS]; uint32_t end_block[NO_MAX_LAYERS]; int32_t n; };

// A job takes the larger tiles (fewer cuts per product) where they make blocks with products for most compute units, a function of the
// batch's row count (backward pass of a layer, us, in large tiles / in small ones: 56 blocks, 3.4 K rows, 128 x 256: 47 / 39; 80 blocks, 5 K
// rows, 128 x 256: 50 / 42; 112 blocks, 3.4 K rows, 256 x 256: 52 / 45; 128 blocks, 8 K rows: 128 x 256 57 / 55, 256 x 128 61 / 63; 160 blocks:
// 5 K rows, 256 x 256 60 / 61, 10 K rows, 128 x 256 69 / 63; 256 blocks, 16 K rows: 85 / 86; 8 K rows, 256 x 256: 78 / 82), unless it is narrow (60 K
// rows: 256 x 2 192 / 164; 256 x 16 152 / 143; 3 x 256 121 / 84); its share of the grid is sized for either.
constexpr uint32_t TN_LARGE_BLOCKS = 160;
constexpr int tn_shared_bytes(int T) { return 6 * T * SPITCH * 2 > T * (T + 4) * 4 ? 6 * T * SPITCH * 2 : T * (T + 4) * 4; }

// Block `id` of a job: a T x T tile of one product over one slice; 2 x 2 wavefronts. Half of the threads bring a tile of A, the
// other half one of G, each W = T / 32 columns x eight rows. Column W q + c of a tile stands in LDS row 32 c + q (a
// wavefront then writes neighbouring rows); the output tile is put back in order on its way through LDS. The bias gradient, the column sums of G,
// is added up by the blocks of product 0's first row tile from the rows that they bring.
// The tiles of a slice read the same rows, so they get consecutive logical ids, dealt to the dies in chunks (a job starts at a multiple of the
// dies), and a slice is fetched into one L2 (10 K rows, 2 x 602 x 256: the loads alone 30 -> 18 us, the launch 57.3 -> 55.6).
// BF16: the operands are taken in bf16 instead (the first as it is stored, the others rounded to nearest-even), so there is one
// plane and one partial product; the bias gradient stays the fp32 column sum.
template <int T, bool BF16>
__device__ __forceinline__ void cut_tn_tile(const GemmTNArgs& g, uint32_t id, int R, int used, unsigned char* smem) {
    constexpr int W = T / 32, Q = 32, PLANE = T * SPITCH, OPITCH = T + 4, I = T / 64, PLANES = BF16 ? 1 : 3;
    uint16_t* As = reinterpret_cast<uint16_t*>(smem);
    uint16_t* Gs = As + PLANES * PLANE;
    const uint32_t gx = (uint32_t)((g.N + T - 1) / T), gy = (uint32_t)((g.Kp + T - 1) / T);
    const uint32_t per = gx * gy * (uint32_t)g.n_problems, total = per * (uint32_t)used, padded = (total + N_XCD - 1) / N_XCD * N_XCD;
    if (id >= padded) return;
    const uint32_t lid = id % N_XCD * (padded / N_XCD) + id / N_XCD, rem = lid % per;
    if (lid >= total) return;
    const int split = (int)(lid / per), bx = (int)(rem % gx), by = (int)((rem / gx) % gy), prob = (int)(rem / (gx * gy));
    int chunk = (R + used - 1) / used;
    chunk = (chunk + SK - 1) / SK * SK;
    const int r0 = split * chunk, r1 = min(R, r0 + chunk);
    const int m0 = by * T, n0 = bx * T, tid = (int)threadIdx.x;
    float* P = g.P + ((int64_t)prob * g.splits + split) * (int64_t)(g.Kp + 1) * g.N;
    const int wave = tid >> 6, wm = wave >> 1, wn = wave & 1, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    floatx16 acc[BF16 ? 1 : 2][I][I];
#pragma unroll
    for (int i = 0; i < I; ++i)
#pragma unroll
        for (int j = 0; j < I; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[0][i][j][r] = acc[BF16 ? 0 : 1][i][j][r] = 0.f;
    // this thread's W columns and its eight rows of a step
    const bool mine_a = wave < 2;
    const float* src = mine_a ? g.A[prob] : g.G;
    const bool src16 = BF16 && mine_a && prob == 0;               // (uniform in a wavefront)
    const int64_t ld = mine_a ? g.lda[prob] : g.ldg;
    const int q = tid % Q, k8 = (tid % 128) / Q * 8;
    const int col = (mine_a ? m0 : n0) + q * W, lim = mine_a ? g.Kp : g.N;
    const bool sums = prob == 0 && by == 0;
    double sum[W];      // (in 64 bits: no less exact than the product with a column of ones that this replaces)
#pragma unroll
    for (int c = 0; c < W; ++c) sum[c] = 0.0;
    // Columns past the operand are never stored, but must be read inside it: a unit that sticks out is read where it ends with
    // the row and shifted.
    const bool edge = m0 + T > g.Kp || n0 + T > g.N;
    const int col_r = max(0, min(col, lim - W)), sh = col - col_r;
    uint16_t* S = (mine_a ? As : Gs) + q * SPITCH + k8;
    auto store = [&](ColumnUnit<W>& u, int lo, int hi, int shift) {       // rows [lo, hi) of the 32 count
        if (src16) u.spread();
        if (edge) {
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int c = 0; c < W; ++c) {
                    float v = u.f[j][c];
#pragma unroll
                    for (int b = 1; c + b < W; ++b) v = shift == b ? u.f[j][c + b] : v;
                    u.f[j][c] = v;
                }
        }
        if (lo > 0 || hi < SK) {
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int c = 0; c < W; ++c) u.f[j][c] = k8 + j >= lo && k8 + j < hi ? u.f[j][c] : 0.f;
        }
        if (sums && !mine_a) {
#pragma unroll
            for (int c = 0; c < W; ++c)
#pragma unroll
                for (int j = 0; j < 8; ++j) sum[c] += (double)u.f[j][c];
        }
#pragma unroll
        for (int c = 0; c < W; ++c) {
            float f[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) f[j] = u.f[j][c];
            if (BF16) {
                *reinterpret_cast<uint4*>(S + c * Q * SPITCH) =
                    make_uint4(bf16_pair(f[0], f[1]), bf16_pair(f[2], f[3]), bf16_pair(f[4], f[5]), bf16_pair(f[6], f[7]));
            } else {
                uint4 p[3];
                cut8(f, p);
#pragma unroll
                for (int e = 0; e < 3; ++e) *reinterpret_cast<uint4*>(S + e * PLANE + c * Q * SPITCH) = p[e];
            }
        }
    };
    auto multiply = [&]() {
#pragma unroll
        for (int ks = 0; ks < SK / 16; ++ks) {
            bf16x8_t a[I][PLANES], b[I][PLANES];
#pragma unroll
            for (int i = 0; i < I; ++i)
#pragma unroll
                for (int p = 0; p < PLANES; ++p) {
                    a[i][p] = cut_fragment(As + p * PLANE + (wm * (T / 2) + i * 32 + l32) * SPITCH + ks * 16 + half * 8);
                    b[i][p] = cut_fragment(Gs + p * PLANE + (wn * (T / 2) + i * 32 + l32) * SPITCH + ks * 16 + half * 8);
                }
#pragma unroll
            for (int t = BF16 ? CUT_TERMS - 1 : 0; t < CUT_TERMS; ++t)       // (the last: high x high)
#pragma unroll
                for (int i = 0; i < I; ++i)
#pragma unroll
                    for (int j = 0; j < I; ++j)
                        acc[BF16 ? 0 : CUT_TERM[t].acc][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][CUT_TERM[t].a], b[j][CUT_TERM[t].b],
                                                                                              acc[BF16 ? 0 : CUT_TERM[t].acc][i][j], 0, 0, 0);
        }
    };
    const int steps = r0 < r1 ? (r1 - r0 + SK - 1) / SK : 0;
    if (r1 - r0 >= SK && g.Kp >= W && g.N >= W) {
        // the last step is moved back to end with the slice, and the rows it shares with the step before it count nothing
        const float* p = src + col_r + (int64_t)k8 * ld;
        ColumnUnit<W> u0, u1;
        const uint16_t* p16 = BF16 ? g.A16 + col_r + (int64_t)k8 * ld : nullptr;
        auto request = [&](ColumnUnit<W>& u, int s) {
            const int64_t at = (int64_t)min(r0 + s * SK, r1 - SK) * ld;
            if (src16) u.request(p16 + at, ld);
            else u.request(p + at, ld);
        };
        auto step = [&](ColumnUnit<W>& u, int s) {
            if (s > 0) __syncthreads();
            store(u, max(0, r0 + (s + 1) * SK - r1), SK, sh);
            __syncthreads();
            request(u, s + 2);                   // two steps ahead (past the end: the last rows again, not used)
            multiply();
        };
        request(u0, 0);
        request(u1, 1);
        for (int s = 0; s < steps; s += 2) {
            step(u0, s);
            if (s + 1 < steps) step(u1, s + 1);
        }
    } else {
        ColumnUnit<W> u;
        auto request = [&](int s) {
            const int64_t at = col + (int64_t)(r0 + s * SK + k8) * ld;
            const int rows = r1 - (r0 + s * SK + k8);
            if (src16) u.request_short(g.A16 + at, ld, rows, lim - col);
            else u.request_short(src + at, ld, rows, lim - col);
        };
        if (steps > 0) request(0);
        for (int s = 0; s < steps; ++s) {
            if (s > 0) __syncthreads();
            store(u, 0, min(SK, r1 - (r0 + s * SK)), 0);
            __syncthreads();
            if (s + 1 < steps) request(s + 1);
            multiply();
        }
    }
    float* Cs = reinterpret_cast<float*>(smem);
    float bad = 0.f;
    __syncthreads();
    if (sums) {      // four groups of rows, in order
        if (!mine_a) {
#pragma unroll
            for (int c = 0; c < W; ++c) reinterpret_cast<double*>(smem)[k8 / 8 * T + q * W + c] = sum[c];
        }
        __syncthreads();
        const double* part = reinterpret_cast<const double*>(smem) + tid;
        if (tid < T && n0 + tid < g.N) P[(int64_t)g.Kp * g.N + n0 + tid] = (float)(((part[0] + part[T]) + part[2 * T]) + part[3 * T]);
        __syncthreads();
    }
    // the output tile through LDS, its rows and columns back in order
#pragma unroll
    for (int i = 0; i < I; ++i)
#pragma unroll
        for (int j = 0; j < I; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int x = wm * (T / 2) + i * 32 + acc_row(r, lane), y = wn * (T / 2) + j * 32 + l32;
                const float v = BF16 ? acc[0][i][j][r] : (acc[BF16 ? 0 : 1][i][j][r] + acc[0][i][j][r]) * CUT_UNSCALE;
                Cs[(x % Q * W + x / Q) * OPITCH + y % Q * W + y / Q] = v;
                if (!BF16) note_not_finite(bad, v);
            }
    __syncthreads();
    constexpr int C4 = T / 4;
    const int c4 = tid % C4 * 4, n = n0 + c4;
    const bool vec = (g.N % 4 == 0) && ((reinterpret_cast<uintptr_t>(P) & 15) == 0) && n + 4 <= g.N;
#pragma unroll 4
    for (int lr = tid / C4; lr < T; lr += 256 / C4) {
        const int row = m0 + lr;
        if (row >= g.Kp || n >= g.N) continue;
        const float4 t = *reinterpret_cast<const float4*>(&Cs[lr * OPITCH + c4]);
        float* dst = P + (int64_t)row * g.N + n;
        if (vec) *reinterpret_cast<float4*>(dst) = t;
        else {
            const float v[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n + e < g.N) dst[e] = v[e];
        }
    }
    if (BF16 || !__any(bad != 0.f)) return;
    // Some output of this wavefront is not finite: its products once more on the fp32 instruction, from memory (two rows of the
    // operands at a time, lanes 0-31 the first of them, a column a lane: the one whose LDS row the lane's fragment was).
    auto column = [](int x) { return x % Q * W + x / Q; };
    const float *pa[I], *pg[I];
#pragma unroll
    for (int i = 0; i < I; ++i) {
        const int m = m0 + column(wm * (T / 2) + i * 32 + l32);
        pa[i] = g.A[prob] + min(m, g.Kp - 1);
        pg[i] = g.G + min(n0 + column(wn * (T / 2) + i * 32 + l32), g.N - 1);
#pragma unroll
        for (int j = 0; j < I; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[0][i][j][r] = 0.f;
    }
    constexpr int U = 8;      // pairs of rows in flight
    for (int r = r0; r < r1; r += 2 * U) {
        float a[U][I], b[U][I];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int at = r + 2 * u + half;
            const bool in = at < r1;
#pragma unroll
            for (int i = 0; i < I; ++i) {
                const float va = pa[i][(int64_t)min(at, r1 - 1) * g.lda[prob]], vb = pg[i][(int64_t)min(at, r1 - 1) * g.ldg];
                a[u][i] = in ? va : 0.f;
                b[u][i] = in ? vb : 0.f;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < I; ++i)
#pragma unroll
                for (int j = 0; j < I; ++j) acc[0][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u][i], b[u][j], acc[0][i][j], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < I; ++i)
#pragma unroll
        for (int j = 0; j < I; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int x = column(wm * (T / 2) + i * 32 + acc_row(r, lane)), y = column(wn * (T / 2) + j * 32 + l32);
                if (m0 + x >= g.Kp || n0 + y >= g.N || finite(Cs[x * OPITCH + y])) continue;
                P[(int64_t)(m0 + x) * g.N + n0 + y] = acc[0][i][j][r];
            }
}

static __host__ __device__ inline uint32_t tn_tiles(const GemmTNArgs& g, int T) {
    return (uint32_t)((g.N + T - 1) / T) * (uint32_t)((g.Kp + T - 1) / T) * (uint32_t)g.n_problems;
}

// A product with a side this short fills a quarter of a larger tile and is cut no less often in small ones.
static __host__ __device__ inline bool tn_narrow(const GemmTNArgs& g) { return g.N <= 32 || g.Kp <= 32; }

// The slices of a job in large tiles on fp32 operands. A block alone on a compute unit takes 2.2 us a step of 32 rows, two together 2.6, so that the
// jobs of a launch are cut, all into slices of as many rows, to fill TN_SLOTS places once: with 256 rows a slice some units had two blocks
// and others one (sums over 90 K rows, 2 x 256 x 256, 320 blocks: 182 us; 504: 151; 13 K rows, 320: 38.6, 472: 32.0; 10 K rows, 2 x 602 x 256,
// 400: 54.8; 500: 48.9; 25 K rows, 2 x 100 x 256, 256: 35.9; 448: 31.9). Blocks in small tiles and on bf16 operands are short: four of them count as one.
// (A function of the row counts and shapes alone, so the order of the sums is the same in every run.)
__device__ __forceinline__ int tn_rows(const GemmTNArgs& g) { return min(*g.d_R, g.R_cap); }
__device__ __forceinline__ int tn_plain_slices(const GemmTNArgs& g, int R) { return tn_used_splits(R, g.plain_splits, g.rows_per_split, g.few_splits); }
__device__ __forceinline__ int tn_plan(const CutTNLaunch& launch, int job, int R, bool* large) {
    const GemmTNArgs& g = launch.job[job];
    const int plain = tn_plain_slices(g, R);
    *large = !tn_narrow(g) && tn_tiles(g, 128) * plain >= TN_LARGE_BLOCKS;
    if (!*large || g.A16) return plain;
    int others = 0, tiles = 0;
    float work = 0.f;
    for (int j = 0; j < launch.n; ++j) {
        const GemmTNArgs& o = launch.job[j];
        const int rows = tn_rows(o), s = tn_plain_slices(o, rows), t = (int)tn_tiles(o, 128);
        const bool lg = !tn_narrow(o) && t * s >= (int)TN_LARGE_BLOCKS;
        if (lg && !o.A16) {
            tiles += t;
            work += (float)t * (float)rows;
        } else {
            others += (lg ? t : (int)tn_tiles(o, 64)) * s;
        }
    }
    const int room = max(TN_SLOTS - others / 4, TN_SLOTS / 2);
    if (2 * tiles > room) return plain;
    // (a job's last slices, one a tile, may be short ones: room for them)
    const int rows = max(((int)(work / (float)(room - tiles)) + SK) / SK * SK, TN_LEAST_ROWS);
    return max(min((R + rows - 1) / rows, g.splits), plain);
}

// All jobs in small tiles, four blocks on a compute unit (31 KB of LDS, 118 registers) in place of two: they hide each other's waits, and fewer slices
// leave less to reduce. Faster as long as the whole launch is short (us, large and small tiles in one kernel / this: 1 K rows, 2 x 256 x 47
// 7.8 / 5.6; 3.4 K rows, 2 x 256 x 256 14.1 / 12.2; 5 K rows 20.3 / 15.2; 13 K rows 32.2 / 30.6; 25 K rows, 2 x 100 x 256 31.9 / 30.6; 10 K rows, 2 x 602 x 256
// 46.7 / 53.4; 40 K rows, 2 x 256 x 256 68.1 / 78.3). Not in steps, where more of the chip is left to the next batch's sampling by fewer blocks
// (dense GCN-style 151 / 157, sparse 313 / 314).
__global__ void __launch_bounds__(256, 4) cut_tn_small_kernel(CutTNLaunch launch) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[tn_shared_bytes(64)];
    int job = 0;
    uint32_t first = 0;
    while (job + 1 < launch.n && blockIdx.x >= launch.end_block[job]) first = launch.end_block[job++];
    const GemmTNArgs& g = launch.job[job];
    const int R = tn_rows(g), used = tn_plain_slices(g, R);
    const uint32_t id = blockIdx.x - first;
    if (id == 0 && threadIdx.x == 0) *tn_used_word(g.P, g.splits, g.Kp, g.N) = used;      // (the reduction reads the first `used` partials only)
    cut_tn_tile<64, false>(g, id, R, used, smem);
}
// What a layer call's launch has to do, about, in steps of 32 rows of a large tile, and up to where small tiles win.
constexpr int64_t TN_SMALL_WORK = 3500, TN_SMALL_WORK_WITH_INPUT_GRADIENT = 5000;
static int64_t tn_work(const GemmTNArgs& t) { return (int64_t)tn_tiles(t, 128) * t.small_up_to / SK; }

__global__ void __launch_bounds__(256, 2) cut_tn_kernel(CutTNLaunch launch) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[tn_shared_bytes(128)];
    int job = 0;
    uint32_t first = 0;
    while (job + 1 < launch.n && blockIdx.x >= launch.end_block[job]) first = launch.end_block[job++];
    const GemmTNArgs& g = launch.job[job];
    const int R = tn_rows(g);
    bool large;
    const int used = tn_plan(launch, job, R, &large);
    const uint32_t id = blockIdx.x - first;
    if (id == 0 && threadIdx.x == 0) *tn_used_word(g.P, g.splits, g.Kp, g.N) = used;      // (the reduction reads the first `used` partials only)
    if (g.A16) {
        if (large) cut_tn_tile<128, true>(g, id, R, used, smem);
        else cut_tn_tile<64, true>(g, id, R, used, smem);
    } else {
        if (large) cut_tn_tile<128, false>(g, id, R, used, smem);
        else cut_tn_tile<64, false>(g, id, R, used, smem);
    }
}

// Input gradient and weight gradients of a layer call in one launch (nn_blocks: a multiple of the dies): neither waits for the other, and a layer
// of some thousand rows fills the chip with neither. In small tiles: beside blocks of large ones, which leave room for two on a compute unit, the
// input gradient takes longer than before them (3.4 K rows, 256 x 256: 30 us -> 26 in small tiles, 24 with room for large ones; steps of 25 K rows 311 ->
// 321 us). Forward and backward pass of a layer, us, in two launches / in one: 3.4 K rows, 256 x 256 70.7 / 65.2; 5.2 K 96.2 / 80.3; 10 K 129 / 119; 20 K 211 /
// 205; 4 K rows, 602 x 64 104 / 88; 12 K 223 / 204; 8 K rows, 602 x 256 213 / 211; 30 K rows, 100 x 256 180 / 170.
template <int MI, int NJ, int WN>
__global__ void __launch_bounds__(256, 3) cut_grads_kernel(GemmNNArgs g, uint32_t nn_blocks, GemmTNArgs t) {
    constexpr int NN = NNTile<MI, NJ, WN>::BYTES, TN = tn_shared_bytes(64);
    __shared__ __attribute__((aligned(16))) unsigned char smem[NN > TN ? NN : TN];
    __shared__ float scale_sh[NNTile<MI, NJ, WN>::BM];
    if (blockIdx.x < nn_blocks) {
        cut_nn_tile<MI, NJ, WN>(g, smem, scale_sh);
        return;
    }
    const int R = tn_rows(t), used = tn_plain_slices(t, R);
    const uint32_t id = blockIdx.x - nn_blocks;
    if (id == 0 && threadIdx.x == 0) *tn_used_word(t.P, t.splits, t.Kp, t.N) = used;
    cut_tn_tile<64, false>(t, id, R, used, smem);
}
int32_t gemm_tn_partials(const GemmTNArgs* jobs, int32_t n_jobs, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
    CutTNLaunch launch{};
    uint64_t blocks = 0;
    int64_t work = 0;
    bool all_small = true;
    for (int32_t j = 0; j < n_jobs; ++j)
        if (jobs[j].Kp > 0 && jobs[j].N > 0) {
            work += tn_work(jobs[j]);
            all_small = all_small && !jobs[j].A16 && jobs[j].small_up_to > 0;
        }
    all_small = all_small && work <= TN_SMALL_WORK;
    for (int32_t j = 0; j < n_jobs && launch.n < NO_MAX_LAYERS; ++j) {
        const GemmTNArgs& a = jobs[j];
        if (a.Kp <= 0 || a.N <= 0) continue;
        // (small tiles are only taken while there are few large ones, or by a narrow job)
        const uint64_t small = (uint64_t)tn_tiles(a, 64), large = (uint64_t)tn_tiles(a, 128);
        const uint64_t most_small = all_small || tn_narrow(a) ? (uint64_t)a.splits : std::min<uint64_t>((uint64_t)a.splits, (TN_LARGE_BLOCKS - 1) / tn_tiles(a, 128));
        blocks += (uint64_t)ceil_div((int64_t)std::max(small * most_small, all_small ? 0 : large * (uint64_t)a.splits), N_XCD) * N_XCD;
        NO_REQUIRE(blocks < (1ull << 31), NO_ERR_CAPACITY, "gemm_tn: too many blocks");
        launch.job[launch.n] = a;
        launch.end_block[launch.n] = (uint32_t)blocks;
        ++launch.n;
    }
    if (launch.n == 0) return NO_OK;
    if (all_small) NO_LAUNCH_TIMED(cut_tn_small_kernel, dim3((unsigned)blocks), dim3(256), st, ev0, ev1, launch);
    else NO_LAUNCH_TIMED(cut_tn_kernel, dim3((unsigned)blocks), dim3(256), st, ev0, ev1, launch);
    return launch_status("gemm_tn");
}

template <int MI, int NJ, int WN>
static int32_t launch_cut_nn(const GemmNNArgs& a, const GemmTNArgs* job, bool* job_done, hipStream_t st) {
    const unsigned blocks = xcd_padded(ceil_div(a.N, NNTile<MI, NJ, WN>::BN) * ceil_div(a.M_cap, NNTile<MI, NJ, WN>::BM) * a.n_problems);
    if constexpr (WN > 1) {
        if (job && tn_work(*job) <= TN_SMALL_WORK_WITH_INPUT_GRADIENT) {
            const unsigned tn_blocks = xcd_padded((int64_t)tn_tiles(*job, 64) * tn_used_splits(job->R_cap, job->splits, job->rows_per_split, job->few_splits));
            hipLaunchKernelGGL((cut_grads_kernel<MI, NJ, WN>), dim3(blocks + tn_blocks), dim3(256), 0, st, a, blocks, *job);
            *job_done = true;
            return launch_status("cut_grads");
        }
    }
    hipLaunchKernelGGL((cut_nn_kernel<MI, NJ, WN>), dim3(blocks), dim3(256), 0, st, a);
    return launch_status("cut_nn");
}

int32_t cut_nn(const GemmNNArgs& a, const GemmTNArgs* job, bool* job_done, hipStream_t st) {
    // Few rows: 32-row blocks (twice as many; measured at 3.4 K / 5.5 K rows x 256 columns: 12.9 / 15.8 us against 15.2 / 18.9 with 64-row
    // blocks, at 25 K rows 37 against 31), by the capacity, which the host knows when it launches: a batch that fills a small part of a larger
    // one pays for it (backward pass of a layer in a capacity of 19 K / 21 K rows, us: 3.4 K rows, 100 x 256 39.1 / 41.5, 256 x 256 50.6 / 50.3;
    // 5.5 K rows 48.0 / 49.2, 67.6 / 68.8; 12 K rows 68.3 / 70.3, 99.6 / 98.6). Narrow outputs: all four wavefronts below each other.
    if (a.N <= 64) return launch_cut_nn<1, 2, 1>(a, job, job_done, st);
    if (a.M_cap <= 20000) return launch_cut_nn<1, 1, 4>(a, job, job_done, st);
    return launch_cut_nn<2, 1, 4>(a, job, job_done, st);
}

}  // namespace no
