// The forward products of Eq. 2 on the bf16 matrix cores: every fp32 operand in three bf16 pieces, six partial products of a pair
// (gemm_cut.hip says why that is no less exact than the fp32 instruction). C = sum over the phases p of A_p B_p, + bias, ReLU; the rows of A_p
// may be picked out of a table, the rows of C scattered (GemmNNArgs).
//
// A block owns a BM x BN tile of C, 2 x 2 wavefronts. Rows of A are requested two steps of 32 reduction indices ahead and cut, once a block,
// into one of two LDS copies while the other is multiplied (one barrier a step); fragments of B come straight from the planes that
// cut_weights made of the weights in this step or call (a lane's eight indices are 16 contiguous bytes, the 32 lanes of a fragment 512: L1 and L2
// reads, half a step ahead). LDS delivers 64 bytes a cycle here, a third of a fragment's products in matrix cycles: with both operands in LDS it
// was the bound (90 K rows, 2 x 256 x 256, 64 x 128 tiles: 174 us; like this 161).
// Bound: 416 TFLOP/s of fp32 products by the matrix rate, 234 by what a large bf16 product reaches here. Measured, fp32 instruction -> this, the
// launch alone: 90 K rows, 2 x 256 x 256: 231 -> 161 us (147 TFLOP/s); 13 K rows 47.5 -> 31; 11 K rows, 2 x 602 x 256: 80 -> 62; 25 K rows,
// 2 x 100 x 256: 45.5 -> 35. Relative 2-norm error against fp64: 2.1e-7 -> 0.94e-7, 3.8e-7 -> 1.7e-7 (602 columns),
// 1.1e-7 -> 0.52e-7 (100).
#include <algorithm>

#include "gemm_tile.hpp"

namespace no {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

constexpr int FK = 32, FPITCH = FK + 8;      // reduction indices a step; bf16 elements an LDS row (rows start 20 banks apart)

__device__ __forceinline__ bf16x8_t fwd_fragment(const uint16_t* p) {
    bf16x8_t v;
    __builtin_memcpy(&v, __builtin_assume_aligned(p, 16), 16);
    return v;
}

constexpr int FWD_THREADS = 256;
constexpr int fwd_shared_bytes(int BM, int BN) { return 6 * BM * FPITCH * 2 > BM * (BN + 4) * 4 ? 6 * BM * FPITCH * 2 : BM * (BN + 4) * 4; }

template <int BM, int BN>
__device__ __forceinline__ void cut_fwd_tile(const GemmNNArgs& g, int M, int bx, int by, unsigned char* smem, int32_t* crow_sh, int32_t* krow_sh) {
    constexpr int I = BM / 64, J = BN / 64, PLANE = BM * FPITCH, COPY = 3 * PLANE;
    uint16_t* As = reinterpret_cast<uint16_t*>(smem);
    const int m0 = by * BM, n0 = bx * BN, N = g.N, tid = (int)threadIdx.x;
    const int wave = tid >> 6, wm = wave >> 1, wn = wave & 1, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    for (int r = (int)threadIdx.x; r < BM; r += FWD_THREADS) {
        const int row = min(m0 + r, M - 1);
        crow_sh[r] = g.c_rows ? g.c_rows[row] : row;
        krow_sh[r] = g.c_keep_rows ? g.c_keep_rows[row] : -1;
    }
    floatx16 acc[2][I][J];
#pragma unroll
    for (int i = 0; i < I; ++i)
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[0][i][j][r] = acc[1][i][j][r] = 0.f;
    const int phases = g.n_problems, K0 = g.K[0], K1 = phases > 1 ? g.K[1] : 0;
    const int steps0 = (K0 + FK - 1) / FK, steps = steps0 + (K1 + FK - 1) / FK;
    // this thread's rows of A, and its columns of B (those past the operand repeat the last one and are never stored)
    const int kq = (tid & 3) * 8;
    const float* arow[2][I];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int i = 0; i < I; ++i) {
            const int q = p < phases ? p : 0, row = min(m0 + 64 * i + (tid >> 2), M - 1);
            arow[p][i] = g.A[q] + (int64_t)(g.a_rows[q] ? g.a_rows[q][row] : row) * g.lda[q];
        }
    uint32_t boff[J];
#pragma unroll
    for (int j = 0; j < J; ++j) boff[j] = (uint32_t)(half * N + min(n0 + wn * (BN / 2) + j * 32 + l32, N - 1)) * 16u;
    const char* const b0 = reinterpret_cast<const char*>(g.cut_B[0]);
    const char* const b1 = reinterpret_cast<const char*>(phases > 1 ? g.cut_B[1] : g.cut_B[0]);
    auto request_a = [&](RowUnit (&t)[I], int s) {        // (past the last step: that one again, not used)
        s = min(s, steps - 1);
        const bool second = s >= steps0;
        const int K = second ? K1 : K0, k = (second ? s - steps0 : s) * FK + kq;
#pragma unroll
        for (int i = 0; i < I; ++i) t[i].request(second ? arow[1][i] : arow[0][i], k, K);
    };
    auto store_a = [&](RowUnit (&t)[I], int s, uint16_t* S) {
        const bool second = s >= steps0;
        const int K = second ? K1 : K0, k = (second ? s - steps0 : s) * FK + kq;
        if (k - kq + FK > K) {
#pragma unroll
            for (int i = 0; i < I; ++i) t[i].trim(k, K);
        }
#pragma unroll
        for (int i = 0; i < I; ++i) {
            uint4 p[3];
            cut8(t[i].f, p);
            uint16_t* at = S + (64 * i + (tid >> 2)) * FPITCH + kq;
#pragma unroll
            for (int e = 0; e < 3; ++e) *reinterpret_cast<uint4*>(at + e * PLANE) = p[e];
        }
    };
    // (the planes hold zeros from a phase's last index on)
    auto request_b = [&](bf16x8_t (&b)[J][3], int s, int ks) {
        s = min(s, steps - 1);
        const bool second = s >= steps0;
        const int64_t plane = (int64_t)cut_pad(second ? K1 : K0) * N * 2;
        const char* base = (second ? b1 : b0) + (int64_t)((second ? s - steps0 : s) * 2 + ks) * N * 32;
#pragma unroll
        for (int p = 0; p < 3; ++p, base += plane)
#pragma unroll
            for (int j = 0; j < J; ++j) b[j][p] = fwd_fragment(reinterpret_cast<const uint16_t*>(base + boff[j]));
    };
    auto multiply = [&](const uint16_t* S, const bf16x8_t (&b)[J][3], int ks) {
        bf16x8_t a[I][3];
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int i = 0; i < I; ++i) a[i][p] = fwd_fragment(S + p * PLANE + (wm * (BM / 2) + i * 32 + l32) * FPITCH + ks * 16 + half * 8);
#pragma unroll
        for (int t = 0; t < CUT_TERMS; ++t)
#pragma unroll
            for (int i = 0; i < I; ++i)
#pragma unroll
                for (int j = 0; j < J; ++j)
                    acc[CUT_TERM[t].acc][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][CUT_TERM[t].a], b[j][CUT_TERM[t].b],
                                                                                          acc[CUT_TERM[t].acc][i][j], 0, 0, 0);
    };
    RowUnit ta[2][I];
    bf16x8_t first[J][3], last[J][3];
    request_a(ta[0], 0);
    request_a(ta[1], 1);
    request_b(first, 0, 0);
    store_a(ta[0], 0, As);
    request_a(ta[0], 2);
    __syncthreads();
    auto step = [&](int s, const uint16_t* cur, uint16_t* nxt, RowUnit (&t)[I]) {
        request_b(last, s, 1);
        multiply(cur, first, 0);
        request_b(first, s + 1, 0);
        if (s + 1 < steps) store_a(t, s + 1, nxt);
        request_a(t, s + 3);
        multiply(cur, last, 1);
        __syncthreads();
    };
    for (int s = 0; s < steps; s += 2) {
        step(s, As, As + COPY, ta[1]);
        if (s + 1 < steps) step(s + 1, As + COPY, As, ta[0]);
    }
    // the output tile through LDS: 16-byte stores along rows
    constexpr int CPITCH = BN + 4, C4 = BN / 4;
    float* Cs = reinterpret_cast<float*>(smem);
    float bad = 0.f;
#pragma unroll
    for (int i = 0; i < I; ++i)
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float v = (acc[1][i][j][r] + acc[0][i][j][r]) * CUT_UNSCALE;
                bad = fmaf(v, 0.f, bad);      // (0 while every sum is finite, NaN from then on)
                Cs[(wm * (BM / 2) + i * 32 + acc_row(r, lane)) * CPITCH + wn * (BN / 2) + j * 32 + l32] = v;
            }
    // Some sum of this wavefront is not finite: its products once more on the fp32 instruction, from memory (as in gemm_cut.hip; a lane
    // brings four consecutive indices of a row of A and of a column of B, lanes 0-31 the first four of eight).
    if (__any(bad != 0.f)) {
        const float *pa[2][I], *pb[2][J];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int e = p < phases ? p : 0;
#pragma unroll
            for (int i = 0; i < I; ++i) {
                const int row = min(m0 + wm * (BM / 2) + i * 32 + l32, M - 1);
                pa[p][i] = g.A[e] + (int64_t)(g.a_rows[e] ? g.a_rows[e][row] : row) * g.lda[e];
            }
#pragma unroll
            for (int j = 0; j < J; ++j) {
                pb[p][j] = g.B[e] + min(n0 + wn * (BN / 2) + j * 32 + l32, N - 1);
            }
        }
#pragma unroll
        for (int i = 0; i < I; ++i)
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[0][i][j][r] = 0.f;
        for (int p = 0; p < phases; ++p) {
            const int K = p ? K1 : K0;
            const int64_t ldb = g.ldb[p];
            for (int k = half * 4; k - half * 4 < K; k += 8) {
                float a[I][4], b[J][4];
#pragma unroll
                for (int i = 0; i < I; ++i) {
                    const float4 v = load4_guarded((p ? pa[1][i] : pa[0][i]) + k, K - k);
                    a[i][0] = v.x; a[i][1] = v.y; a[i][2] = v.z; a[i][3] = v.w;
                }
#pragma unroll
                for (int j = 0; j < J; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) b[j][e] = k + e < K ? (p ? pb[1][j] : pb[0][j])[(int64_t)(k + e) * ldb] : 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int i = 0; i < I; ++i)
#pragma unroll
                        for (int j = 0; j < J; ++j) acc[0][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], b[j][e], acc[0][i][j], 0, 0, 0);
            }
        }
#pragma unroll
        for (int i = 0; i < I; ++i)
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    float* c = &Cs[(wm * (BM / 2) + i * 32 + acc_row(r, lane)) * CPITCH + wn * (BN / 2) + j * 32 + l32];
                    if (!(fabsf(*c) < INFINITY)) *c = acc[0][i][j][r];
                }
    }
    __syncthreads();
    const int c4 = (int)threadIdx.x % C4 * 4, n = n0 + c4;
    if (n >= N) return;
    float* C = g.C[0];
    const int64_t ldc = g.ldc[0];
    const bool vec = (ldc % 4 == 0) && ((reinterpret_cast<uintptr_t>(C) & 15) == 0) &&
                     (!g.c_keep_rows || (reinterpret_cast<uintptr_t>(g.c_keep) & 15) == 0) && n + 4 <= N;
    float bias[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) bias[e] = g.bias ? g.bias[min(n + e, N - 1)] : 0.f;
#pragma unroll 4
    for (int lr = (int)threadIdx.x / C4; lr < BM; lr += FWD_THREADS / C4) {
        if (m0 + lr >= M) break;
        const float4 t = *reinterpret_cast<const float4*>(&Cs[lr * CPITCH + c4]);
        float v[4] = {t.x + bias[0], t.y + bias[1], t.z + bias[2], t.w + bias[3]};
        if (g.relu) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
        }
        const int kr = krow_sh[lr];
        if (g.positive) g.positive[(int64_t)crow_sh[lr] * (N / 4) + n / 4] = positive_of(v[0], v[1], v[2], v[3]);
        float* dst = C + (int64_t)crow_sh[lr] * ldc + n;
        float* keep = kr >= 0 ? g.c_keep + (int64_t)kr * ldc + n : nullptr;
        if (vec) {
            *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
            if (keep) *reinterpret_cast<float4*>(keep) = make_float4(v[0], v[1], v[2], v[3]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n + e < N) {
                    dst[e] = v[e];
                    if (keep) keep[e] = v[e];
                }
        }
        if (keep && n == 0 && g.c_keep_stamp) g.c_keep_stamp[kr] = g.stamp;
    }
}

// The larger tiles (LARGE) or the smaller: by what the compute unit with the most of them takes, per step, in hundredths of a microsecond (one tile
// alone / each of several: 64 x 64 71 / 55, 64 x 128 98 / 88). Whole launches, us, 64 x 64 / 64 x 128: 3.4 K rows, 2 x 256 x 256
// 15.8 / 19.9; 13 K rows 38.6 / 31.1; 90 K rows 208 / 161; 11 K rows, 2 x 602 x 256 67 / 62; 25 K rows, 2 x 100 x 256 40 / 35.
// (128 x 128: 148 at 90 K rows, 32 at 25 K; but two of its blocks take every register of a compute unit, and nothing of the next batch's
// sampling runs beside them: steps on the dense graph 221 us, 208 with these.)
template <int BM, int BN>
__host__ __device__ inline int64_t fwd_tiles(int64_t M, int64_t N) { return ((M + BM - 1) / BM) * ((N + BN - 1) / BN); }
__device__ __forceinline__ int64_t fwd_cost(int64_t tiles, int alone, int each) { return tiles <= 256 ? alone : (tiles + 255) / 256 * each; }

// Three workgroups a compute unit, which take their tiles in turn: consecutive tiles (those of the same rows of A among them) stay on one die, and
// no block of a grid for the row capacity waits for a place only to find that it has no tile.
constexpr int FWD_BLOCKS = 768;
__global__ void __launch_bounds__(FWD_THREADS, 3) cut_fwd_kernel(GemmNNArgs g) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[fwd_shared_bytes(64, 128)];
    __shared__ int32_t crow_sh[64], krow_sh[64];
    int M = *g.d_M;
    if (M > g.M_cap) M = g.M_cap;
    if (M <= 0) return;
    const int64_t small = fwd_tiles<64, 64>(M, g.N), large = fwd_tiles<64, 128>(M, g.N);
    const bool use_large = fwd_cost(large, 98, 88) < fwd_cost(small, 71, 55);
    const int64_t total = use_large ? large : small, per_die = (total + N_XCD - 1) / N_XCD, die = blockIdx.x % N_XCD;
    const int BN = use_large ? 128 : 64, gx = (g.N + BN - 1) / BN;
    for (int64_t t = blockIdx.x / N_XCD; t < per_die && die * per_die + t < total; t += gridDim.x / N_XCD) {
        const int64_t lid = die * per_die + t;
        const int bx = (int)(lid % gx), by = (int)(lid / gx);
        __syncthreads();      // (the tile before is stored)
        if (use_large) cut_fwd_tile<64, 128>(g, M, bx, by, smem, crow_sh, krow_sh);
        else cut_fwd_tile<64, 64>(g, M, bx, by, smem, crow_sh, krow_sh);
    }
}

int32_t cut_fwd(const GemmNNArgs& a, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
    const int64_t blocks = std::min<int64_t>(FWD_BLOCKS, ceil_div(fwd_tiles<64, 64>(a.M_cap, a.N), N_XCD) * N_XCD);
    NO_LAUNCH_TIMED(cut_fwd_kernel, dim3((unsigned)blocks), dim3(FWD_THREADS), st, ev0, ev1, a);
    return launch_status("cut_fwd");
}

}  // namespace no
