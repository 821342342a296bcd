// fp32 matrix products for the dense UPDATE of Eq. 2 and its gradients, on the gfx950 matrix
// cores (gemm_cut.hip: gradients; gemm.hip: forward products and small gradients). Two shapes:
//   NN: C[M,N] = sum_p A_p[M,K_p] * B_p[K_p,N] (+ bias, ReLU, optional 1/len row scale); M is a
//       device scalar (rows past it are skipped); B may be given transposed; the rows of A_p may be
//       picked out of a larger table by an index (gather fused into the operand load).
//   TN: P[s][K',N] = A[rows of split s]^T * G[rows of split s]; the reduction length is a device
//       scalar; splits are summed in a fixed order afterwards (no float atomics).
#pragma once
#include "common.hpp"

namespace no {

struct GemmNNArgs {
    const float* A[2]; int64_t lda[2];
    const int32_t* a_rows[2];             // per problem: row m of the operand is row a_rows[m] of A (NULL: row m)
    const float* B[2]; int64_t ldb[2];
    int32_t K[2];
    // large products take the B operands as bf16 planes (cut_weights): made by the caller, or, for an input gradient, here in cut_scratch
    const uint16_t* cut_B[2];
    void* cut_scratch; size_t cut_scratch_bytes;
    float* C[2]; int64_t ldc[2];
    const int32_t* row_scale_indptr[2];   // per problem: multiply row m by 1/(indptr[m+1]-indptr[m]+row_scale_plus) (0 if that is 0)
    int32_t row_scale_plus;               // 1 when the row itself counts in the average (Eq. 1 over N_in(v) U {v})
    int32_t row_scale_rsqrt;              // 1: the factor is that count to the power -1/2 (symmetric normalisation)
    int32_t n_problems;                   // 1 or 2
    int32_t accumulate;                   // 1: both products are summed into C[0]; 0: independent problems (grid.z)
    const int32_t* d_M; int32_t M_cap; int32_t N;
    const float* bias; int32_t relu;
    // Scattered output of C[0] (layer 1 with reuse, Section 4.1.2): row m goes to row c_rows[m] (NULL: m); a row with
    // c_keep_rows[m] >= 0 is also stored as row c_keep_rows[m] of c_keep (same leading dimension) and
    // c_keep_stamp[that row] = stamp: the cache refresh of a recomputed hot vertex.
    const int32_t* c_rows;
    float* c_keep; const int32_t* c_keep_rows; int32_t* c_keep_stamp; int32_t stamp;
    // which outputs of C[0] are positive, a byte for every four columns of a row (N a multiple of 4), at the output's row; NULL: not asked for
    uint8_t* positive;
};

struct GemmTNArgs {
    const float* A[2]; int64_t lda[2];                    // [R, Kp] row-major; two problems share G
    const float* G; int64_t ldg;                         // [R, N]
    float* P;                                            // partials [2][splits][Kp+1][N]; row Kp of product 0 = column sums of G
    int32_t Kp, N;
    const int32_t* d_R; int32_t R_cap; int32_t splits;   // splits: the most row slices (the partials' layout is sized for it)
    int32_t plain_splits = 0;                            // the most slices of rows_per_split rows (splits: of any)
    int32_t small_up_to = 0;                             // > 0: R is about this, and small tiles may be taken for short launches
    int32_t n_problems = 2;                              // 1: only A[0]
    const uint16_t* A16 = nullptr;                       // products with bf16 operands: the first one's rows in place of A[0]
    int32_t rows_per_split = 0;                          // > 0: only ceil(R / rows_per_split) slices are used when that is fewer (large tiles: tn_plan) ...
    int32_t few_splits = 0;                              // ... though these many, if they keep TN_FEWEST_ROWS rows each
};

constexpr int32_t TN_FEWEST_ROWS = 64;
// Places of a chip for blocks of large tiles, two a compute unit, and the fewest rows of a slice that is cut to fill them (tn_plan).
constexpr int TN_SLOTS = 512, TN_LEAST_ROWS = 128;

// The number of row slices a split product over R rows really uses: the capacity-sized bound `splits`, cut down so that a
// slice keeps about rows_per_split rows, but few_splits of them where those keep TN_FEWEST_ROWS each (a function of R and the shape alone, so
// the summation order is the same in every run).
__host__ __device__ inline int32_t tn_used_splits(int32_t R, int32_t splits, int32_t rows_per_split, int32_t few_splits) {
    if (rows_per_split <= 0) return splits;
    int32_t s = (R + rows_per_split - 1) / rows_per_split;
    int32_t fill = (R + TN_FEWEST_ROWS - 1) / TN_FEWEST_ROWS;
    if (fill > few_splits) fill = few_splits;
    if (s < fill) s = fill;
    if (s < 1) s = 1;
    return s < splits ? s : splits;
}

// Where the product leaves the number of slices it used for the reduction: in the place of the column sums that product 1 does not have.
__host__ __device__ inline int32_t* tn_used_word(float* P, int32_t splits, int32_t Kp, int32_t N) {
    return reinterpret_cast<int32_t*>(P + ((int64_t)splits * (Kp + 1) + Kp) * N);
}

// Products with bf16 operands (a layer fed by a bf16 feature table): see gemm_bf16.hip.
struct GemmBf16NNArgs {
    const uint16_t* X; int64_t ldx; const int32_t* x_rows;   // first operand: bf16 rows; row m is row x_rows[m] of X (NULL: m)
    const float* Mn; int64_t ldm;                            // second operand: fp32 rows, rounded to bf16 on load
    const uint16_t* Wt[2]; int32_t Kpad;                     // the two weight matrices as bf16 [N][Kpad] (weights_to_bf16_t)
    int32_t K, N;
    float* C; int64_t ldc;
    const int32_t* d_M; int32_t M_cap;
    const float* bias; int32_t relu;
    const int32_t* c_rows; float* c_keep; const int32_t* c_keep_rows; uint8_t* positive;   // as in GemmNNArgs
};
// Weights cut for the large gradient products (gemm_cut.hip): planes of the transpose of one matrix [K][N], the reduction index (over
// the N columns) padded to 32.
__host__ __device__ inline int32_t cut_pad(int32_t N) { return (N + 31) / 32 * 32; }
__host__ __device__ inline size_t cut_weights_elements(int32_t K, int32_t N, bool forward = false) {
    return forward ? (size_t)3 * cut_pad(K) * N : (size_t)3 * cut_pad(N) * K;
}
// w1 may be NULL; the second matrix's planes follow the first's (cut_weights_elements apart). forward: planes of the matrix itself, for a
// forward product (gemm_fwd.hip), the reduction over its K rows.
int32_t cut_weights(const float* w0, const float* w1, int32_t K, int32_t N, bool forward, uint16_t* out, hipStream_t st);
// Whether an input gradient of M_cap x N (reduction over K columns) reads planes: more output tiles than compute units for the
// kernel for small products to keep busy by splitting the reduction.
inline bool input_grad_takes_planes(int32_t M_cap, int32_t K, int32_t N, int32_t n_problems) {
    return ceil_div(M_cap, 64) * ceil_div(N, 64) * n_problems > 128 && K >= 8;
}
// Whether a forward product of about `rows` rows in a step or a bulk refresh does. The line lies where a launch of its own for the weights paid, as that of
// layer 1 in a batch prepared ahead still has; the others' weights go with the aggregation now and would pay earlier (layer_takes_planes). It stays
// there because a product's last bits turn ReLU decisions that are zero to within rounding: the step of the sparse graph, batch 1024, takes 307 us
// with both hidden layers on planes and 317 without, but after 12 steps its parameters are off by 0.8 % from those it had. Measured, two
// products / one, with a launch for the weights, us on the fp32 instruction / on planes: 256 columns, 9 K rows, K = 128 65.2 / 66.9; 20 K rows, K = 64 74.5 / 75.1, 100
// 89.8 / 88.2; 90 K rows, K = 47 266 / 248; one product, 12 K rows, K = 256 32 / 37, 602 60.3 / 59.9; 20 K rows, K = 100 30.3 / 31.2, 256 44.9 / 43.3; 90 K rows, 172 columns,
// K = 32 41 / 47, 200 117 / 109.
inline bool forward_takes_planes(int64_t rows, int32_t K, int32_t N, int32_t n_problems) {
    const int64_t tiles = ceil_div(rows, 64) * ceil_div(N, 64);
    if (K < 8 || N == 64 || tiles < 512 || tiles * (K + 50) < 150000) return false;
    const bool half_empty = N % 128 > 0 && N % 128 <= 64;      // (the last column tile, of 128)
    return n_problems > 1 || (tiles * (K + 150) >= 325000 && (K >= 128 || !half_empty));
}
// Whether the forward product of a layer call does. Its weights are cut by extra blocks of the aggregation in front of it. Measured, aggregation
// and product, two products / one, time on planes over that on the fp32 instruction: 256 columns, 3.4 K rows, K = 256 1.10 / 1.15, 602 1.02 / 1.07; 5 K rows,
// 100 1.02 / 1.05, 256 0.91 / 1.02, 602 0.82 / 0.89; 9 K rows, 64 1.05 / 1.18, 100 1.00 / 1.09, 256 0.90 / 1.01; 13 K rows, 32 0.95 / 1.03, 64 0.89 / 0.95, 100 0.83 /
// 0.87, 256 0.77 / 0.85; 20 K rows, 32 1.00 / 1.04, 64 0.94 / 0.99, 100 0.92 / 0.93; 40 K rows, 16 0.81 / 0.91. 128 columns, 5 K rows, 602 1.00 / 1.05; 9 K rows, 100 1.03 /
// 1.04, 256 0.91 / 1.02, 602 0.82 / 0.90; 20 K rows, 100 1.03 / 1.13, 256 0.91 / 1.00; 40 K rows, 100 0.94 / 0.97. 64 columns are one whole tile, for which rows are cut
// as often as for 128: 13 K rows, 602 1.02 / 1.04, 20 K rows, 100 1.08 / 1.10, 256 0.95 / 1.05, 602 0.89 / 0.96. Columns that are no multiple of 64 the fp32
// instruction reads one by one: 172 columns, K = 256, 3.4 K rows 0.80 / 0.97, 7 K 0.78 / 0.91; 100 columns, 5 K rows 0.81 / 0.97, 9 K 0.79 / 0.92; 47 columns, 9 K rows
// 0.88 / 1.01, 40 K 0.84 / 0.96, K = 100 0.96 / 1.08 and 0.94 / 1.08; 100 columns, K = 32, 20 K rows 1.20 / 1.34, 40 K 0.99 / 1.06, 90 K 0.89 / 0.95;
// one product, 90 K rows, 200 columns, K = 8 0.86, 172, K = 32 1.15.
inline bool layer_takes_planes(int64_t rows, int32_t K, int32_t N, int32_t n_problems) {
    const int64_t tiles = ceil_div(rows, 64) * ceil_div(N, 64);
    const bool whole = N % 64 == 0, wide = N > 64, half_empty = N % 128 > 0 && N % 128 <= 64;      // (the last column tile, of 128)
    if (K < 8) return false;
    if (n_problems > 1)
        return (K >= 200 && tiles >= (whole ? 300 : 140)) || (K >= 64 && tiles >= (N > 128 ? 700 : 1200) && wide) || (tiles >= (K >= 16 ? 2000 : 2600) && N != 64);
    return wide && (K >= 128 || !half_empty) && ((K >= (whole ? 400 : 200) && tiles >= 300) || (K >= 64 && tiles >= (N > 128 ? 800 : 1200)) || tiles >= 2400);
}
// Matrices cut by extra blocks of another launch of blocks of 256 threads: matrix j, [K][N], takes the
// blocks [end_block[j-1], end_block[j]) of them.
struct CutJobs {
    static constexpr int MOST = 2 * NO_MAX_LAYERS;
    const float* w[MOST]; uint16_t* out[MOST]; int32_t K[MOST], N[MOST];
    uint32_t end_block[MOST]; int32_t n = 0; uint32_t forward = 0;      // (bit j: matrix j in the forward layout)
    void add(const float* matrix, int32_t rows, int32_t cols, uint16_t* planes, bool fwd = false) {
        w[n] = matrix; out[n] = planes; K[n] = rows; N[n] = cols;
        forward |= fwd ? 1u << n : 0u;
        end_block[n] = blocks() + (uint32_t)ceil_div((int64_t)cut_weights_elements(rows, cols, fwd) / 24, 256);
        ++n;
    }
    uint32_t blocks() const { return n ? end_block[n - 1] : 0u; }
};
int32_t cut_all(const CutJobs& cut, hipStream_t st, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);      // in a launch of their own
inline int32_t bf16_kpad(int32_t K) { return (K + 15) / 16 * 16; }
int32_t weights_to_bf16_t(const float* w, int32_t K, int32_t N, int32_t Kpad, uint16_t* out, hipStream_t st);
int32_t gemm_bf16_nn(const GemmBf16NNArgs& a, hipStream_t st, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);

// Statistics of a training step, written by one extra block of the last gradient reduction of the step (they are
// nobody's input, so they do not get a launch of their own on the step's dependency chain): mean of the per-seed
// losses in a fixed order and the block sizes.
struct StatsJob {
    const float* row_loss = nullptr; int32_t n = 0;
    const int32_t* counts = nullptr; int32_t n_layers = 0; int32_t used_cache = 0;
    int32_t call_id = 0;                  // a flag word of `counts` is raised iff it holds this value
    int32_t feat_row_bytes = 0, emb_row_bytes = 0;
    no_step_stats* stats = nullptr;       // NULL: no job
};

// The reduction that follows a split product: sums the partials in split order into the three gradients; with
// lr != 0 also applies W <- W - lr * g.
struct ReduceArgs {
    float* P; int32_t splits, Kp, N;
    float* g_self; float* g_neigh; float* g_bias;
    float lr; float* w_self; float* w_neigh; float* w_bias;
    int32_t n_problems;                                  // 2, or 1: only g_self and g_bias
    // bf16 copies of the two matrices ([N][Kpad], weights_to_bf16_t's layout), rewritten with the updated values (or NULL)
    uint16_t* wt_self = nullptr; uint16_t* wt_neigh = nullptr; int32_t Kpad = 0;
};

// Weight-gradient work of several layers carried by one product launch and one reduction launch: the gradients of an
// upper layer are nobody's input within the step, so they need not sit on the step's chain of dependent launches
// between that layer's input gradient and the layer below. Job 0's blocks are dealt out first.
struct GradJobs {
    GemmTNArgs tn[NO_MAX_LAYERS]; ReduceArgs red[NO_MAX_LAYERS];
    int32_t n = 0;
    bool reuses_rows = false;      // the step takes rows from a cache
};

// ev0 / ev1 (optional): events that take the product kernel's own start and end times
// forward: one result, the sum of the products; input gradient: independent results, B transposed
int32_t gemm_nn_forward(const GemmNNArgs& a, hipStream_t st, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
// job: weight gradients that the launch may take along (*job_done: they went with it)
int32_t gemm_nn_input_grad(const GemmNNArgs& a, hipStream_t st, const GemmTNArgs* job, bool* job_done);
int32_t gemm_tn_partials(const GemmTNArgs* jobs, int32_t n_jobs, hipStream_t st, hipEvent_t ev0 = nullptr,
                         hipEvent_t ev1 = nullptr);
int32_t reduce_grads(const ReduceArgs* jobs, int32_t n_jobs, hipStream_t st, const StatsJob* stats_job = nullptr);

}  // namespace no
