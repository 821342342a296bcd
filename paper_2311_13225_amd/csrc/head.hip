// The last layer of a training step over the seeds and the loss, forward and backward, in one launch: aggregate, product, softmax
// cross-entropy and both input gradients.
//
// A batch has 1 to 4 thousand seeds and some tens of classes: each of these passes is a few microseconds of waiting for memory behind a
// launch of its own, and none fills the chip. A block owns 16 seeds from their neighbours' rows to the gradients of these rows, so
// that nothing but weights and rows comes from memory: mean and own rows, then the logits, then their gradients stand in LDS. The
// weights are asked for ahead of the rows, which are two dependent reads away.
// Measured on the training stream, four launches -> this, us: 1024 seeds, 2 x 256 columns, 47 classes, 9 neighbours 26 -> 14; 41 classes, 22
// neighbours, beside the next batch's sampling 33 -> 19; 172 classes 37 -> 25; 4096 seeds 73 -> 32; 256 seeds, 2 x 64 columns, 16 classes 20 -> 10. (With the
// gradients of the rows in one chain of the fp32 instruction; as they are now up to 1.1 us more up to 64 classes, 0.5 to 1.5 above.)
//
// The logits' product on the fp32 instruction (v_mfma_f32_16x16x4_f32), the reduction dealt to the wavefronts and their parts added in pairs: relative 2-norm
// error against 64 bits 1.2e-7 at 2 x 256 terms, as that of the launches before it or less (1.2e-7 in small blocks, 2.1e-7 in tiles). The gradients of the
// rows in 64 bits up to 64 classes (v_mfma_f64_16x16x4_f64, half that rate); of more, where that would cost 2 to 6 us, in runs of 8 terms, or of 16 from 129 classes on, of
// the fp32 instruction, which are added up in 64 bits beside it. Their errors, the launches before this / one chain / this, 1e-7, 256 columns, 4096 seeds: 41 classes
// 0.57 / 0.93 / 0.25, 64 0.64 / 1.07 / 0.25, 65 0.64 / - / 0.59, 128 0.88 / - / 0.58, 129 0.87 / - / 0.81, 172 1.00 / 1.69 / 0.76, 240 1.09 / - / 0.75; 1024 seeds 0.96 to 1.17 before.
//
// Operands straight from LDS (rows) and L2 (weights). Bound by round trips (launched
// alone, 47 classes: rows 6.6 of 13.1 us, product 2.8, gradients of the rows 2.5), with 172 classes by the 64 compute units that 1024 seeds fill (product 8 of
// 20 us, 5.1 of them at the instruction's rate). Eight wavefronts, two rows each:
// with four, whose rows queue up, the 41 classes took 27 us, and instructions are fetched faster than used only in short code: unrolled
// loads with 64-bit addresses and guards (16 KB) cost another 2 us.
#include "gemm_tile.hpp"
#include "handles.hpp"
#include "layers.hpp"
#include "riders.hpp"

#include <algorithm>
#include <type_traits>

namespace no {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

// 16 bytes at a 4-byte aligned byte offset from a pointer that the whole wavefront shares (one instruction, no 64-bit address per lane)
__device__ __forceinline__ float4 load4_at(const float* base, uint32_t bytes) {
    return load4_fast(reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + bytes));
}

constexpr int HEAD_WAVES = 8, HEAD_THREADS = 64 * HEAD_WAVES;

template <int G, typename Side>      // G: 64-column groups of the classes
__global__ void __launch_bounds__(HEAD_THREADS) head_kernel(HeadArgs g, Side side) {
    if (blockIdx.x >= side.first_block) {
        // (the tasks' barriers wait for the wavefronts that have not ended: the other half of the block has no part in them)
        if (threadIdx.x < SIDE_THREADS) run_side_tasks(side);
        return;
    }
    constexpr int R = HEAD_ROWS, NW = HEAD_WAVES, RW = R / NW, ZP = 64 * G + 4, CP = 68;
    constexpr int ROWS = R * (2 * HEAD_MOST_COLUMNS + 4), PARTS = NW * R * CP;
    __shared__ __attribute__((aligned(16))) float tile[ROWS > PARTS ? ROWS : PARTS];      // own rows | aggregates; then the partial logits
    __shared__ __attribute__((aligned(16))) float Z[R * ZP];                            // logits, then their gradients
    __shared__ int32_t idx_sh[R * NO_MAX_FANOUT], len_sh[R];
    const int tid = (int)threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l16 = lane & 15, quad = lane >> 4;
    const int d = g.d, C = g.C, n = g.n, m0 = (int)(blockIdx.x % g.row_blocks) * R, part = (int)(blockIdx.x / g.row_blocks);
    const bool two = g.w_neigh != nullptr;
    const int phases = two ? 2 : 1, P = phases * d + 4, units = d / 4;

    // Rows of the block that this wavefront collects: their ends, their entries, then the rows themselves, each a read behind the one before.
    const int r0 = wave * RW;
    const int seg = g.indptr[min(m0 + r0 + min(lane, RW), n)];
    // this thread's seed from the logits on, 32 threads a seed
    const int r32 = tid >> 5, j32 = tid & 31, row = m0 + r32;
    const int seed = g.seeds[min(row, n - 1)];
    const bool stores = row < n && part == 0;

    // Weights of this wavefront's first chunks (16 indices of the reduction: lane group q has rows 4 q .. 4 q + 3 of them; of 64 columns a lane has
    // four neighbouring ones, each of another 16 x 16 product. Past the last column: the last four again, whose results are the same.)
    const int nc = (d + 15) / 16, chunks = phases * nc, mine = chunks > wave ? (chunks - wave + NW - 1) / NW : 0;
    constexpr int AHEAD = G == 1 ? 4 : G < 4 ? 2 : 1, B = 8;      // (what the registers of two wavefronts a SIMD hold)
    uint32_t cb[G];
#pragma unroll
    for (int j = 0; j < G; ++j) cb[j] = 4u * (uint32_t)min(64 * j + 4 * l16, C - 4);
    const uint32_t pitch = 4u * (uint32_t)C;
    float4 wbuf[AHEAD][4][G];
    auto request = [&](float4 (&w)[4][G], int i) {      // (past the last chunk: that one again, not used)
        const int c = wave + NW * min(i, max(mine - 1, 0));
        const bool second = c >= nc;
        const uint32_t k = (uint32_t)min((second ? c - nc : c) * 16 + 4 * quad, d - 4) * pitch;
        const float* W = second ? g.w_neigh : g.w_self;
#pragma unroll
        for (int s = 0; s < 4; ++s, W += C)
#pragma unroll
            for (int j = 0; j < G; ++j) w[s][j] = load4_at(W, k + cb[j]);
    };
    float bias[G][2];      // of the columns that this thread adds up
#pragma unroll
    for (int j = 0; j < G; ++j)
#pragma unroll
        for (int e = 0; e < 2; ++e) bias[j][e] = g.bias[min(64 * j + (2 * j32 & ~3), C - 4) + (2 * j32 & 2) + e];
    {
        const int e0 = __builtin_amdgcn_readlane(seg, 0), n_idx = min(__builtin_amdgcn_readlane(seg, RW) - e0, RW * NO_MAX_FANOUT);
        int32_t* const idx_w = idx_sh + r0 * NO_MAX_FANOUT;
        static_assert(RW * NO_MAX_FANOUT <= 128 && RW * HEAD_MOST_COLUMNS / 4 <= 128, "two entries, and two units of the own rows, a lane");
        int32_t entry[2];
        float4 own[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int i = lane + 64 * h, r = r0 + i / units, u = i % units;
            if (i < n_idx) entry[h] = g.idx[e0 + i];
            own[h] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (two && i < RW * units && m0 + r < n) own[h] = *reinterpret_cast<const float4*>(g.x + (int64_t)(m0 + r) * d + 4 * u);
        }
        if (mine > 0) {      // (behind the entries, ahead of the rows)
#pragma unroll
            for (int a = 0; a < AHEAD; ++a) request(wbuf[a], a);
        }
        const int32_t next = __shfl(seg, (lane + 1) & 63, 64);
        if (lane < RW) len_sh[r0 + lane] = next - seg;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int i = lane + 64 * h;
            if (i < n_idx) idx_w[i] = entry[h];
            if (two && i < RW * units) *reinterpret_cast<float4*>(&tile[(r0 + i / units) * P + 4 * (i % units)]) = own[h];
        }
        __builtin_amdgcn_wave_barrier();      // (the entries are this wavefront's own)
        // the aggregate, in the order of the row (as segment_rows_kernel sums it)
        int g_log2 = 0;
        while ((1 << g_log2) < units) ++g_log2;
        const int u = lane & ((1 << g_log2) - 1);
        for (int q = lane >> g_log2; q < RW; q += 64 >> g_log2) {
            if (u >= units) continue;
            const int r = r0 + q;
            float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
            if (m0 + r < n) {
                const int len = len_sh[r];
                int p = 0;
                for (int h = 0; h < q; ++h) p += len_sh[r0 + h];
                const int e = p + len;
                const uint32_t at = 16u * (uint32_t)u, row_bytes = 4u * (uint32_t)d;      // (head_takes: the rows end below 2^32 bytes)
                if (g.agg_mode != AGG_NEIGH_MEAN) acc = load4_at(g.x, at + (uint32_t)(m0 + r) * row_bytes);
                for (; p < e; p += B) {
                    float4 v[B];
#pragma unroll
                    for (int j = 0; j < B; ++j) v[j] = load4_at(g.x, at + (uint32_t)idx_w[min(p + j, e - 1)] * row_bytes);      // (past the end: the last again, not added)
#pragma unroll
                    for (int j = 0; j < B; ++j)
                        if (p + j < e) { acc.x += v[j].x; acc.y += v[j].y; acc.z += v[j].z; acc.w += v[j].w; }
                }
                const float scale = g.agg_mode == AGG_NEIGH_MEAN ? (len > 0 ? 1.f / (float)len : 0.f)
                                  : g.agg_mode == AGG_SELF_MEAN  ? 1.f / (float)(len + 1) : 1.f;
                acc.x *= scale; acc.y *= scale; acc.z *= scale; acc.w *= scale;
                if (part == 0) *reinterpret_cast<float4*>(g.mean + (int64_t)(m0 + r) * d + 4 * u) = acc;
            }
            *reinterpret_cast<float4*>(&tile[r * P + (phases - 1) * d + 4 * u]) = acc;
        }
    }
    const int label = g.labels[seed];
    __syncthreads();
    floatx4 acc[G][4];
#pragma unroll
    for (int j = 0; j < G; ++j)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[j][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int i0 = 0; i0 < mine; i0 += AHEAD) {
#pragma unroll
        for (int a = 0; a < AHEAD; ++a) {
            if (i0 + a >= mine) break;
            const int c = wave + NW * (i0 + a), second = c >= nc ? 1 : 0, k = (c - second * nc) * 16 + 4 * quad;
            float4 x = *reinterpret_cast<const float4*>(&tile[l16 * P + second * d + min(k, d - 4)]);
            if (d % 16 && c - second * nc == nc - 1 && k >= d) {      // (a lane's four indices are in or out together: d is a multiple of 4)
                x = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int j = 0; j < G; ++j) wbuf[a][s][j] = x;
            }
            const float xs[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int j = 0; j < G; ++j) {
                    const float4 w = wbuf[a][s][j];
                    acc[j][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(xs[s], w.x, acc[j][0], 0, 0, 0);
                    acc[j][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(xs[s], w.y, acc[j][1], 0, 0, 0);
                    acc[j][2] = __builtin_amdgcn_mfma_f32_16x16x4f32(xs[s], w.z, acc[j][2], 0, 0, 0);
                    acc[j][3] = __builtin_amdgcn_mfma_f32_16x16x4f32(xs[s], w.w, acc[j][3], 0, 0, 0);
                }
            request(wbuf[a], i0 + a + AHEAD);
        }
    }
    // Gradients of the rows, below: 16 columns of one matrix's product at a time, the reduction over the classes in 16s. The weights of the first
    // are asked for here.
    const int per = (d + 15) / 16, n_tiles = phases * per, nk = (C + 15) / 16;
    float4 tbuf[4 * G];
    auto request_t = [&](int t) {
        const float* W = t >= per ? g.w_neigh : g.w_self;
        const uint32_t at = (uint32_t)min((t >= per ? t - per : t) * 16 + l16, d - 1) * pitch;
#pragma unroll
        for (int q = 0; q < 4 * G; ++q) tbuf[q] = load4_at(W, at + 4u * (uint32_t)min(q * 16 + 4 * quad, C - 4));
    };
    const int first_tile = part * NW + wave;
    if (first_tile < n_tiles) request_t(first_tile);
    // the wavefronts' parts of the logits, 64 columns at a time, over the rows, which are not needed any more
#pragma unroll
    for (int j = 0; j < G; ++j) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r)      // (element r of a lane: row 4 quad + r, column l16 of the product)
            *reinterpret_cast<float4*>(&tile[(wave * R + 4 * quad + r) * CP + 4 * l16]) = make_float4(acc[j][0][r], acc[j][1][r], acc[j][2][r], acc[j][3][r]);
        __syncthreads();
        if (64 * j + (2 * j32 & ~3) < C) {
            const int c = min(64 * j + (2 * j32 & ~3), C - 4) + (2 * j32 & 2);
            float2 s[NW];
#pragma unroll
            for (int w = 0; w < NW; ++w) s[w] = *reinterpret_cast<const float2*>(&tile[(w * R + r32) * CP + 2 * j32]);
#pragma unroll
            for (int o = NW / 2; o > 0; o >>= 1)
#pragma unroll
                for (int w = 0; w < o; ++w) { s[w].x += s[w + o].x; s[w].y += s[w + o].y; }
            const float z[2] = {s[0].x + bias[j][0], s[0].y + bias[j][1]};
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                Z[r32 * ZP + c + e] = z[e];
                if (stores) g.logits[(int64_t)row * C + c + e] = z[e];
            }
        }
    }
    __syncthreads();
    // softmax cross-entropy (as softmax_xent_kernel; the threads of a seed are 32 lanes of one wavefront)
    {
        float* z = &Z[r32 * ZP];
        float v[2 * G];
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < 2 * G; ++i) {
            v[i] = j32 + 32 * i < C ? z[j32 + 32 * i] : -INFINITY;
            mx = fmaxf(mx, v[i]);
        }
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
        float s = 0.f;
        const bool on = row < n && (uint32_t)label < (uint32_t)C;
        const float zy = on ? z[label] : 0.f;
#pragma unroll
        for (int i = 0; i < 2 * G; ++i) {
            const float e = expf(v[i] - mx);
            v[i] = j32 + 32 * i < C ? e : 0.f;
            s += v[i];
        }
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        const float inv = 1.f / s, inv_n = 1.f / (float)n;
        if (j32 == 0 && stores) {
            // a label outside [0, C): the seed adds nothing to the loss or the gradient, and the step is flagged
            g.row_loss[row] = on ? -(zy - mx - logf(s)) : 0.f;
            if (!on) *g.bad_label_flag = g.flag_value;
        }
#pragma unroll
        for (int i = 0; i < 2 * G; ++i) {
            const int c = j32 + 32 * i;
            const float p = on && c < C ? (v[i] * inv - (c == label ? 1.f : 0.f)) * inv_n : 0.f;
            z[c] = p;
            if (stores && c < C) g.grad[(int64_t)row * C + c] = p;
        }
    }
    __syncthreads();
    for (int t = first_tile; t < n_tiles; t += g.parts * NW) {
        const bool second = t >= per;
        doublex4 sum = {0.0, 0.0, 0.0, 0.0};
        if (t != first_tile) request_t(t);
#pragma unroll
        for (int q = 0; q < 4 * G; ++q) {
            if (q < nk) {
                const int k = q * 16 + 4 * quad;
                const float4 z = *reinterpret_cast<const float4*>(&Z[l16 * ZP + k]);
                float v[4] = {tbuf[q].x, tbuf[q].y, tbuf[q].z, tbuf[q].w};
                if (16 * q + 16 > C) {      // the last classes: read where they end, put right here
                    const int sh = k - min(k, C - 4);
                    const float f[4] = {v[0], v[1], v[2], v[3]};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        v[e] = 0.f;
#pragma unroll
                        for (int h = 0; h < 4; ++h)
                            if (e + h < 4) v[e] = sh == h ? f[(e + h) & 3] : v[e];
                    }
                }
                const float zs[4] = {z.x, z.y, z.z, z.w};
                if constexpr (G == 1) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum = __builtin_amdgcn_mfma_f64_16x16x4f64((double)zs[e], (double)v[e], sum, 0, 0, 0);
                } else {
                    constexpr int RUN = G == 2 ? 2 : 4;      // (four terms each)
#pragma unroll
                    for (int e = 0; e < 4; e += RUN) {
                        floatx4 run{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int i = e; i < e + RUN; ++i) run = __builtin_amdgcn_mfma_f32_16x16x4f32(zs[i], v[i], run, 0, 0, 0);
#pragma unroll
                        for (int r = 0; r < 4; ++r) sum[r] += (double)run[r];
                    }
                }
            }
        }
        const int i = (second ? t - per : t) * 16 + l16;
        if (i >= d) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int lr = G == 1 ? 4 * r + quad : 4 * quad + r;      // (element r of a lane: the 64-bit instruction's row 4 r + quad, the fp32 one's 4 quad + r)
            if (m0 + lr >= n) continue;
            const int len = len_sh[lr];
            const float s = two ? (second ? (len > 0 ? 1.f / (float)len : 0.f) : 1.f) : g.agg_mode == AGG_SELF_MEAN ? 1.f / (float)(len + 1) : 1.f;
            const float o = (float)sum[r] * s;
            const int64_t at = (int64_t)(m0 + lr) * d + i;
            if (!second) g.grad_self[at] = o;
            if (second || !two) g.grad_mean[at] = o;
        }
    }
}

int32_t head_forward_backward(const HeadArgs& args, const CutJobs& cut, no_blocks_s* side_of, hipStream_t st) {
    // Few seeds leave compute units idle: up to four blocks then go the same way to the logits' gradients, and each makes its part of the columns
    // of the gradients of the rows (at least a 16-column tile a wavefront).
    HeadArgs a = args;
    a.row_blocks = (uint32_t)ceil_div(a.n, HEAD_ROWS);
    const int64_t tiles = (a.w_neigh ? 2 : 1) * ceil_div(a.d, 16);
    a.parts = (int32_t)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(4, 256 / a.row_blocks), ceil_div(tiles, HEAD_WAVES)));
    const uint32_t own = a.row_blocks * (uint32_t)a.parts;
    launch_with_riders(&cut, side_of, own, [&](const auto& side, uint32_t grid) {
        using Side = std::decay_t<decltype(side)>;
        switch ((a.C + 63) / 64) {
            case 1: hipLaunchKernelGGL((head_kernel<1, Side>), dim3(grid), dim3(HEAD_THREADS), 0, st, a, side); break;
            case 2: hipLaunchKernelGGL((head_kernel<2, Side>), dim3(grid), dim3(HEAD_THREADS), 0, st, a, side); break;
            case 3: hipLaunchKernelGGL((head_kernel<3, Side>), dim3(grid), dim3(HEAD_THREADS), 0, st, a, side); break;
            default: hipLaunchKernelGGL((head_kernel<4, Side>), dim3(grid), dim3(HEAD_THREADS), 0, st, a, side); break;
        }
    });
    return launch_status("head");
}

}  // namespace no
