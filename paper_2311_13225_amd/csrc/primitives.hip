// Error state, fills, the tile-offset stage of the prefix sum and a stable LSD radix sort of
// (key, value) pairs. The sort is what makes the block transpose, the CSR build and the hot-set
// ranking deterministic: equal keys keep their input order.
#include "primitives.hpp"
#include "radix.hpp"

#include <string.h>

namespace no {

static thread_local char g_err[512] = "";

void set_error(const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
}
void clear_error() { g_err[0] = 0; }

// ------------------------------------------------------------------------------------ fill

__global__ void fill_i32_kernel(int32_t* d, int32_t value, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) d[i] = value;
}

int32_t fill_i32(int32_t* d, int32_t value, int64_t n, hipStream_t st) {
    if (n <= 0) return NO_OK;
    int64_t blocks = ceil_div(n, 256 * 8);
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)blocks), dim3(256), 0, st, d, value, n);
    return launch_status("fill_i32");
}

// ------------------------------------------------------------------------------------ scan

__global__ void __launch_bounds__(1024) scan_tile_offsets_kernel(const int32_t* d_n, int64_t cap, int64_t* tile_sums) {
    int64_t n = d_n ? (int64_t)*d_n : cap;
    if (n > cap) n = cap;
    int64_t tiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    __shared__ int64_t smem[1024 / 64 + 1];
    int64_t carry = 0;
    for (int64_t base = 0; base < tiles; base += 1024) {
        int64_t i = base + threadIdx.x;
        int64_t v = i < tiles ? tile_sums[i] : 0;
        int64_t total;
        int64_t ex = block_exclusive_scan<int64_t, 1024>(v, &total, smem);
        if (i < tiles) tile_sums[i] = carry + ex;
        carry += total;
    }
}

size_t scan_ws_bytes(int64_t cap) { return scan_ws_bytes_impl(cap); }

int32_t exclusive_scan_i32(const int32_t* d_in, const int32_t* d_n, int64_t cap, int32_t* d_out, int32_t* d_total,
                           void* ws, hipStream_t st) {
    return exclusive_scan<ArrayLoader, int32_t>(ArrayLoader{d_in}, d_n, cap, d_out, d_total, ws, st);
}

// ------------------------------------------------------------------------------------ radix sort

__global__ void __launch_bounds__(RS_THREADS) rs_chunks_kernel(uint32_t* chunk, int64_t n_chunks, uint32_t* totals) {
    __shared__ uint32_t sums[RS_WAVES][64];
    const int lane = lane_id(), wave = (int)(threadIdx.x >> 6);
    const int64_t per = (n_chunks + RS_WAVES - 1) / RS_WAVES, c0 = wave * per, c1 = min(n_chunks, c0 + per);
    uint32_t* col = chunk + blockIdx.x * 64 + lane;
    uint32_t s = 0;
#pragma unroll 8
    for (int64_t c = c0; c < c1; ++c) s += col[c * RS_RADIX];
    sums[wave][lane] = s;
    __syncthreads();
    uint32_t run = 0, all = 0;
#pragma unroll
    for (int w = 0; w < RS_WAVES; ++w) {
        if (w < wave) run += sums[w][lane];
        all += sums[w][lane];
    }
    if (wave == 0) totals[blockIdx.x * 64 + lane] = all;
#pragma unroll 8
    for (int64_t c = c0; c < c1; ++c) {
        const uint32_t x = col[c * RS_RADIX];
        col[c * RS_RADIX] = run;
        run += x;
    }
}

size_t radix_ws_bytes(int64_t n) { return RadixPlan(n).ws_words() * sizeof(uint32_t); }

int32_t radix_sort_pairs(const uint32_t* keys_in, const uint32_t* vals_in, uint32_t* keys_out, uint32_t* vals_out,
                         uint32_t* keys_tmp, uint32_t* vals_tmp, int64_t n, int bits, void* ws, hipStream_t st) {
    if (n <= 0) return NO_OK;
    if (n >= (1ll << 32)) { set_error("radix sort: more than 2^32-1 items"); return NO_ERR_UNSUPPORTED; }
    const int passes = radix_passes(bits), width = radix_digit_bits(bits);
    const RadixPlan plan(n);
    PairArrays in{keys_in, vals_in};
    for (int p = 0; p < passes; ++p) {
        const bool to_out = (passes - 1 - p) % 2 == 0;
        uint32_t* k = to_out ? keys_out : keys_tmp;
        uint32_t* v = to_out ? vals_out : vals_tmp;
        NO_CHECK(radix_pass(in, plan, p * width, width, k, v, ws, st));
        in = PairArrays{k, v};
    }
    return NO_OK;
}

}  // namespace no

extern "C" const char* no_last_error(void) { return no::g_err; }
