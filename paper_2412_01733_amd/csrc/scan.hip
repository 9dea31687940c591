// Row-wise exclusive prefix sums of a u32 table, one workgroup a row: the tile
// counts of the radix sort (a row per digit) and the block counts of the tree
// build (a row per level).  Each row is 4 bytes a tile of thousands of
// particles, so a workgroup a row is latency-bound (about 5 us at 1e7
// particles) and replaces the three launches of a device-wide scan (17 us).
#include "tc_internal.h"

namespace tc {
namespace {

constexpr int kRowThreads = 512;
constexpr int kRowItems = 4;

__global__ __launch_bounds__(kRowThreads) void k_scan_rows(uint32_t* __restrict__ table, int64_t cols,
                                                           uint32_t* __restrict__ totals)
{
    __shared__ uint32_t wsum[2][kRowThreads / 64];
    uint32_t* row = table + (int64_t)blockIdx.x * cols;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t carry = 0;
    int turn = 0;
    for (int64_t b = 0; b < cols; b += kRowThreads * kRowItems, turn ^= 1) {
        const int64_t i0 = b + (int64_t)threadIdx.x * kRowItems;
        uint32_t v[kRowItems], sum = 0;
#pragma unroll
        for (int k = 0; k < kRowItems; ++k) {
            v[k] = i0 + k < cols ? row[i0 + k] : 0u;
            sum += v[k];
        }
        uint32_t inc = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t u = __shfl_up(inc, o, 64);
            if (lane >= o) inc += u;
        }
        if (lane == 63) wsum[turn][w] = inc;
        __syncthreads();  // one barrier a turn: the two buffers alternate
        uint32_t off = carry, tot = 0;
#pragma unroll
        for (int i = 0; i < kRowThreads / 64; ++i) {
            const uint32_t s = wsum[turn][i];
            if (i < w) off += s;
            tot += s;
        }
        carry += tot;
        uint32_t ex = off + inc - sum;
#pragma unroll
        for (int k = 0; k < kRowItems; ++k) {
            if (i0 + k < cols) row[i0 + k] = ex;
            ex += v[k];
        }
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

}  // namespace

void launch_scan_rows(uint32_t* table, int rows, int64_t cols, uint32_t* totals, hipStream_t s)
{
    if (rows > 0) k_scan_rows<<<(unsigned)rows, kRowThreads, 0, s>>>(table, cols, totals);
}

}  // namespace tc
