// Stable LSD radix sort of (u64 key, u32 value) pairs, 9-bit digits: the 63-bit
// keys take 7 passes (8 with 8-bit digits).
//
// Each pass is reduce-then-scan: per-tile digit counts (digit-major table), an
// exclusive scan of each digit's row, then a stable scatter, whose blocks add up
// the digit totals themselves.  Within a tile the
// rank of an element among equal digits comes from 64-lane ballots (the peer
// mask of lanes holding the same digit), accumulated wave by wave in LDS, so
// element order inside every digit run is the input order: the sort is
// stable, which makes ties fall back to the original particle index.
// The scatter goes through LDS so that every digit run is written to HBM as
// contiguous, coalesced stores.
//
// A pass moves 32 bytes a pair.  What bounds it is the scatter's runs, which
// start and end inside cache lines: neighbouring tiles complete each other's
// lines, so each XCD takes a contiguous range of tiles and its L2 puts the lines
// together.  Sort stage (with the gather) at 1e7 keys: 1.02 ms with tiles dealt
// round robin over the XCDs, 8-bit digits and 256 threads; 0.86 with the ranges,
// 0.84 with 512 threads and 9-bit digits (1.21 with 9-bit digits and tiles dealt
// round robin).
#include "tc_internal.h"

namespace tc {
namespace {

constexpr int kRadixBits = 9;
constexpr int kRadix = 1 << kRadixBits;
constexpr int kSortThreads = 512;
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kDigitsLane = kRadix / kSortThreads;
static_assert(kDigitsLane * kSortThreads == kRadix && kDigitsLane >= 1, "a block serves every digit");

// Keys per lane.  6: the scatter's 47 KB of LDS fit 3 blocks (24 waves) a CU; 7
// measured the same, 8 fits 2 blocks and is 3 % slower.  4 below kFewKeys, where
// tiles of 3072 leave CUs with one block beside CUs with two: sort stage 176 us
// instead of 188 at 1e6 keys, 136 / 140 at 5.3e5, 205 / 205 at 1.5e6, 885 / 841
// at 1e7.
constexpr int kItemsLarge = 6;
constexpr int kItemsSmall = 4;
constexpr int64_t kFewKeys = 5 << 18;

constexpr int sort_tile(int items) { return kSortThreads * items; }

__device__ inline uint32_t lane_id() { return threadIdx.x & 63; }

// Count of set bits of m strictly below this lane.
__device__ inline uint32_t popc_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Inclusive prefix sum over the block's threads.
__device__ inline uint32_t scan_block(uint32_t v, uint32_t lane, int w, uint32_t* wsum)
{
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = __shfl_up(v, o, 64);
        if ((int)lane >= o) v += u;
    }
    if (lane == 63) wsum[w] = v;
    __syncthreads();
    for (int i = 0; i < w; ++i) v += wsum[i];
    return v;
}

// Mask of the lanes of this wave whose (valid) digit equals ours.
__device__ inline uint64_t peer_mask(uint32_t d, bool valid)
{
    uint64_t m = __ballot(valid);
#pragma unroll
    for (int b = 0; b < kRadixBits; ++b) {
        uint64_t bal = __ballot((d >> b) & 1u);
        m &= ((d >> b) & 1u) ? bal : ~bal;
    }
    return m;
}

// Blocks are dealt to the 8 XCDs in turn; XCD x takes the x-th eighth of the
// tiles (the first ntiles % 8 eighths are one longer).  The grid is the tiles.
__device__ inline int64_t tile_of_block()
{
    const uint32_t x = blockIdx.x & 7u, q = gridDim.x >> 3, r = gridDim.x & 7u;
    return (int64_t)(x * q + (x < r ? x : r) + (blockIdx.x >> 3));
}

template <int ITEMS>
__global__ __launch_bounds__(kSortThreads) void k_upsweep(const uint64_t* __restrict__ keys, int64_t n,
                                                          int shift, uint32_t* __restrict__ counts,
                                                          int64_t ntiles)
{
    __shared__ uint32_t hist[kSortWaves][kRadix];
    for (int j = threadIdx.x; j < kSortWaves * kRadix; j += kSortThreads) (&hist[0][0])[j] = 0;
    __syncthreads();
    const int w = threadIdx.x >> 6;
    const uint32_t lane = lane_id();
    const int64_t tile = tile_of_block();
    const int64_t base = tile * sort_tile(ITEMS) + (int64_t)w * (64 * ITEMS);
    uint64_t key[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int64_t i = base + k * 64 + lane;
        key[k] = i < n ? keys[i] : 0ull;
    }
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const bool valid = base + k * 64 + lane < n;
        const uint32_t d = (uint32_t)(key[k] >> shift) & (kRadix - 1);
        uint64_t peers = peer_mask(d, valid);
        if (valid && popc_below(peers) == 0) hist[w][d] += (uint32_t)__popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    for (int d = threadIdx.x; d < kRadix; d += kSortThreads) {
        uint32_t t = 0;
        for (int ww = 0; ww < kSortWaves; ++ww) t += hist[ww][d];
        counts[(int64_t)d * ntiles + tile] = t;
    }
}

template <int ITEMS>
__global__ __launch_bounds__(kSortThreads) void k_downsweep(const uint64_t* __restrict__ kin,
                                                            const uint32_t* __restrict__ vin,
                                                            uint64_t* __restrict__ kout,
                                                            uint32_t* __restrict__ vout, int64_t n,
                                                            int shift,
                                                            const uint32_t* __restrict__ offsets,
                                                            const uint32_t* __restrict__ totals,
                                                            int64_t ntiles)
{
    constexpr int kTile = sort_tile(ITEMS);
    static_assert(kTile < 1 << 16, "places within a tile are kept in 16 bits");
    __shared__ uint16_t wcnt[kSortWaves][kRadix];
    __shared__ uint32_t gbase[kRadix];
    __shared__ uint32_t dsum[2][kSortWaves];
    __shared__ uint64_t sk[kTile];
    __shared__ uint32_t sv[kTile];

    const int64_t tile = tile_of_block();
    const int w = threadIdx.x >> 6;
    const uint32_t lane = lane_id();
    const int d0 = (int)threadIdx.x * kDigitsLane;
    for (int j = threadIdx.x; j < kSortWaves * kRadix / 2; j += kSortThreads) ((uint32_t*)&wcnt[0][0])[j] = 0;
    {
        // first place of each digit: the totals of the digits below it, and of this digit's tiles before
        uint32_t tot[kDigitsLane], sum = 0;
#pragma unroll
        for (int j = 0; j < kDigitsLane; ++j) { tot[j] = totals[d0 + j]; sum += tot[j]; }
        uint32_t v = scan_block(sum, lane, w, dsum[0]) - sum;
#pragma unroll
        for (int j = 0; j < kDigitsLane; ++j) {
            gbase[d0 + j] = v + offsets[(int64_t)(d0 + j) * ntiles + tile];
            v += tot[j];
        }
    }

    const int64_t tbase = tile * kTile;
    const int64_t base = tbase + (int64_t)w * (64 * ITEMS);

    uint64_t key[ITEMS];
    uint32_t val[ITEMS];
    uint32_t rank[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        int64_t i = base + k * 64 + lane;
        bool valid = i < n;
        key[k] = valid ? kin[i] : 0ull;
        val[k] = valid ? vin[i] : 0u;
    }
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        int64_t i = base + k * 64 + lane;
        bool valid = i < n;
        uint32_t d = (uint32_t)(key[k] >> shift) & (kRadix - 1);
        uint64_t peers = peer_mask(d, valid);
        uint32_t below = popc_below(peers);
        uint32_t old = valid ? wcnt[w][d] : 0u;
        __builtin_amdgcn_wave_barrier();
        if (valid && below == 0) wcnt[w][d] = (uint16_t)(old + (uint32_t)__popcll(peers));
        __builtin_amdgcn_wave_barrier();
        rank[k] = old + below;
    }
    __syncthreads();
    // first place in the tile of each wave's digits; gbase becomes what takes a
    // place in the tile to its place in the output (modulo 2^32: n is below it)
    uint32_t tot[kDigitsLane], sum = 0;
#pragma unroll
    for (int j = 0; j < kDigitsLane; ++j) {
        tot[j] = 0;
        for (int ww = 0; ww < kSortWaves; ++ww) tot[j] += wcnt[ww][d0 + j];
        sum += tot[j];
    }
    uint32_t v = scan_block(sum, lane, w, dsum[1]) - sum;
#pragma unroll
    for (int j = 0; j < kDigitsLane; ++j) {
        gbase[d0 + j] -= v;
        for (int ww = 0; ww < kSortWaves; ++ww) {
            const uint32_t c = wcnt[ww][d0 + j];
            wcnt[ww][d0 + j] = (uint16_t)v;
            v += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        if (base + k * 64 + lane < n) {
            const uint32_t p = wcnt[w][(uint32_t)(key[k] >> shift) & (kRadix - 1)] + rank[k];
            sk[p] = key[k];
            sv[p] = val[k];
        }
    }
    __syncthreads();
    const int64_t rem = n - tbase;
    const int tn = rem < kTile ? (int)rem : kTile;
    for (int j = threadIdx.x; j < tn; j += kSortThreads) {
        uint64_t k = sk[j];
        uint32_t d = (uint32_t)(k >> shift) & (kRadix - 1);
        const uint32_t g = gbase[d] + (uint32_t)j;
        if (g < n) {  // always true for consistent counts; guards the store
            kout[g] = k;
            vout[g] = sv[j];
        }
    }
}

int sort_items(int64_t n) { return n < kFewKeys ? kItemsSmall : kItemsLarge; }

int64_t sort_tiles(int64_t n)
{
    const int tile = sort_tile(sort_items(n));
    return (n + tile - 1) / tile;
}

}  // namespace

size_t radix_temp_bytes(int64_t n)
{
    return ((size_t)(sort_tiles(n) + 1) * kRadix * 4 + 255) & ~(size_t)255;
}

void radix_sort_pairs(uint64_t* keys, uint32_t* vals, uint64_t* keys_alt, uint32_t* vals_alt, int64_t n,
                      int bits, void* temp, hipStream_t s, uint64_t** keys_out, uint32_t** vals_out)
{
    *keys_out = keys;
    *vals_out = vals;
    if (n <= 1) return;
    const bool small = sort_items(n) == kItemsSmall;
    const int64_t ntiles = sort_tiles(n);
    uint32_t* counts = (uint32_t*)temp;
    uint32_t* totals = counts + ntiles * kRadix;
    uint64_t* kin = keys;
    uint32_t* vin = vals;
    uint64_t* ko = keys_alt;
    uint32_t* vo = vals_alt;
    for (int shift = 0; shift < bits; shift += kRadixBits) {
        const dim3 grid((unsigned)ntiles), block(kSortThreads);
        if (small) k_upsweep<kItemsSmall><<<grid, block, 0, s>>>(kin, n, shift, counts, ntiles);
        else k_upsweep<kItemsLarge><<<grid, block, 0, s>>>(kin, n, shift, counts, ntiles);
        launch_scan_rows(counts, kRadix, ntiles, totals, s);
        if (small) k_downsweep<kItemsSmall><<<grid, block, 0, s>>>(kin, vin, ko, vo, n, shift, counts, totals, ntiles);
        else k_downsweep<kItemsLarge><<<grid, block, 0, s>>>(kin, vin, ko, vo, n, shift, counts, totals, ntiles);
        uint64_t* tk = kin; kin = ko; ko = tk;
        uint32_t* tv = vin; vin = vo; vo = tv;
    }
    *keys_out = kin;
    *vals_out = vin;
}

}  // namespace tc
