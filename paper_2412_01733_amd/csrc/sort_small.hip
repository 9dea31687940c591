// Keys, sort and gather for inputs that a radix sort's passes do not pay for.
//
// A pass of sort.hip costs three launches, and seven passes are needed whatever
// n is (keys, sort and gather: 120 us at 1.3e5 particles, against 92 here; 140 and
// 125 at 4e5; 150 and 138 at 5.2e5; 183 and 248 at 8e5).
// Here one launch computes the keys of tiles of 2048 particles and sorts each
// tile in LDS; then every launch merges up to 8 neighbouring runs by rank: a
// key's place is its own place in its run plus the number of keys before it in
// each of the other runs, found by binary search (equal keys keep the order of
// their runs, so the sort is stable).  The searches of a key are independent
// and neighbouring threads probe neighbouring keys, so a pass is a few L2
// round trips.  The last launch gathers the particles into key order.
#include "keys_common.h"
#include "walk_common.h"

namespace tc {
namespace {

constexpr int kTileThreads = 512;
constexpr int kTileWaves = kTileThreads / 64;
constexpr int kTileItems = 4;
constexpr int kWaveItems = 64 * kTileItems;
constexpr int kTile = kTileThreads * kTileItems;  // 2048
constexpr int kDigits = 256;

template <typename T>
__device__ inline void gather_one(const T* __restrict__ pos, const T* __restrict__ mass, uint32_t i, Particle* __restrict__ out)
{
    const double x = (double)pos[3 * (int64_t)i + 0], y = (double)pos[3 * (int64_t)i + 1], z = (double)pos[3 * (int64_t)i + 2];
    double2* o = reinterpret_cast<double2*>(out);
    o[0] = make_double2(x, y);
    o[1] = make_double2(z, (double)mass[i]);
}

// One tile: root cube (from the bounds' partials, or from the tile itself if it
// is the only one), keys, sort in LDS; a lone tile is gathered too.  Ranks come
// from 64-lane ballots as in sort.hip.  Bound by the instructions of 8 passes
// (~2000 a wave; 8 us at 512 threads), not by its 32 bytes a particle.
template <typename T>
__global__ __launch_bounds__(kTileThreads) void k_tile_sort(const T* __restrict__ pos, const T* __restrict__ mass,
                                                            int64_t n, const double* __restrict__ part, int nparts,
                                                            Geom* __restrict__ geom, uint64_t* __restrict__ keys,
                                                            uint32_t* __restrict__ vals, Particle* __restrict__ sp)
{
    __shared__ uint64_t sk[kTile];
    __shared__ uint16_t sv[kTile];
    __shared__ uint32_t cnt[kTileWaves][kDigits];
    __shared__ uint32_t start[kDigits];
    __shared__ uint32_t dsum[kDigits / 64];
    __shared__ double red[kTileWaves][8];
    __shared__ Geom g;
    const int w = threadIdx.x >> 6;
    const uint32_t lane = threadIdx.x & 63;
    const int64_t tbase = (int64_t)blockIdx.x * kTile;
    const int tn = n - tbase < kTile ? (int)(n - tbase) : kTile;

    {
        double mm[6] = {DBL_MAX, DBL_MAX, DBL_MAX, -DBL_MAX, -DBL_MAX, -DBL_MAX};
        uint32_t bad = 0;
        if (nparts == 0) {
            for (int j = threadIdx.x; j < tn; j += kTileThreads) bounds_add(pos, mass, j, mm, bad);
        } else {
            for (int b = threadIdx.x; b < nparts; b += kTileThreads) {
                for (int k = 0; k < 3; ++k) {
                    mm[k] = fmin(mm[k], part[8 * b + k]);
                    mm[3 + k] = fmax(mm[3 + k], part[8 * b + 3 + k]);
                }
                bad |= (uint32_t)part[8 * b + 6];
            }
        }
        bounds_wave(mm, bad);
        if (lane == 0) {
            for (int k = 0; k < 6; ++k) red[w][k] = mm[k];
            red[w][6] = (double)bad;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int u = 1; u < kTileWaves; ++u) {
                for (int k = 0; k < 3; ++k) {
                    mm[k] = fmin(mm[k], red[u][k]);
                    mm[3 + k] = fmax(mm[3 + k], red[u][3 + k]);
                }
                bad |= (uint32_t)red[u][6];
            }
            g = make_geom(mm, bad);
            if (blockIdx.x == 0) *geom = g;
        }
        __syncthreads();
    }

    uint64_t key[kTileItems];
    uint32_t val[kTileItems], rank[kTileItems];
#pragma unroll
    for (int k = 0; k < kTileItems; ++k) {
        const int j = w * kWaveItems + k * 64 + (int)lane;
        key[k] = 0;
        val[k] = (uint32_t)j;
        if (j < tn) {
            const int64_t i = tbase + j;
            key[k] = morton(quantise((double)pos[3 * i + 0], g.lo[0], g.scale), quantise((double)pos[3 * i + 1], g.lo[1], g.scale),
                            quantise((double)pos[3 * i + 2], g.lo[2], g.scale));
        }
    }
    for (int shift = 0; shift < 64; shift += 8) {
        for (int j = threadIdx.x; j < kTileWaves * kDigits; j += kTileThreads) (&cnt[0][0])[j] = 0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kTileItems; ++k) {
            const bool valid = w * kWaveItems + k * 64 + (int)lane < tn;
            const uint32_t d = (uint32_t)(key[k] >> shift) & (kDigits - 1);
            uint64_t peers = __ballot(valid);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const uint64_t bal = __ballot((d >> b) & 1u);
                peers &= ((d >> b) & 1u) ? bal : ~bal;
            }
            const uint32_t below = popc_below(peers);
            const uint32_t old = valid ? cnt[w][d] : 0u;
            __builtin_amdgcn_wave_barrier();
            if (valid && below == 0) cnt[w][d] = old + (uint32_t)__popcll(peers);
            __builtin_amdgcn_wave_barrier();
            rank[k] = old + below;
        }
        __syncthreads();
        uint32_t tot = 0, inc = 0;
        if (threadIdx.x < kDigits) {
#pragma unroll
            for (int u = 0; u < kTileWaves; ++u) {
                const uint32_t c = cnt[u][threadIdx.x];
                cnt[u][threadIdx.x] = tot;
                tot += c;
            }
            inc = tot;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t u = __shfl_up(inc, o, 64);
                if ((int)lane >= o) inc += u;
            }
            if (lane == 63) dsum[w] = inc;
        }
        __syncthreads();
        if (threadIdx.x < kDigits) {
            uint32_t off = 0;
            for (int u = 0; u < w; ++u) off += dsum[u];
            start[threadIdx.x] = off + inc - tot;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kTileItems; ++k) {
            if (w * kWaveItems + k * 64 + (int)lane < tn) {
                const uint32_t d = (uint32_t)(key[k] >> shift) & (kDigits - 1);
                const uint32_t p = start[d] + cnt[w][d] + rank[k];
                sk[p] = key[k];
                sv[p] = (uint16_t)val[k];
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kTileItems; ++k) {
            const int j = w * kWaveItems + k * 64 + (int)lane;
            if (j < tn) {
                key[k] = sk[j];
                val[k] = sv[j];
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kTileItems; ++k) {
        const int j = w * kWaveItems + k * 64 + (int)lane;
        if (j < tn) {
            const uint32_t i = (uint32_t)tbase + val[k];
            keys[tbase + j] = key[k];
            vals[tbase + j] = i;
            if (sp) gather_one(pos, mass, i, sp + tbase + j);
        }
    }
}

// Merges groups of K neighbouring sorted runs (each of `run` keys, a power of
// two; the last ones shorter or empty).  GATHER: the last pass also writes the
// particles in key order.
template <int K, bool GATHER, typename T>
__global__ __launch_bounds__(256) void k_merge(const uint64_t* __restrict__ kin, const uint32_t* __restrict__ vin,
                                               uint64_t* __restrict__ kout, uint32_t* __restrict__ vout, int64_t n,
                                               int64_t run, const T* __restrict__ pos, const T* __restrict__ mass,
                                               Particle* __restrict__ sp)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t key = kin[i];
    const uint32_t val = vin[i];
    const int64_t r = i / run, g0 = r / K * K;
    const int mine = (int)(r - g0);
    const uint64_t* start[K - 1];
    uint32_t len[K - 1], p[K - 1];
    uint64_t lim[K - 1];  // keys below lim come first: an equal key of an earlier run does
#pragma unroll
    for (int q = 0; q < K - 1; ++q) {
        const int o = q < mine ? q : q + 1;
        const int64_t b = (g0 + o) * run;
        start[q] = kin + (b < n ? b : 0);
        len[q] = b < n ? (uint32_t)(n - b < run ? n - b : run) : 0u;
        lim[q] = key + (o < mine ? 1ull : 0ull);
        p[q] = 0;
    }
    for (uint32_t b = (uint32_t)run; b; b >>= 1) {
#pragma unroll
        for (int q = 0; q < K - 1; ++q) {
            const uint32_t at = p[q] + b;
            const bool in = at <= len[q];
            const uint64_t kq = start[q][in ? at - 1 : 0];
            if (in && kq < lim[q]) p[q] = at;
        }
    }
    int64_t d = g0 * run + (i - r * run);
#pragma unroll
    for (int q = 0; q < K - 1; ++q) d += p[q];
    kout[d] = key;
    vout[d] = val;
    if constexpr (GATHER) gather_one(pos, mass, val, sp + d);
}

template <typename T>
void sort_small_t(const T* pos, const T* mass, int64_t n, const double* part, int nparts, Geom* geom, uint64_t* k0,
                  uint32_t* v0, uint64_t* k1, uint32_t* v1, Particle* sp, hipStream_t s, uint64_t** keys_out,
                  uint32_t** vals_out)
{
    int64_t runs = (n + kTile - 1) / kTile, run = kTile;
    k_tile_sort<T><<<(unsigned)runs, kTileThreads, 0, s>>>(pos, mass, n, part, nparts, geom, k0, v0, runs == 1 ? sp : nullptr);
    int passes = 0;
    for (int64_t c = 1; c < runs; c *= 8) ++passes;
    const unsigned grid = (unsigned)((n + 255) / 256);
    for (; passes > 0; --passes) {
        // the least K of 2, 4, 8 with which the remaining passes suffice
        int K = 2;
        for (; K < 8; K *= 2) {
            int64_t c = 1;
            for (int q = 0; q < passes; ++q) c *= K;
            if (c >= runs) break;
        }
        const bool last = passes == 1;
#define TC_MERGE(KK)                                                                                              \
    do {                                                                                                          \
        if (last) k_merge<KK, true, T><<<grid, 256, 0, s>>>(k0, v0, k1, v1, n, run, pos, mass, sp);              \
        else k_merge<KK, false, T><<<grid, 256, 0, s>>>(k0, v0, k1, v1, n, run, pos, mass, sp);                  \
    } while (0)
        if (K == 2) TC_MERGE(2);
        else if (K == 4) TC_MERGE(4);
        else TC_MERGE(8);
#undef TC_MERGE
        run *= K;
        runs = (runs + K - 1) / K;
        uint64_t* tk = k0; k0 = k1; k1 = tk;
        uint32_t* tv = v0; v0 = v1; v1 = tv;
    }
    *keys_out = k0;
    *vals_out = v0;
}

}  // namespace

bool sort_small_lone(int64_t n) { return n <= kTile; }

void launch_sort_small(const void* pos, const void* mass, int64_t n, tc_dtype dt, const double* part, int nparts,
                       Geom* geom, uint64_t* k0, uint32_t* v0, uint64_t* k1, uint32_t* v1, Particle* sp, hipStream_t s,
                       uint64_t** keys_out, uint32_t** vals_out)
{
    if (dt == TC_F32)
        sort_small_t<float>((const float*)pos, (const float*)mass, n, part, nparts, geom, k0, v0, k1, v1, sp, s, keys_out, vals_out);
    else
        sort_small_t<double>((const double*)pos, (const double*)mass, n, part, nparts, geom, k0, v0, k1, v1, sp, s, keys_out, vals_out);
}

}  // namespace tc
