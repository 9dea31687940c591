// Upward pass: monopole moments of every node (TreeCode description of
// section 2: a distant cell acts as its total mass at its centre of mass).
//
// A node needs its children's finished records, which are consecutive in the
// breadth-first array.  Up to kByBlocks particles a workgroup takes a part of the
// particles' order and sums the nodes within it level by level, deepest first;
// the few nodes that cross from one part into the next follow, again level by
// level, in one workgroup.  Above, one launch per populous level
// and one single-workgroup launch per run of small levels.
// The parts are bound by the dependent reads of their levels (two round trips to
// the L2 each, ~2 us), the populous levels by HBM (39 us a level at 1e7).
// Everything is FP64 with no FMA contraction, summed in a fixed order
// (particles in key order inside a leaf, children in octant order), so the
// result does not depend on scheduling:
//   leaf of one particle:  M = m_j, X = x_j exactly;
//   otherwise:             M = sum M_c, X = (sum M_c X_c) / M,
//                          X = the cell centre when M = 0.
// The same pass writes the node's whole walk record.
#include "tc_internal.h"

namespace tc {
namespace {

// Up to kByBlocks particles a workgroup sums the nodes within its part of the
// order, whatever their level; above, every level has its launch.  Moments stage
// (with the target order), by parts / by levels: 24 / 26 us at 1000, 41 / 56 at
// 20000, 47 / 72 at 1e5, 64 / 91 at 2.6e5, 76 / 112 at 5.2e5, 91 / 123 at 6.4e5; with
// parts of 1024 114 / 107 at 7e5, 144 / 119 at 1e6 and 0.92 / 0.87 ms at 1e7, where
// a part's few nodes a level wait for memory one level after the other, while a
// level's launch fills the chip.
constexpr int64_t kByBlocks = 5 << 17;
constexpr int kMaxParts = 1024;  // threads of the workgroup that follows the parts

// Particles a part.  The whole tree in one workgroup saves the launches of the
// nodes that cross parts (29 us instead of 36 at 2000, 35 / 38 at 4000, but 47 / 40
// at 8000); larger parts again once the chip is full (65 / 63 us with 1024 / 2048
// at 3e5, 86 / 76 at 5.2e5, but 41 / 46 at 20000).
constexpr int64_t part_particles(int64_t n)
{
    return kTreeBlock * (n <= 4 * kTreeBlock ? 4 : n <= 1 << 18 ? 1 : 2);
}
static_assert(kByBlocks <= kMaxParts * part_particles(kByBlocks) && 1 << 18 <= kMaxParts * part_particles(1 << 18),
              "a thread for every part");

__device__ inline uint32_t compact3(uint64_t v)
{
    v &= 0x1249249249249249ull;
    v = (v | (v >> 2)) & 0x10C30C30C30C30C3ull;
    v = (v | (v >> 4)) & 0x100F00F00F00F00Full;
    v = (v | (v >> 8)) & 0x001F0000FF0000FFull;
    v = (v | (v >> 16)) & 0x001F00000000FFFFull;
    v = (v | (v >> 32)) & 0x00000000001FFFFFull;
    return (uint32_t)v;
}

__device__ inline void cell_centre(uint64_t key, int level, const Geom* g, double X[3])
{
    uint32_t q[3] = {compact3(key >> 2), compact3(key >> 1), compact3(key)};
    const uint32_t span = 1u << (kMaxLevel - level);
    for (int k = 0; k < 3; ++k) {
        uint32_t corner = q[k] & ~(span - 1u);
        X[k] = g->lo[k] + ((double)corner + 0.5 * (double)span) * g->h;
    }
}

#define MOM_ARGS                                                                                               \
    const uint4 *__restrict__ topo, const uint2 *__restrict__ ends, const uint64_t *__restrict__ skeys,        \
        const Particle *__restrict__ sp, const Geom *__restrict__ g, WalkNode *__restrict__ wn
#define MOM_PASS topo, ends, skeys, sp, g, wn

// Node b, if it ends by limit.  One-particle leaves are complete already (k_emit).
__device__ inline void moments_node(int64_t b, int l, uint32_t limit, const uint4 rec, const uint2 en, MOM_ARGS)
{
    // rec = topo[b] = {first, child, meta}, en = ends[b] = {end, last child}
    if (meta_single(rec.z) || en.x > limit) return;
    const uint32_t f = rec.x, c = en.x - f, child = rec.y;
    const uint32_t nc = meta_leaf(rec.z) ? 0u : en.y - child + 1u;
    double M = 0.0, S0 = 0.0, S1 = 0.0, S2 = 0.0, X[3];
    if (nc == 0) {
        for (uint32_t j = f; j < f + c; ++j) {
            const Particle q = sp[j];
            M += q.m;
            S0 += q.m * q.x;
            S1 += q.m * q.y;
            S2 += q.m * q.z;
        }
    } else {
        // the children's records are asked for together, then summed in octant order
        double2 xy[8], zm[8];
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k) {
            if (k < nc) {
                xy[k] = *reinterpret_cast<const double2*>(&wn[child + k].x);
                zm[k] = *reinterpret_cast<const double2*>(&wn[child + k].z);
            }
        }
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k) {
            if (k < nc) {
                const double mc = zm[k].y;
                M += mc;
                S0 += mc * xy[k].x;
                S1 += mc * xy[k].y;
                S2 += mc * zm[k].x;
            }
        }
    }
    if (M == 0.0) {
        cell_centre(skeys[f], l, g, X);
    } else {
        X[0] = S0 / M;
        X[1] = S1 / M;
        X[2] = S2 / M;
    }
    uint4* o = reinterpret_cast<uint4*>(wn + b);
    o[0] = make_uint4(__double2loint(X[0]), __double2hiint(X[0]), __double2loint(X[1]), __double2hiint(X[1]));
    o[1] = make_uint4(__double2loint(X[2]), __double2hiint(X[2]), __double2loint(M), __double2hiint(M));
    o[2] = make_uint4(f, c, child, rec.z | nc);
}

// The nodes that begin and end within one part of the order: one workgroup,
// level by level.  The links of a level are asked for while the level below is
// summed (100000 particles: 57 us without, 50 with it).
__global__ __launch_bounds__(1024) void k_moments_block(int64_t n, int64_t nb, int64_t part,
                                                        const uint32_t* __restrict__ table, LevelOffsets off, MOM_ARGS)
{
    __shared__ uint32_t lo[kLevels], hi[kLevels];
    const int64_t first = blockIdx.x * part, after = first + part;
    if (threadIdx.x < kLevels) {
        const int l = threadIdx.x;
        const uint32_t* row = table + l * nb;
        lo[l] = off.off[l] + row[first / kTreeBlock];
        hi[l] = after < n ? off.off[l] + row[after / kTreeBlock] : off.off[l + 1];
    }
    __syncthreads();
    const uint32_t limit = (uint32_t)(after < n ? after : n);
    const int lane = threadIdx.x & 63;
    uint32_t levels = (uint32_t)__ballot(lane < kLevels && lo[lane < kLevels ? lane : 0] < hi[lane < kLevels ? lane : 0]);
    if (!levels) return;
    int l = 31 - __clz((int)levels);
    uint32_t b = lo[l] + threadIdx.x, b1 = hi[l];
    const uint4 none = make_uint4(0u, 0u, 1u << 17, 0u);  // passes for a one-particle leaf
    uint4 rec = none;
    uint2 en = make_uint2(0u, 0u);
    if (b < b1) {
        rec = topo[b];
        en = ends[b];
    }
    for (;;) {
        levels &= ~(1u << l);
        const int above = levels ? 31 - __clz((int)levels) : 0;
        const uint32_t a = lo[above] + threadIdx.x, a1 = levels ? hi[above] : 0u;
        uint4 arec = none;
        uint2 aen = make_uint2(0u, 0u);
        if (a < a1) {
            arec = topo[a];
            aen = ends[a];
        }
        moments_node(b, l, limit, rec, en, MOM_PASS);
        for (b += blockDim.x; b < b1; b += blockDim.x) moments_node(b, l, limit, topo[b], ends[b], MOM_PASS);
        if (!levels) break;
        __syncthreads();
        l = above;
        b = a;
        b1 = a1;
        rec = arec;
        en = aen;
    }
}

// The nodes that cross from one part into the next: one workgroup, a thread a
// part, level by level.  Those that begin in a part and cross its end s | s + 1
// are the nodes of s at the levels that s + 1 shares with it and the particle
// before the part does not.
__global__ __launch_bounds__(kMaxParts) void k_moments_cross(int64_t n, int64_t nb, int64_t part,
                                                             const uint32_t* __restrict__ table, LevelOffsets off, MOM_ARGS)
{
    const int64_t first = threadIdx.x * part, after = first + part;
    int above = kMaxLevel, deepest = -1;  // levels above + 1 ... deepest
    if (after < n) {
        const uint64_t key = skeys[after - 1];
        deepest = shared_level(key, skeys[after]);
        above = first > 0 ? shared_level(skeys[first - 1], key) : -1;
    }
    __shared__ uint32_t used;
    if (threadIdx.x == 0) used = 0u;
    __syncthreads();
    if (above < deepest) atomicOr(&used, (2u << deepest) - (1u << (above + 1)));
    __syncthreads();
    uint32_t levels = used;
    const int64_t next = after / kTreeBlock;  // the block that begins where the part ends
    while (levels) {
        const int l = 31 - __clz((int)levels);
        levels &= ~(1u << l);
        if (above < l && l <= deepest) {
            const uint32_t b = off.off[l] + table[l * nb + next] - 1u;
            moments_node(b, l, (uint32_t)n, topo[b], ends[b], MOM_PASS);
        }
        __syncthreads();
    }
}

// One level with many nodes: one thread per node.
__global__ __launch_bounds__(256) void k_moments_level(int l, uint32_t b0, uint32_t b1, MOM_ARGS)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t b = (int64_t)b0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b < (int64_t)b1; b += stride)
        moments_node(b, l, ~0u, topo[b], ends[b], MOM_PASS);
}

// A run of consecutive small levels [llo, lhi], deepest first, in one
// workgroup: a barrier separates the levels (the waves of one workgroup share
// a CU and its L1, so the barrier's workgroup-scope fence makes the finished
// level visible).
__global__ __launch_bounds__(kSmallLevelThreads) void k_moments_small(int lhi, int llo, LevelOffsets off, MOM_ARGS)
{
    for (int l = lhi; l >= llo; --l) {
        for (int64_t b = (int64_t)off.off[l] + threadIdx.x; b < (int64_t)off.off[l + 1]; b += blockDim.x)
            moments_node(b, l, ~0u, topo[b], ends[b], MOM_PASS);
        __syncthreads();
    }
}

void launch_blocks(int64_t n, const uint32_t* table, const LevelOffsets& off, MOM_ARGS, hipStream_t s)
{
    const int64_t nb = (n + kTreeBlock - 1) / kTreeBlock;
    const int64_t part = part_particles(n), parts = (n + part - 1) / part;
    k_moments_block<<<(unsigned)parts, parts == 1 ? 1024 : 512, 0, s>>>(n, nb, part, table, off, MOM_PASS);
    if (parts > 1) k_moments_cross<<<1, (unsigned)((parts + 63) / 64 * 64), 0, s>>>(n, nb, part, table, off, MOM_PASS);
}

void launch_levels(const LevelOffsets& off, MOM_ARGS, hipStream_t s)
{
    int l = kMaxLevel;
    while (l >= 0) {
        if (off.size(l) <= kSmallLevel) {
            int lo = l;
            while (lo > 0 && off.size(lo - 1) <= kSmallLevel) --lo;
            if (off.off[l + 1] > off.off[lo]) k_moments_small<<<1, kSmallLevelThreads, 0, s>>>(l, lo, off, MOM_PASS);
            l = lo - 1;
            continue;
        }
        int64_t blocks = ((int64_t)off.size(l) + 255) / 256;
        if (blocks > 8192) blocks = 8192;
        k_moments_level<<<(unsigned)blocks, 256, 0, s>>>(l, off.off[l], off.off[l + 1], MOM_PASS);
        --l;
    }
}

}  // namespace

void launch_moments(int64_t n, const uint32_t* table, const uint32_t* level_off_host, const uint4* topo, const uint2* ends,
                    const uint64_t* skeys, const Particle* sp, const Geom* g, WalkNode* wn, hipStream_t s)
{
    LevelOffsets off;
    for (int l = 0; l <= kLevels; ++l) off.off[l] = level_off_host[l];
    if (n <= kByBlocks) launch_blocks(n, table, off, MOM_PASS, s);
    else launch_levels(off, MOM_PASS, s);
}

}  // namespace tc
