// Upward pass: monopole moments of every node (TreeCode description of
// section 2: a distant cell acts as its total mass at its centre of mass).
//
// Level by level, deepest first, over that level's contiguous range of the
// breadth-first node array, so a parent reads finished children, which are
// consecutive records: one launch per populous level, one single-workgroup
// launch per run of small levels.
// The small runs are bound by a few dependent reads a level (a third less with
// the children's records asked for together: 27 -> 16 us a run at 16384), the
// populous levels by HBM (39 us a level at 1e7).
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

// Node b.  One-particle leaves are complete already (k_emit).
__device__ inline void moments_node(int64_t b, int l, const uint4* __restrict__ topo, const uint2* __restrict__ ends,
                                    const uint64_t* __restrict__ skeys, const Particle* __restrict__ sp,
                                    const Geom* __restrict__ g, WalkNode* __restrict__ wn)
{
    const uint4 rec = topo[b];  // first, child, meta
    if (meta_single(rec.z)) return;
    const uint2 en = ends[b];   // end, last child
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

#define MOM_ARGS                                                                                               \
    const uint4 *__restrict__ topo, const uint2 *__restrict__ ends, const uint64_t *__restrict__ skeys,        \
        const Particle *__restrict__ sp, const Geom *__restrict__ g, WalkNode *__restrict__ wn
#define MOM_PASS topo, ends, skeys, sp, g, wn

// One level with many nodes: one thread per node.
__global__ __launch_bounds__(256) void k_moments_level(int l, uint32_t b0, uint32_t b1, MOM_ARGS)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t b = (int64_t)b0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b < (int64_t)b1; b += stride)
        moments_node(b, l, MOM_PASS);
}

// A run of consecutive small levels [llo, lhi], deepest first, in one
// workgroup: a barrier separates the levels (the waves of one workgroup share
// a CU and its L1, so the barrier's workgroup-scope fence makes the finished
// level visible).
__global__ __launch_bounds__(kSmallLevelThreads) void k_moments_small(int lhi, int llo, LevelOffsets off, MOM_ARGS)
{
    for (int l = lhi; l >= llo; --l) {
        for (int64_t b = (int64_t)off.off[l] + threadIdx.x; b < (int64_t)off.off[l + 1]; b += blockDim.x)
            moments_node(b, l, MOM_PASS);
        __syncthreads();
    }
}

}  // namespace

void launch_moments(const uint32_t* level_off_host, const uint4* topo, const uint2* ends, const uint64_t* skeys,
                    const Particle* sp, const Geom* g, WalkNode* wn, hipStream_t s)
{
    LevelOffsets off;
    for (int l = 0; l <= kLevels; ++l) off.off[l] = level_off_host[l];
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

}  // namespace tc
