// Octree construction from sorted Morton keys.
//
// The tree is the canonical octree of the TreeCode description (section 2):
// a level-l cell (particles sharing the top 3l key bits) is a node iff it is
// the root or its parent cell holds >= 2 particles; cells of one particle and
// level-21 cells are leaves; a cell whose particles all fall in one octant
// keeps its single child (chain node).
//
// With c_s = the deepest level at which keys s and s+1 share a cell
// (c_s = min(21, floor((clz64(k_s ^ k_{s+1}) - 1) / 3)), c_{-1} = c_{n-1} = -1),
// particle s lies in nodes of the levels 0 ... m_s = min(21, max(c_{s-1}, c_s) + 1),
// is the first particle of those of levels c_{s-1} + 1 ... m_s and the last of
// those of levels c_s + 1 ... m_s.
//
// The walk wants siblings contiguous and the upward pass wants each level
// contiguous, so nodes are numbered breadth first: by (level, first).  The
// level-l node that holds s is then number
//   off_l + (level-l nodes whose first particle is <= s) - 1,
// a count that a block gets from ballots, one per level, on top of the counts
// of the blocks before it.  So every particle knows the number of each node that
// begins or ends with it, of its parent and of its child there, and writes
// them down: no sort by level, no search for a node's end, no links to follow.
// (At 1e7 particles the tree and the upward pass took 1.92 ms with a radix pass
// over the levels, a galloping search per node and gathers through the pre-order
// numbers; see moments.hip for the present figures.)
#include "tc_internal.h"
#include "walk_common.h"

namespace tc {
namespace {

constexpr int kTreeThreads = kTreeBlock;  // a particle each
constexpr int kTreeWaves = kTreeThreads / 64;

inline unsigned grid_for(int64_t n, int threads) { return (unsigned)((n + threads - 1) / threads); }

LevelOffsets level_offsets(const uint32_t* host)
{
    LevelOffsets off;
    for (int l = 0; l <= kLevels; ++l) off.off[l] = host[l];
    return off;
}

// c_{s-1}, c_s and m_s of particle s, and its key.
struct Span {
    int before, after, deepest;
    uint64_t key;
};

__device__ inline Span particle_span(const uint64_t* __restrict__ k, int64_t n, int64_t s)
{
    Span r;
    r.key = k[s];
    r.before = s > 0 ? shared_level(k[s - 1], r.key) : -1;
    r.after = s + 1 < n ? shared_level(r.key, k[s + 1]) : -1;
    const int m = (r.before > r.after ? r.before : r.after) + 1;
    r.deepest = m < kMaxLevel ? m : kMaxLevel;
    return r;
}

// Per block: nodes that begin in it, by level (rows 0..21 of the table), leaves
// (22) and multi-particle leaves (23; the leaf that begins at s holds several
// particles iff it sits at level 21 and s + 1 shares it).  A lone block's counts
// are the totals.
__global__ __launch_bounds__(kTreeThreads) void k_tree_counts(const uint64_t* __restrict__ k, int64_t n,
                                                              uint32_t* __restrict__ table, uint32_t* __restrict__ totals)
{
    __shared__ uint32_t h[kTreeWaves][kTreeRows];
    const int64_t s = (int64_t)blockIdx.x * kTreeThreads + threadIdx.x;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    Span sp = {kMaxLevel, -1, 0, 0};  // begins nothing
    if (s < n) sp = particle_span(k, n, s);
    uint32_t acc = 0;  // lane l keeps row l
    for (int l = 0; l < kLevels; ++l) {
        const uint32_t b = (uint32_t)__popcll(__ballot(sp.before < l && l <= sp.deepest));
        if (lane == l) acc = b;
    }
    const bool leaf = sp.before < sp.deepest;
    const uint32_t bl = (uint32_t)__popcll(__ballot(leaf));
    const uint32_t bm = (uint32_t)__popcll(__ballot(leaf && sp.after == kMaxLevel));
    if (lane == kLevels) acc = bl;
    if (lane == kLevels + 1) acc = bm;
    if (lane < kTreeRows) h[w][lane] = acc;
    __syncthreads();
    if (threadIdx.x < kTreeRows) {
        uint32_t t = 0;
        for (int u = 0; u < kTreeWaves; ++u) t += h[u][threadIdx.x];
        if (gridDim.x == 1) {
            totals[threadIdx.x] = t;
            t = 0;
        }
        table[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = t;
    }
}

// Of the block's particles by wavefront and level.
struct BlockNodes {
    uint64_t begins[kTreeWaves][kLevels];  // lanes whose particle begins a level-l node
    uint32_t before[kTreeWaves][kLevels];  // number of the next level-l node at the wavefront's start
};

// Fills them in, and the span of this thread's particle s (none if s >= n).
__device__ inline Span number_nodes(const uint64_t* __restrict__ k, int64_t n, const uint32_t* __restrict__ table,
                                    const LevelOffsets& off, int64_t s, BlockNodes& nodes)
{
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    Span span = {kMaxLevel, -1, 0, 0};
    if (s < n) span = particle_span(k, n, s);
    uint64_t mine = 0;
    for (int l = 0; l < kLevels; ++l) {
        const uint64_t b = __ballot(span.before < l && l <= span.deepest);
        if (lane == l) mine = b;
    }
    if (lane < kLevels) nodes.begins[w][lane] = mine;
    __syncthreads();
    if (threadIdx.x < kLevels) {
        const int l = threadIdx.x;
        uint32_t t = off.off[l] + table[(int64_t)l * gridDim.x + blockIdx.x];
        for (int u = 0; u < kTreeWaves; ++u) {
            nodes.before[u][l] = t;
            t += (uint32_t)__popcll(nodes.begins[u][l]);
        }
    }
    __syncthreads();
    return span;
}

// Number of the level-l node that holds the particle of this lane.
__device__ inline uint32_t node_number(const BlockNodes& nodes, int w, int lane, int l)
{
    const uint64_t upto = lane == 63 ? ~0ull : (2ull << lane) - 1ull;
    return nodes.before[w][l] + (uint32_t)__popcll(nodes.begins[w][l] & upto) - 1u;
}

// Writes down the nodes (see above).  topo[b] = {first particle, first child,
// meta, 0} comes from the node's first particle, ends[b] = {end, last child} from
// its last one (not for one-particle leaves, whose walk record is complete here);
// leaf_of[s] is the leaf that holds s.
// Bound by HBM: 8 + 32 bytes read, 4 + 48 written a particle, 24 a node.
__global__ __launch_bounds__(kTreeThreads) void k_emit(const uint64_t* __restrict__ k, int64_t n,
                                                       const uint32_t* __restrict__ table, LevelOffsets off,
                                                       const Particle* __restrict__ sp, uint4* __restrict__ topo,
                                                       uint2* __restrict__ ends, WalkNode* __restrict__ wn,
                                                       uint32_t* __restrict__ leaf_of, uint32_t* __restrict__ status)
{
    __shared__ BlockNodes nodes;
    const int64_t s = (int64_t)blockIdx.x * kTreeThreads + threadIdx.x;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (s == 0) *status = 0u;  // a build clears the walks' status word
    const Span span = number_nodes(k, n, table, off, s, nodes);
    if (s >= n) return;
    auto number = [&](int l) { return node_number(nodes, w, lane, l); };
    const int lowest = (span.before < span.after ? span.before : span.after) + 1;
    uint32_t below = 0;  // number of the node one level down
    for (int l = span.deepest; l >= lowest; --l) {
        const uint32_t b = number(l);
        const bool leaf = l == span.deepest;
        if (leaf) leaf_of[s] = b;
        const bool single = leaf && span.before < l && span.after < l;
        if (span.before < l) {
            const uint32_t oct = l > 0 ? (uint32_t)((span.key >> (3 * (kMaxLevel - l))) & 7u) : 0u;
            const uint32_t meta = ((uint32_t)l << 8) | (single ? (1u << 13) | (1u << 17) : 0u) | (leaf ? 1u << 16 : 0u) | (oct << 18);
            topo[b] = make_uint4((uint32_t)s, leaf ? 0u : below, meta, 0u);
            if (single) {
                const double2* p = reinterpret_cast<const double2*>(sp + s);
                double2* o = reinterpret_cast<double2*>(wn + b);
                o[0] = p[0];
                o[1] = p[1];
                reinterpret_cast<uint4*>(wn + b)[2] = make_uint4((uint32_t)s, 1u, 0u, meta);
            }
        }
        if (span.after < l && !single) ends[b] = make_uint2((uint32_t)s + 1u, leaf ? 0u : below);
        below = b;
    }
    if (lowest > span.deepest) leaf_of[s] = number(span.deepest);  // inside a leaf of coincident keys
}

// The canonical export: the nodes in pre-order, i.e. by (first, level).  The nodes
// that begin at one particle follow each other there, after as many as begin before
// it at any level.  Reads the handle's tables only.
__global__ __launch_bounds__(kTreeThreads) void k_export_nodes(const uint64_t* __restrict__ k, int64_t n,
                                                               const uint32_t* __restrict__ table, LevelOffsets off,
                                                               const uint2* __restrict__ ends, const WalkNode* __restrict__ wn,
                                                               uint8_t* __restrict__ level, uint32_t* __restrict__ first,
                                                               uint32_t* __restrict__ count, double* __restrict__ com,
                                                               double* __restrict__ mass)
{
    __shared__ BlockNodes nodes;
    const int64_t s = (int64_t)blockIdx.x * kTreeThreads + threadIdx.x;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const Span span = number_nodes(k, n, table, off, s, nodes);
    if (s >= n) return;
    const uint64_t below = (1ull << lane) - 1ull;
    uint32_t pre = 0;
    for (int l = 0; l < kLevels; ++l) pre += nodes.before[w][l] - off.off[l] + (uint32_t)__popcll(nodes.begins[w][l] & below);
    for (int l = span.before + 1; l <= span.deepest; ++l) {
        const uint32_t b = node_number(nodes, w, lane, l);
        const int64_t p = (int64_t)pre + (l - span.before - 1);
        if (level) level[p] = (uint8_t)l;
        if (first) first[p] = (uint32_t)s;
        if (count) count[p] = l == span.deepest && span.after < l ? 1u : ends[b].x - (uint32_t)s;  // 1: a one-particle leaf
        if (com) {
            com[3 * p + 0] = wn[b].x;
            com[3 * p + 1] = wn[b].y;
            com[3 * p + 2] = wn[b].z;
        }
        if (mass) mass[p] = wn[b].m;
    }
}

}  // namespace

size_t tree_table_bytes(int64_t n) { return (size_t)grid_for(n, kTreeThreads) * kTreeRows * sizeof(uint32_t); }

void launch_tree_counts(const uint64_t* skeys, int64_t n, uint32_t* table, uint32_t* totals, hipStream_t s)
{
    const unsigned nb = grid_for(n, kTreeThreads);
    k_tree_counts<<<nb, kTreeThreads, 0, s>>>(skeys, n, table, totals);
    if (nb > 1) launch_scan_rows(table, kTreeRows, nb, totals, s);
}

void launch_emit(const uint64_t* skeys, int64_t n, const uint32_t* table, const uint32_t* level_off_host, const Particle* sp,
                 uint4* topo, uint2* ends, WalkNode* wn, uint32_t* leaf_of, uint32_t* status, hipStream_t s)
{
    k_emit<<<grid_for(n, kTreeThreads), kTreeThreads, 0, s>>>(skeys, n, table, level_offsets(level_off_host), sp, topo, ends, wn,
                                                              leaf_of, status);
}

void launch_export_nodes(const uint64_t* skeys, int64_t n, const uint32_t* table, const uint32_t* level_off_host,
                         const uint2* ends, const WalkNode* wn, uint8_t* level, uint32_t* first, uint32_t* count,
                         double* com, double* mass, hipStream_t s)
{
    k_export_nodes<<<grid_for(n, kTreeThreads), kTreeThreads, 0, s>>>(skeys, n, table, level_offsets(level_off_host), ends, wn,
                                                                      level, first, count, com, mass);
}

}  // namespace tc
