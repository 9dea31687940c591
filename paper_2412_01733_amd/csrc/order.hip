// The walk's target order: the particles along the Hilbert curve.
//
// The walk gives each wavefront 8, 16 or 64 consecutive targets of this order.  The
// tree, its keys and its node table stay in Morton (key) order; only the
// grouping of targets into wavefronts changes.  A Hilbert segment of 64
// particles is spatially more compact than a Morton segment, which jumps
// between distant cells at the Z-curve's seams, so the targets open fewer
// nodes between them.  No result depends on the order: every target's
// interaction set and terms are its own.
//
// Every octree cell is a contiguous range of the Hilbert order, just as it is
// of the key order: a node's children follow each other in the order of their
// Hilbert digits at their level (siblings share all higher digits), and a leaf
// lays out its particles in key order.  A child's distance from its parent's
// start is the count of its siblings with lower digits; a particle's place is
// the sum of these distances along its path.  The digits depend on the key
// alone, so neither pass goes level by level: one thread per internal node steps
// the state of the curve down the node's key and ranks the children, then one
// thread per particle climbs to the root.  (0.29 ms at 1e7 particles and 55 us at
// 1000, in 13 and 2 launches, when the offsets came down level by level.)
//
// Hilbert digits.  The index is that of the transposition algorithm of
// J. Skilling, "Programming the Hilbert curve", AIP Conf. Proc. 707, 381
// (2004), read out with the first transposed coordinate highest in each
// triple.  That algorithm visits the bit levels top down; at each level it
// reflects or exchanges the lower bits of the coordinates according to the
// current level's bits, and its Gray-code step makes each output digit depend
// on the current level and on the parity of the higher levels only.  The
// reflections and exchanges accumulated above a level therefore form a signed
// permutation of the three axes, which together with that parity is the state
// a cell hands to its children:
//   X_a   = raw bit of axis perm[a], xor flip[a]          (a = 0, 1, 2)
//   digit = (X_0, X_0^X_1, X_0^X_1^X_2), each xor parity  (first bit highest)
//   then, for i = 0, 1, 2 in turn: if X_i, flip[0] ^= 1, else exchange
//   (perm, flip) entries 0 and i; parity ^= X_0^X_1^X_2.
// State word: perm[a] in bits 2a..2a+1, flip[a] in bit 6 + a, parity in bit 9.
#include <cstddef>

#include "tc_internal.h"

namespace tc {
namespace {

constexpr uint32_t kRootState = 0u | (1u << 2) | (2u << 4);  // identity permutation, no flips, even parity

// Hilbert digit of octant d (key digit: x bit 2, y bit 1, z bit 0) under
// state st, and the state the child in that octant inherits.
constexpr uint32_t hilbert_step(uint32_t st, uint32_t d, uint32_t* child_state)
{
    uint32_t perm[3] = {}, flip[3] = {}, X[3] = {};
    for (int a = 0; a < 3; ++a) {
        perm[a] = (st >> (2 * a)) & 3u;
        flip[a] = (st >> (6 + a)) & 1u;
    }
    const uint32_t par = (st >> 9) & 1u;
    for (int a = 0; a < 3; ++a) X[a] = ((d >> (2 - perm[a])) & 1u) ^ flip[a];
    const uint32_t g0 = X[0], g1 = X[0] ^ X[1], g2 = g1 ^ X[2];
    const uint32_t digit = ((g0 ^ par) << 2) | ((g1 ^ par) << 1) | (g2 ^ par);
    for (int i = 0; i < 3; ++i) {
        if (X[i]) {
            flip[0] ^= 1u;
        } else if (i > 0) {
            const uint32_t tp = perm[0], tf = flip[0];
            perm[0] = perm[i];
            flip[0] = flip[i];
            perm[i] = tp;
            flip[i] = tf;
        }
    }
    uint32_t ns = (par ^ g2) << 9;
    for (int a = 0; a < 3; ++a) ns |= (perm[a] << (2 * a)) | (flip[a] << (6 + a));
    *child_state = ns;
    return digit;
}

// The states that can be reached from the root's, numbered as they are found
// (the root is 0), as a table: next[state][octant] and digits[state], 4 bits an
// octant.  A step down the key is one LDS read instead of ~40 instructions.
struct HilbertTable {
    alignas(8) uint8_t next[128][8];
    uint32_t digits[128];
    int count;
};

constexpr HilbertTable make_hilbert_table()
{
    HilbertTable t{};
    uint32_t state[128] = {};
    state[0] = kRootState;
    t.count = 1;
    for (int s = 0; s < t.count; ++s) {
        for (uint32_t d = 0; d < 8; ++d) {
            uint32_t ns = 0;
            t.digits[s] |= hilbert_step(state[s], d, &ns) << (4 * d);
            int f = 0;
            while (f < t.count && state[f] != ns) ++f;
            if (f == t.count) state[t.count++] = ns;
            t.next[s][d] = (uint8_t)f;
        }
    }
    return t;
}

constexpr HilbertTable kHilbertHost = make_hilbert_table();
constexpr int kHilbertStates = kHilbertHost.count;
static_assert(kHilbertStates <= 96, "6 permutations, 8 flips, 2 parities");
__constant__ HilbertTable kHilbert = make_hilbert_table();

// Distances of an internal node's children from its start, with the link up:
// up[child] = {distance, parent}.
__global__ __launch_bounds__(256) void k_order_children(int64_t nn, const uint64_t* __restrict__ skeys,
                                                        const uint4* __restrict__ topo, const uint2* __restrict__ ends,
                                                        uint2* __restrict__ up)
{
    __shared__ uint2 next[kHilbertStates];  // a byte an octant
    __shared__ uint32_t digits[kHilbertStates];
    static_assert(alignof(HilbertTable) % alignof(uint2) == 0 && offsetof(HilbertTable, next) % alignof(uint2) == 0 &&
                      sizeof(kHilbert.next[0]) == sizeof(uint2), "a row is read as a uint2");
    for (int i = threadIdx.x; i < kHilbertStates; i += blockDim.x) {
        next[i] = *reinterpret_cast<const uint2*>(kHilbert.next[i]);
        digits[i] = kHilbert.digits[i];
    }
    __syncthreads();
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nn) return;
    const uint4 rec = topo[b];  // first, child, meta
    if (b == 0) up[0] = make_uint2(0u, 0u);
    if (meta_leaf(rec.z)) return;
    const uint64_t key = skeys[rec.x];
    const uint8_t* step = reinterpret_cast<const uint8_t*>(next);
    uint32_t st = 0;
    for (int l = 1; l <= (int)meta_level(rec.z); ++l)
        st = step[8 * st + ((uint32_t)(key >> (3 * (kMaxLevel - l))) & 7u)];
    const uint32_t dg = digits[st];
    const uint2 en = ends[b];  // end, last child
    const uint32_t nc = en.y - rec.y + 1u < 8u ? en.y - rec.y + 1u : 8u;
    // fixed-size, fully unrolled, so that the arrays stay in registers; an
    // absent child counts 0 and sorts last (digit 8).  Siblings follow each other, so a
    // child ends where the next begins (with the children's own ends read, 260 instead
    // of 217 us at 1e7).
    uint32_t first[9], cnt[8], dig[8];
    first[8] = en.x;
#pragma unroll
    for (int k = 7; k >= 0; --k) {
        first[k] = en.x;
        dig[k] = 8u;
        if ((uint32_t)k < nc) {
            const uint4 c = topo[rec.y + (uint32_t)k];
            first[k] = c.x;
            dig[k] = (dg >> (4 * meta_octant(c.z))) & 7u;
        }
    }
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) cnt[k] = first[k + 1] - first[k];
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) {
        if (k < nc) {
            uint32_t o = 0u;
#pragma unroll
            for (uint32_t j = 0; j < 8; ++j)
                if (dig[j] < dig[k]) o += cnt[j];
            up[rec.y + k] = make_uint2(o, (uint32_t)b);
        }
    }
}

__global__ __launch_bounds__(256) void k_order_place(int64_t n, const uint4* __restrict__ topo,
                                                     const uint32_t* __restrict__ leaf_of, const uint2* __restrict__ up,
                                                     uint32_t* __restrict__ order)
{
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    uint32_t b = leaf_of[s];
    uint32_t o = (uint32_t)s - topo[b].x;
    for (int l = 0; l < kMaxLevel && b != 0u; ++l) {  // at most one step a level
        const uint2 u = up[b];
        o += u.x;
        b = u.y;
    }
    order[o] = (uint32_t)s;
}

}  // namespace

void launch_target_order(int64_t n, int64_t nn, const uint64_t* skeys, const uint4* topo, const uint2* ends,
                         const uint32_t* leaf_of, uint2* up, uint32_t* order, hipStream_t s)
{
    k_order_children<<<(unsigned)((nn + 255) / 256), 256, 0, s>>>(nn, skeys, topo, ends, up);
    k_order_place<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(n, topo, leaf_of, up, order);
}

}  // namespace tc
