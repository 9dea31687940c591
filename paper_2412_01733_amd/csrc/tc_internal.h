// Internal definitions shared by the HIP translation units of libtreecode.
// Nothing here is part of the C ABI (include/treecode.h is).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/treecode.h"

namespace tc {

constexpr int kMaxLevel = 21;          // 21 bits per axis, 63-bit keys
constexpr int kLevels = kMaxLevel + 1;  // levels 0..21
constexpr uint32_t kQMax = (1u << 21) - 1;

// Root cube and input checks produced on the device by the bounds pass.
struct Geom {
    double lo[3];
    double L;        // root side, a power of two
    double scale;    // 2^21 / L (exact)
    double h;        // L 2^-21, the finest cell side
    int32_t log2L;
    uint32_t bad;    // bit 0: non-finite position, bit 1: negative / non-finite mass
    uint32_t nnodes; // filled by the build (node count read back to the host)
    uint32_t pad;
};

// One node as the walk reads it.  Nodes are stored in breadth-first order:
// sorted by (level, first), so the root is at 0, every level is contiguous
// and the children of every internal node are consecutive in octant order.
struct __align__(16) WalkNode {
    double x, y, z;   // centre of mass
    double m;         // total mass
    uint32_t first;   // sorted index of the first particle
    uint32_t count;   // particles in the node
    uint32_t child;   // group index of the first child (internal nodes)
    uint32_t meta;    // bits 0-3 nchild, bits 8-12 level, bit 16 leaf, bit 17 one-particle leaf,
                      // bits 18-20 the node's octant in its parent (key digit at its level)
};
static_assert(sizeof(WalkNode) == 48, "WalkNode layout");

// A particle in key order: position and mass, FP64 (one 32-byte record, so
// that a leaf or a target reads one aligned line).
struct __align__(32) Particle {
    double x, y, z, m;
};

// Breadth-first offsets of the levels (level l occupies [off[l], off[l+1])),
// passed by value to the level-batched kernels.  Levels with at most
// kSmallLevel nodes are processed in runs by a single workgroup.
struct LevelOffsets {
    uint32_t off[kLevels + 1];
    __host__ __device__ uint32_t size(int l) const { return off[l + 1] - off[l]; }
};
constexpr int kTreeBlock = 1024;  // particles a column of the tree's table
constexpr uint32_t kSmallLevel = 4096;
constexpr int kSmallLevelThreads = 1024;

__host__ __device__ inline uint32_t meta_nchild(uint32_t m) { return m & 0xFu; }
__host__ __device__ inline uint32_t meta_level(uint32_t m) { return (m >> 8) & 0x1Fu; }
__host__ __device__ inline bool meta_leaf(uint32_t m) { return (m >> 16) & 1u; }
__host__ __device__ inline bool meta_single(uint32_t m) { return (m >> 17) & 1u; }
__host__ __device__ inline uint32_t meta_octant(uint32_t m) { return (m >> 18) & 7u; }
// level + 32 * single (bit 13 repeats the single flag): the walk's threshold table index
__host__ __device__ inline uint32_t meta_tau_index(uint32_t m) { return (m >> 8) & 0x3Fu; }

// Deepest level at which two keys share a cell.
__device__ inline int shared_level(uint64_t a, uint64_t b)
{
    const uint64_t x = a ^ b;
    return x ? (__clzll((long long)x) - 1) / 3 : kMaxLevel;
}

// ---------------------------------------------------------------------------
// launch wrappers (each defined next to its kernels)
// ---------------------------------------------------------------------------

// keys.hip
// (the partials only if geom is null)
void launch_bounds(const void* pos, const void* mass, int64_t n, tc_dtype dt, double* partials,
                   int nblocks, Geom* geom, hipStream_t s);
int bounds_blocks(int64_t n);
// keys also writes the packed {x, y, z, m} record (record_bytes) that the gather reads
size_t record_bytes(int64_t n, tc_dtype dt);
void launch_keys(const void* pos, const void* mass, int64_t n, tc_dtype dt, const Geom* geom, uint64_t* keys,
                 uint32_t* idx, void* rec, hipStream_t s);
void launch_gather(const void* rec, int64_t n, tc_dtype dt, const uint32_t* perm, Particle* sp, hipStream_t s);

// scan.hip: exclusive scan of each row of a [rows, cols] table in place, its total in totals[row]
void launch_scan_rows(uint32_t* table, int rows, int64_t cols, uint32_t* totals, hipStream_t s);

// sort.hip: stable LSD radix sort of (u64 key, u32 value) pairs over the
// low `bits` key bits.  Result ends in (keys_out, vals_out); the *_alt
// buffers are scratch.
size_t radix_temp_bytes(int64_t n);
void radix_sort_pairs(uint64_t* keys, uint32_t* vals, uint64_t* keys_alt, uint32_t* vals_alt,
                      int64_t n, int bits, void* temp, hipStream_t s, uint64_t** keys_out,
                      uint32_t** vals_out);

// sort_small.hip: keys, sort and gather in one (kSortSmall: up to which n it is used).
// part: the bounds' partials (nparts of them; none needed for a lone tile); writes geom.
constexpr int64_t kSortSmall = 1 << 19;
bool sort_small_lone(int64_t n);
void launch_sort_small(const void* pos, const void* mass, int64_t n, tc_dtype dt, const double* part, int nparts,
                       Geom* geom, uint64_t* k0, uint32_t* v0, uint64_t* k1, uint32_t* v1, Particle* sp, hipStream_t s,
                       uint64_t** keys_out, uint32_t** vals_out);

// build.hip: the tree's rows of counts (nodes that begin, by level; leaves; multi-particle
// leaves) per block of particles and in total, then the breadth-first node tables:
// topo {first particle, first child, meta without nchild, 0}, ends {end, last child} (not for
// one-particle leaves), the walk records of one-particle leaves, leaf_of[particle].
constexpr int kTreeRows = kLevels + 2;
size_t tree_table_bytes(int64_t n);
void launch_tree_counts(const uint64_t* skeys, int64_t n, uint32_t* table, uint32_t* totals, hipStream_t s);
void launch_emit(const uint64_t* skeys, int64_t n, const uint32_t* table, const uint32_t* level_off_host, const Particle* sp,
                 uint4* topo, uint2* ends, WalkNode* wn, uint32_t* leaf_of, uint32_t* status, hipStream_t s);
// Canonical export (pre-order); writes to the outputs only, any of which may be null.
void launch_export_nodes(const uint64_t* skeys, int64_t n, const uint32_t* table, const uint32_t* level_off_host,
                         const uint2* ends, const WalkNode* wn, uint8_t* level, uint32_t* first, uint32_t* count,
                         double* com, double* mass, hipStream_t s);

// moments.hip: the upward pass.  table as launch_tree_counts left it.
void launch_moments(int64_t n, const uint32_t* table, const uint32_t* level_off_host, const uint4* topo, const uint2* ends, const uint64_t* skeys,
                    const Particle* sp, const Geom* geom, WalkNode* wn, hipStream_t s);

// walk.hip
struct WalkArgs {
    const WalkNode* nodes;
    const Particle* sp;     // particles in key order
    const uint32_t* order;  // [n] targets: a wavefront (or team) takes 64, 16 or 8 that follow each other
    const uint32_t* perm;
    int64_t n;
    double eps2;
    double G;
    double tau0_64;         // (L / theta)^2, +inf for theta == 0; level l uses tau0 4^-l
    float tau0_32;          // the same rounded to FP32 (scaling by 4^-l stays exact)
    void* acc;              // caller order, FP32 (F32C) or FP64 (F64)
    void* pot;              // may be NULL
    uint32_t* counts;       // sorted order (counting walk only)
    double* diag;           // [wavefronts or teams, 4] partials of sum m a, sum m |a|
    uint32_t* status;       // bit 0: stack overflow (never expected)
    unsigned long long* visits;  // counting walk: [kNumVisitCounters], see tc_stats (node_visits ... max_stack)
    // adjoint walk only
    const void* g_acc;      // dL/da [n,3], caller order, walk precision
    const void* g_pot;      // dL/dphi [n] or NULL
    double* node_grad;      // [nodes, 4] breadth-first: dL/dX (3), dL/dM, accumulated
    double* part_grad;      // [n, 4] sorted order: dL/dx_j (3), dL/dm_j from opened multi-particle leaves; null if there are none
    double* target_grad;    // [n, 3] sorted order: dL/dx_i from the target side
    // stored interaction lists: per wave, in visit order, records {node, kind, lane mask lo, hi};
    // kind 0: the node was accepted by the mask's lanes; kind 1: the multi-particle leaf was
    // opened by them.  Written by a storing forward walk, replayed by the adjoint walk.
    uint4* lists;           // [waves, list_cap], or NULL (adjoint: re-walk)
    uint32_t* list_len;     // [waves]: records of the wave, or kListInvalid if they did not fit
    uint32_t list_cap;      // records per wave
};
// counting walk: node evaluations, active lanes, group pops, evaluations with no
// accepting lane, with every active lane accepting, decided "all open" and "all
// accept" by the per-wave box test, deepest stack (atomic max), steps, steps
// that took a single group, evaluations of nodes whose particle range overlaps
// the wavefront's targets, of those taken by the general path with every
// active lane accepting
constexpr int kNumVisitCounters = 12;
constexpr uint32_t kListCap = 8192;                     // records per wave (128 KiB)
constexpr uint32_t kListInvalid = 0xFFFFFFFFu;
constexpr uint64_t kListMaxBytes = 4ull << 30;          // lists are stored only up to this size
int64_t walk_waves(int64_t n);
// storing walk (with or without counting)
void launch_walk(const WalkArgs& a, tc_walk mode, bool count, hipStream_t s);
// walk_forward.hip: the walk that does not store
void launch_walk_forward(const WalkArgs& a, tc_walk mode, bool count, bool team, hipStream_t s);
// adjoint walk: replays stored lists, or walks for the wavefronts that have none
void launch_walk_adjoint(const WalkArgs& a, tc_walk mode, hipStream_t s);
// walk_adjoint.hip: the adjoint walk where no lists are stored
void launch_walk_adjoint_wide(const WalkArgs& a, tc_walk mode, int team, hipStream_t s);

// walk_direct.hip: the direct sum, for theta = 0 and no multi-particle leaves
bool direct_serves(double theta, int64_t multi_leaves);
void launch_direct(const WalkArgs& a, tc_walk mode, hipStream_t s);

// walk_split.hip: the same walks with 8 or 16 targets a wavefront (the adjoint: 8).
// Targets a wavefront for n particles, and, of 64, whether a team of wavefronts takes them.
int walk_targets(int64_t n, tc_walk mode);
int64_t walk_rows_max(int64_t n);  // diagnostic rows (wavefronts) of any walk of n particles at most
bool walk_team(int64_t n, tc_walk mode);
int adjoint_targets(int64_t n);
int adjoint_team(int64_t n, tc_walk mode);  // wavefronts for 64 targets
void launch_walk_split(const WalkArgs& a, int targets, tc_walk mode, hipStream_t s);
void launch_walk_split_adjoint(const WalkArgs& a, tc_walk mode, hipStream_t s);

// order.hip: the walk's target order (Hilbert order of the particles); also
// up[node] = {distance of the node from its parent's start in the order, parent}.
void launch_target_order(int64_t n, int64_t nn, const uint64_t* skeys, const uint4* topo, const uint2* ends,
                         const uint32_t* leaf_of, uint2* up, uint32_t* order, hipStream_t s);

// adjoint.hip: from node gradients to particle gradients.
void launch_adjoint_down(int64_t nn, int64_t n, const uint4* topo, const WalkNode* wn, const uint2* up,
                         const double* node_grad, double* uc, const uint32_t* leaf_of, const Particle* sp,
                         const uint32_t* perm, const double* target_grad, const double* part_grad, void* g_pos,
                         void* g_mass, bool out_f64, hipStream_t s);
void launch_fill_f64_zero(double* p, int64_t n, hipStream_t s);

// integrate.hip: leapfrog pieces and FP64 step diagnostics
void launch_kick_drift(void* pos, void* vel, const void* acc, int64_t n, tc_dtype dt, bool acc64, double tau,
                       hipStream_t s);
void launch_kick(void* vel, const void* acc, int64_t n, tc_dtype dt, bool acc64, double tau, hipStream_t s);
size_t step_diag_temp_bytes();
// out10: kinetic, potential energy, momentum (3), angular momentum (3), total mass, 0
void launch_step_diag(const void* pos, const void* vel, const void* mass, const void* pot, int64_t n, tc_dtype dt,
                      bool pot64, void* temp, double* out10, hipStream_t s);

// diag.hip
size_t diag_temp_bytes(int64_t nwaves);
void launch_diag_final(const double* part, int64_t nwaves, void* temp, double* out4, hipStream_t s);
void launch_fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t s);
void launch_sum_counts(const uint32_t* counts, int64_t n, unsigned long long* out, hipStream_t s);
void launch_scatter_counts(const uint32_t* sorted_counts, const uint32_t* perm, int64_t n,
                           uint32_t* out, hipStream_t s);

}  // namespace tc
