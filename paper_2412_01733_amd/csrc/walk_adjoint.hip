// The adjoint walk for many particles (tc_forces_backward without stored lists).
//
// The traversal is that of walk_forward.hip: 64 targets a wavefront, the same
// decisions bit for bit, several sibling groups a step, sparse groups transposed,
// opened children pushed at once.  Every accepted term is differentiated, the
// tree membership and the interaction sets held fixed: the target side goes to
// registers, the source side (dL/dX, dL/dM of the node) is summed over the
// wavefront and added to the node's gradient with one FP64 atomic per component.
//
// The sum over 64 lanes of 4 values a node: two nodes' values swap halves of the
// wavefront (v_permlane32_swap) and are added, so that 32 partial sums of each
// wait in LDS; every second pair, each lane adds 8 of one (node, component) and
// DPP moves finish: ~8 vector instructions and 2 LDS instructions a node.  A
// transposed group's 8 children are reduced together in the same buffer, and
// their 32 components leave in one atomic instruction.
#include <type_traits>

#include "walk_common.h"

namespace tc {
namespace {

constexpr int kAdjWaves = 4;
constexpr int block_waves(int team) { return team > 1 ? team : kAdjWaves; }  // a team is a block
constexpr uint32_t kXcdRun = 64;  // consecutive blocks one XCD takes at a time

// A team: see walk_forward.hip; its wavefronts are the block, 4, 8 or 16 of them.
constexpr int kTeamStack = 400;

// groups a step, stack entries (the bound of walk_forward.hip), wavefronts per SIMD
template <bool F64> struct AdjShape {
    static constexpr int groups = 8;
    static constexpr int stack = F64 ? 142 : 160;
    static constexpr int waves = F64 ? 4 : 6;
    static constexpr uint32_t min_children = F64 ? 0 : 1;
    static_assert(stack >= 142, "the root's children must be safe");
};

template <bool F64, int TEAM>
__global__ __launch_bounds__(64 * block_waves(TEAM)) __attribute__((amdgpu_waves_per_eu(AdjShape<F64>::waves)))
void k_walk_adj(WalkArgs a)
{
    using R = typename std::conditional<F64, double, float>::type;
    using Shape = AdjShape<F64>;
    constexpr int kGroups = Shape::groups, kStack = TEAM > 1 ? kTeamStack : Shape::stack, kSlots = 64;
    constexpr int kWaves = block_waves(TEAM), kStacks = TEAM > 1 ? 1 : kWaves;
    struct __align__(16) Pos { R x, y, z, m; };
    struct __align__(16) Aux { R tau; uint32_t first, count; };  // opening threshold (-1: a one-particle leaf), particle range
    struct __align__(16) Tgt { R x, y, z, gx, gy, gz, h, pad; };
    __shared__ uint64_t stk_m[kStacks][kStack];  // lanes that opened the parent
    __shared__ uint32_t stk_gs[kStacks][kStack]; // first node
    __shared__ uint8_t stk_b[kStacks][kStack];   // child count - 1 | level of the nodes << 3
    // staged children: slot 8 j + k holds child k of group j; after the walk a team's totals
    constexpr int kTotals = 3;
    struct __align__(16) Stage { Pos pos[kSlots]; Aux aux[kSlots]; };
    __shared__ union { Stage st[kWaves]; double total[TEAM][kTotals][64]; } stage;
    __shared__ Tgt tgt[kWaves][8];          // a sparse group's targets
    // source-side values of two pairs of nodes: row p holds, by component, the lanes' halves of
    // the pair's first node (0-31) and of its second (32-63), each already summed over lanes l, l + 32
    __shared__ __align__(16) R sval[kWaves][2][4][64];
    __shared__ uint32_t pushes[2][TEAM];
    R tau0;
    if constexpr (F64) tau0 = a.tau0_64;
    else tau0 = a.tau0_32;

    // FP64: the wave index made uniform keeps the per-wave LDS slices in scalar registers
    const int w = F64 ? uni((int)(threadIdx.x >> 6)) : (int)(threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63;
    const int sw = TEAM > 1 ? 0 : w;  // whose stack
    // Workgroups are dealt to the 8 XCDs round-robin.  Dealing runs of
    // kXcdRun consecutive blocks instead (a bijection on whole rounds of 8
    // runs, the identity on the tail) keeps each XCD's L2 on compact regions
    // of space: the walk's HBM traffic falls ~2.3x at the same speed.
    const uint32_t nb = gridDim.x, b = blockIdx.x, full = nb / (8 * kXcdRun) * (8 * kXcdRun);
    const uint32_t i8 = b >> 3;
    const uint32_t lb = b < full ? ((i8 / kXcdRun) * 8 + (b & 7u)) * kXcdRun + i8 % kXcdRun : b;
    const int64_t wave_id = TEAM > 1 ? (int64_t)lb : (int64_t)lb * kWaves + w;  // 64 targets
    const int64_t base = wave_id * 64;
    if (base >= a.n) return;  // the whole wave; of a team, the whole block
    // this lane's target (sorted position) and the range of sorted positions the
    // wavefront's targets span (a superset of them: only a node overlapping it
    // can hold one of the targets)
    const bool valid = base + lane < a.n;
    const uint32_t first_t = uni(a.order[base]);
    const uint32_t su = valid ? a.order[base + lane] : first_t;
    const Particle anchor = a.sp[first_t];
    const double Ax = anchor.x, Ay = anchor.y, Az = anchor.z;
    const Particle self = a.sp[su];
    R px, py, pz;
    if constexpr (F64) {
        px = self.x; py = self.y; pz = self.z;
    } else {
        px = (float)(self.x - Ax); py = (float)(self.y - Ay); pz = (float)(self.z - Az);
    }
    const R eps2 = (R)a.eps2;
    // The bounding box [bn, bx] of the wavefront's targets (the same offsets the
    // lanes use; idle lanes repeat the first target).  Rounding is monotone, so
    // for a node at X every lane's |fl(X - p)| lies between the box's fl-gap and
    // its fl-far side per axis, and the lane's d^2 (the same fused operations)
    // between the box's two d^2: a node whose near d^2 exceeds the threshold is
    // far from every lane, one whose far d^2 does not is near to every lane, with
    // no margin needed.
    uint32_t smin = su, smax = su;
    R bnx = px, bny = py, bnz = pz, bxx = px, bxy = py, bxz = pz;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        smin = min(smin, (uint32_t)__shfl_xor((int)smin, o, 64));
        smax = max(smax, (uint32_t)__shfl_xor((int)smax, o, 64));
        bnx = fmin(bnx, __shfl_xor(bnx, o, 64)); bny = fmin(bny, __shfl_xor(bny, o, 64));
        bnz = fmin(bnz, __shfl_xor(bnz, o, 64)); bxx = fmax(bxx, __shfl_xor(bxx, o, 64));
        bxy = fmax(bxy, __shfl_xor(bxy, o, 64)); bxz = fmax(bxz, __shfl_xor(bxz, o, 64));
    }
    const uint32_t wave_lo = uni(smin), wave_end = uni(smax) + 1u;
    bnx = uni_r(bnx); bny = uni_r(bny); bnz = uni_r(bnz);
    bxx = uni_r(bxx); bxy = uni_r(bxy); bxz = uni_r(bxz);

    // running totals: F32C keeps (sum, compensation) pairs fed by plain partial sums
    R tx = 0, ty = 0, tz = 0;
    float cx = 0.f, cy = 0.f, cz = 0.f;
    R bx = 0, by = 0, bz = 0;

    // adjoint: G dL/da and G dL/dphi of this lane's target (no term multiplies by G)
    R gxl = 0, gyl = 0, gzl = 0, hl = 0;
    if (valid) {
        const R Gc = (R)a.G;
        const uint32_t i = a.perm[su];
        const R* ga = (const R*)a.g_acc;
        gxl = Gc * ga[3 * (int64_t)i + 0];
        gyl = Gc * ga[3 * (int64_t)i + 1];
        gzl = Gc * ga[3 * (int64_t)i + 2];
        if (a.g_pot) hl = Gc * ((const R*)a.g_pot)[i];
    }
    int sp = 0;
    const uint32_t rmeta = uni(a.nodes[0].meta);
    if (!meta_leaf(rmeta)) {
        const uint64_t vmask = __ballot(valid);
        if (lane == 0 && w == sw) {
            stk_m[sw][0] = vmask;
            stk_gs[sw][0] = uni(a.nodes[0].child);
            stk_b[sw][0] = (uint8_t)((meta_nchild(rmeta) - 1u) | (1u << 3));
        }
        sp = 1;
    }
    team_sync<TEAM>();

    const uint32_t gj = lane >> 3, gk = lane & 7;
    int npair = 0;
    uint32_t pend = 0;                   // staging lanes of the waiting nodes, a byte each (bit 7: none)
    bool have = false;                   // a node that waits for its pair
    uint32_t hslot = 0;
    R hx = 0, hy = 0, hz = 0, hm = 0;
    // add the waiting pairs' sums to node_grad: 16 lanes a node, of them 4 a component, each adding
    // 8 values; node_v: the staged children's numbers by lane
    auto src_flush = [&](const uint32_t node_v) {
        wave_sync();
        constexpr uint32_t kChunk = 16 / sizeof(R), kChunks = 8 / kChunk;
        const uint32_t nd = lane >> 4, c = (lane >> 2) & 3u, part = lane & 3u;
        const uint32_t from = pend >> (8 * nd);
        const uint32_t to = lane_pull_u(node_v, from & 63u);
        const R* row = &sval[w][nd >> 1][c][32 * (nd & 1u) + 8 * part];
        R t = 0;
#pragma unroll
        for (uint32_t i = 0; i < kChunks; ++i) {
            // 16-byte chunks, started at a different one by neighbouring groups of lanes (LDS banks)
            const R* p = row + kChunk * ((i + (lane >> 3)) % kChunks);
            if constexpr (F64) {
                const double2 v = *reinterpret_cast<const double2*>(p);
                t += v.x + v.y;
            } else {
                const float4 v = *reinterpret_cast<const float4*>(p);
                t += (v.x + v.y) + (v.z + v.w);
            }
        }
        t = part_sum<4>(t);
        if (part == 0 && !(from & 0x80u)) unsafeAtomicAdd(a.node_grad + 4 * (int64_t)to + c, (double)t);
        wave_sync();
        npair = 0;
    };
    auto src_put2 = [&](const uint32_t s0, const uint32_t s1, const uint32_t node_v, R x0, R y0, R z0, R m0, R x1, R y1, R z1, R m1) {
        half_swap(x0, x1); half_swap(y0, y1); half_swap(z0, z1); half_swap(m0, m1);
        R(*row)[64] = sval[w][npair];
        row[0][lane] = x0 + x1;
        row[1][lane] = y0 + y1;
        row[2][lane] = z0 + z1;
        row[3][lane] = m0 + m1;
        const uint32_t two = s0 | (s1 << 8);
        if (npair == 0) {
            pend = two | 0x80800000u;
            npair = 1;
        } else {
            pend = (pend & 0xFFFFu) | (two << 16);
            src_flush(node_v);
        }
    };
    auto src_put = [&](const uint32_t slot, const uint32_t node_v, const R sx, const R sy, const R sz, const R sm) {
        if (have) {
            have = false;
            src_put2(hslot, slot, node_v, hx, hy, hz, hm, sx, sy, sz, sm);
        } else {
            have = true;
            hslot = slot;
            hx = sx; hy = sy; hz = sz; hm = sm;
        }
    };
    int since_fold = 0;
    // F32C: at most 32 terms per lane, and the particles of opened leaves, go into the plain partial sums (median error of dL/dx
    // against FP64 at 1e6: 1.49e-7 with up to 128, 1.32e-7 with 32; 1 % of the walk's time at 1e7)
    auto fold = [&]() {
        since_fold = 0;
        if constexpr (F64) {
            tx += bx; ty += by; tz += bz;
        } else {
            kahan_add(tx, cx, bx);
            kahan_add(ty, cy, by);
            kahan_add(tz, cz, bz);
        }
        bx = 0; by = 0; bz = 0;
    };
    bool stack_over = false;
    uint32_t most = 0;  // children of a staged node at most (more than 8: a corrupt tree)
    int turn = 0;
    while (sp > 0) {
        // take the groups that the stack bound allows off the top; lanes 8 j .. 8 j + 7 stage
        // group j.  Idle lanes do the same work on the bottom entry and node 0, and are
        // masked out of the ballots: no divergence, so the ballots read the compares.
        int ng, q, j0;  // groups the step takes, of them at most q by this wave, from the j0-th off the top
        if constexpr (TEAM == 1) {
            q = kGroups;
            j0 = 0;
        } else {
            const uint32_t lb_ = stk_b[0][max(sp - 1 - (int)lane, 0)];
            const uint64_t okm = __ballot((int)lane < min(sp, TEAM * kGroups)) &
                                 __ballot(sp + 7 * ((int)lane + 1) + 7 * (20 - (int)(lb_ >> 3)) + 1 <= kStack);
            ng = uni(~okm ? (int)__builtin_ctzll(~okm) : 64);
            q = (ng + TEAM - 1) / TEAM;
            j0 = uni(w * q);
        }
        const int at = max(sp - 1 - j0 - (int)gj, 0);
        const uint32_t gs = stk_gs[sw][at], gb = stk_b[sw][at];
        uint32_t om_lo, om_hi;  // the group's mask, later the child's opening lanes
        {
            const uint64_t m = stk_m[sw][at];
            om_lo = (uint32_t)m;
            om_hi = (uint32_t)(m >> 32);
        }
        if constexpr (TEAM == 1) {
            const uint64_t okm = __ballot((int)gj < min(sp, kGroups)) &
                                 __ballot(sp + 7 * ((int)gj + 1) + 7 * (20 - (int)(gb >> 3)) + 1 <= kStack);
            ng = uni(~okm ? (int)(__builtin_ctzll(~okm) >> 3) : 8);
        }
        const int mine = TEAM == 1 ? ng : max(0, min(q, ng - j0));
        sp = uni(sp - ng);
        const bool live = (int)gj < mine && gk <= (gb & 7u);
        const uint64_t live_m = __ballot(live);
        const WalkNode nd = a.nodes[live ? gs + gk : 0u];
        Pos h;
        if constexpr (F64) {
            h.x = nd.x; h.y = nd.y; h.z = nd.z; h.m = nd.m;
        } else {
            h.x = (float)(nd.x - Ax); h.y = (float)(nd.y - Ay); h.z = (float)(nd.z - Az);
            h.m = (float)nd.m;
        }
        const uint32_t child = nd.child, meta = nd.meta, node = gs + gk;
        most = max(most, meta & 15u);
        // opening threshold tau0 4^-l (an exact power-of-two scaling); a
        // one-particle leaf is always taken (-1)
        const R tau = meta_single(meta) ? (R)-1 : (R)ldexp(tau0, -2 * (int)meta_level(meta));
        stage.st[w].pos[lane] = h;
        stage.st[w].aux[lane] = Aux{tau, nd.first, nd.count};
        const R gx = fmax(fmax(bnx - h.x, h.x - bxx), (R)0), fx = fmax(fabs(h.x - bnx), fabs(h.x - bxx));
        const R gy = fmax(fmax(bny - h.y, h.y - bxy), (R)0), fy = fmax(fabs(h.y - bny), fabs(h.y - bxy));
        const R gz = fmax(fmax(bnz - h.z, h.z - bxz), (R)0), fz = fmax(fabs(h.z - bnz), fabs(h.z - bxz));
        // may it hold one of the targets?  decided for all of them: far, near
        const uint64_t ovl_m = __ballot(nd.first < wave_end) & __ballot(nd.first + nd.count > wave_lo) & live_m;
        const uint64_t far_m = __ballot(fma(gx, gx, fma(gy, gy, gz * gz)) > tau) & live_m & ~ovl_m;
        const uint64_t near_m = live_m & ~far_m & ~__ballot(fma(fx, fx, fma(fy, fy, fz * fz)) > tau);
        const uint64_t mixed_m = live_m & ~far_m & ~near_m;
        uint64_t open_m = near_m;  // children opened by some lane
        wave_sync();

        for (int j = 0; j < mine; ++j) {
            if (!F64 && j == kGroups / 2) fold();
            const uint64_t mask = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)om_lo, 8 * j) |
                                  ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)om_hi, 8 * j) << 32);
            uint32_t fast = (uint32_t)(far_m >> (8 * j)) & 0xFFu;
            uint32_t mixed = (uint32_t)(mixed_m >> (8 * j)) & 0xFFu;
            const Pos* g8 = &stage.st[w].pos[8 * j];
            const Aux* x8 = &stage.st[w].aux[8 * j];
            uint32_t pc = (uint32_t)__popcll(mask);
            asm("" : "+s"(pc));  // keeps comparisons of it on the scalar unit, in 32 bits
            if (pc <= 8u && (uint32_t)__popc(fast) > Shape::min_children) {
                // transposed: lane 8 r + k takes target r of the mask and child k; the sums over
                // the children go back to the target's lane
                const bool in = __builtin_amdgcn_inverse_ballot_w64(mask);
                const uint32_t r = popc_below(mask);
                if (in) tgt[w][r] = Tgt{px, py, pz, gxl, gyl, gzl, hl, (R)0};
                wave_sync();
                const uint32_t rows = fast * 0x01010101u;
                const uint64_t on = (((uint64_t)rows << 32) | rows) & (pc >= 8u ? ~0ull : (1ull << (8 * pc)) - 1ull);
                R vx = 0, vy = 0, vz = 0, vm = 0;
                if (__builtin_amdgcn_inverse_ballot_w64(on)) {
                    const Tgt q = tgt[w][lane >> 3];
                    const Pos h = g8[lane & 7];
                    const R dx = h.x - q.x, dy = h.y - q.y, dz = h.z - q.z;
                    adj_term(dx, dy, dz, (R)fma(dx, dx, fma(dy, dy, fma(dz, dz, eps2))), h.m, q.gx, q.gy, q.gz, q.h, vx, vy, vz, vm);
                }
                // source side: lane (4 k + c) 2 + half adds 4 of the 8 targets' values of child k,
                // component c (row 1 of the buffer is free between puts)
                R(*row)[64] = sval[w][1];
                row[0][lane] = vx; row[1][lane] = vy; row[2][lane] = vz; row[3][lane] = vm;
                // target side: the sums over the children go back to the target's lane
                vx = slot_sum<8>(vx); vy = slot_sum<8>(vy); vz = slot_sum<8>(vz);
                vx = lane_pull(vx, 8 * r); vy = lane_pull(vy, 8 * r); vz = lane_pull(vz, 8 * r);
                if (in) {
                    bx -= vx; by -= vy; bz -= vz;
                }
                wave_sync();
                const uint32_t k = lane >> 3, c = (lane >> 1) & 3u;
                const uint32_t to = lane_pull_u(node, 8u * (uint32_t)j + k);
                const R* p = &row[c][32 * (lane & 1) + k];
                const R t = part_sum<2>((p[0] + p[8]) + (p[16] + p[24]));
                if ((lane & 1) == 0 && ((fast >> k) & 1u)) unsafeAtomicAdd(a.node_grad + 4 * (int64_t)to + c, (double)t);
                wave_sync();
                fast = 0u;
            }
            // accepted children, no opening test, in pairs
            auto accepted = [&](const uint32_t k, R& sx, R& sy, R& sz, R& sm) {
                const Pos h = g8[k];
                sx = sy = sz = sm = 0;
                if (__builtin_amdgcn_inverse_ballot_w64(mask)) {
                    const R dx = h.x - px, dy = h.y - py, dz = h.z - pz;
                    adj_term(dx, dy, dz, (R)fma(dx, dx, fma(dy, dy, fma(dz, dz, eps2))), h.m, gxl, gyl, gzl, hl, sx, sy, sz, sm);
                    bx -= sx;
                    by -= sy;
                    bz -= sz;
                }
            };
            while (fast) {
                const uint32_t k0 = __builtin_ctz(fast);
                fast &= fast - 1u;
                R x0, y0, z0, m0;
                accepted(k0, x0, y0, z0, m0);
                if (fast) {
                    const uint32_t k1 = __builtin_ctz(fast);
                    fast &= fast - 1u;
                    R x1, y1, z1, m1;
                    accepted(k1, x1, y1, z1, m1);
                    src_put2(8u * (uint32_t)j + k0, 8u * (uint32_t)j + k1, node, x0, y0, z0, m0, x1, y1, z1, m1);
                } else {
                    src_put(8u * (uint32_t)j + k0, node, x0, y0, z0, m0);
                }
            }
            // undecided children: per-lane opening test, containment where the child may hold a target
            while (mixed) {
                const uint32_t k = __builtin_ctz(mixed);
                mixed &= mixed - 1u;
                const uint32_t slot = 8u * (uint32_t)j + k;
                const Pos h = g8[k];
                const Aux x = x8[k];
                const R dx = h.x - px, dy = h.y - py, dz = h.z - pz;
                const R d2 = fma(dx, dx, fma(dy, dy, dz * dz));
                // lane masks combined on the scalar unit: accepted = active, not containing, far enough
                uint64_t in_m = 0;
                if ((ovl_m >> slot) & 1ull) in_m = __ballot((su - x.first) < x.count);
                const uint64_t am = mask & __ballot(d2 > x.tau) & ~in_m;
                if (am) {
                    R sx = 0, sy = 0, sz = 0, sm = 0;
                    if (__builtin_amdgcn_inverse_ballot_w64(am)) {
                        adj_term(dx, dy, dz, d2 + eps2, h.m, gxl, gyl, gzl, hl, sx, sy, sz, sm);
                        bx -= sx;
                        by -= sy;
                        bz -= sz;
                    }
                    src_put(slot, node, sx, sy, sz, sm);
                }
                const uint64_t om = mask & ~am;
                if (om) {
                    const uint64_t at_slot = 1ull << slot;
                    if (__builtin_amdgcn_inverse_ballot_w64(at_slot)) {
                        om_lo = (uint32_t)om;
                        om_hi = (uint32_t)(om >> 32);
                    }
                    open_m |= at_slot;
                }
            }
        }

        // the next step's nodes have other numbers
        if (have) {
            have = false;
            src_put2(hslot, 0x80u, node, hx, hy, hz, hm, (R)0, (R)0, (R)0, (R)0);
        }
        if (npair) src_flush(node);
        // opened children push their groups, all at once; of the opened leaves only those of
        // several particles contribute (a one-particle leaf is opened by its own target alone)
        const uint64_t leaf_m = __ballot(meta_leaf(meta)) & open_m;
        const uint64_t push_m = open_m & ~leaf_m;
        const int np = (int)__popcll(push_m);
        int before = 0, all = np;
        if constexpr (TEAM > 1) {
            // the waves' pushes follow each other in the order of their groups
            if (lane == 0) pushes[turn][w] = (uint32_t)np;
            __syncthreads();  // also: every wave has read its groups
            all = 0;
            for (int u = 0; u < TEAM; ++u) {
                const int c = (int)pushes[turn][u];
                if (u < w) before += c;
                all += c;
            }
            before = uni(before);
            all = uni(all);
            turn ^= 1;
        }
        if (sp + all > kStack) {
            stack_over = true;
        } else {
            if (__builtin_amdgcn_inverse_ballot_w64(push_m)) {
                const int at = sp + before + (int)popc_below(push_m);
                stk_m[sw][at] = ((uint64_t)om_hi << 32) | om_lo;
                stk_gs[sw][at] = child;
                stk_b[sw][at] = (uint8_t)((meta_nchild(meta) - 1u) | ((meta_level(meta) + 1u) << 3));
            }
            sp = uni(sp + all);
        }
        for (uint64_t lm = leaf_m & ~__ballot(meta_single(meta)); lm; lm &= lm - 1ull) {
            // Particles that share a level-21 cell can sit far closer together than
            // FP32 offsets from the wave's anchor resolve, so their separation is
            // formed in FP64 from this lane's own position (read again: the leaf is
            // rare, and kept in registers the position would cost the walk occupancy).
            const int src = (int)__builtin_ctzll(lm);
            const uint32_t f = uni(stage.st[w].aux[src].first), cnt = uni(stage.st[w].aux[src].count);
            const uint64_t om = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)om_lo, src) |
                                ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)om_hi, src) << 32);
            const volatile double* me = &a.sp[su].x;
            const double mx = me[0], my = me[1], mz = me[2];
            const bool mine = __builtin_amdgcn_inverse_ballot_w64(om);
            for (uint32_t i = f; i < f + cnt; ++i) {
                const Particle pj = a.sp[i];
                R sx = 0, sy = 0, sz = 0, sm = 0;
                if (mine && i != su) {
                    const R ex = (R)(pj.x - mx), ey = (R)(pj.y - my), ez = (R)(pj.z - mz);
                    const R q = fma(ex, ex, fma(ey, ey, ez * ez)) + eps2;
                    adj_term(ex, ey, ez, q, (R)pj.m, gxl, gyl, gzl, hl, sx, sy, sz, sm);
                    bx -= sx;
                    by -= sy;
                    bz -= sz;
                }
                wave_sum4(sx, sy, sz, sm);
                if (lane == 0) add4(a.part_grad + 4 * (int64_t)i, sx, sy, sz, sm);
            }
        }
        team_sync<TEAM>();  // the next step restages the slots and rereads the stack
        if (!F64 || ++since_fold == 2 || sp == 0) fold();
    }
    const bool any_corrupt = __ballot(most > 8u) != 0;
    if (lane == 0 && (stack_over || any_corrupt)) atomicOr(a.status, (stack_over ? 1u : 0u) | (any_corrupt ? 2u : 0u));

    double v[3];
    if constexpr (F64) {
        v[0] = tx; v[1] = ty; v[2] = tz;
    } else {
        v[0] = (double)tx - (double)cx; v[1] = (double)ty - (double)cy; v[2] = (double)tz - (double)cz;
    }
    if constexpr (TEAM > 1) {
        __syncthreads();  // the staged children are done with; the waves' totals, added in the waves' order
#pragma unroll
        for (int c = 0; c < 3; ++c) stage.total[w][c][lane] = v[c];
        __syncthreads();
        if (w > 0) return;
#pragma unroll
        for (int c = 0; c < 3; ++c) v[c] = 0.0;
#pragma unroll
        for (int u = 0; u < TEAM; ++u)
#pragma unroll
            for (int c = 0; c < 3; ++c) v[c] += stage.total[u][c][lane];
    }
    if (valid) {
        double* tg = a.target_grad + 3 * (int64_t)su;
        tg[0] = v[0]; tg[1] = v[1]; tg[2] = v[2];
    }
}

}  // namespace

// A team of 16 fills a CU, so 16384 particles fill the chip; beyond, smaller teams
// waste less on the tree's top, where a step has few groups to share.  Walk times
// in us, teams of 16 / 8 / 4 (lognormal, theta = 0.5; below, 4 / one wavefront, Plummer):
//   F32C  8192: 124 / 139 / 200    16384: 132 / 154 / 222    32768: 254 / 200 / 261    65536: 497 / 352 / 337
//   FP64  8192: 153 / 176 / 237    16384: 170 / 195 / 261    20000: 269 / 239 / 287    32768: 328 / 277 / 341
//         65536: 656 / 522 / 479
//   F32C  262144: 952 / 1363    1000000: 3541 / 3735    2000000: 7079 / 6797
//   FP64  262144: 1621 / 1940   1000000: 6915 / 6237
int adjoint_team(int64_t n, tc_walk mode)
{
    if (n <= 1 << 14) return 16;
    if (n <= 3 << 14) return 8;
    return n <= (mode == TC_WALK_F64 ? 3 << 17 : 1 << 20) ? 4 : 1;
}

namespace {

template <bool F64, int TEAM>
void launch_adj(const WalkArgs& a, hipStream_t s)
{
    const int64_t waves = walk_waves(a.n);
    const unsigned blocks = (unsigned)(TEAM > 1 ? waves : (waves + kAdjWaves - 1) / kAdjWaves);
    k_walk_adj<F64, TEAM><<<blocks, 64 * block_waves(TEAM), 0, s>>>(a);
}

template <bool F64>
void launch_adj_team(const WalkArgs& a, int team, hipStream_t s)
{
    if (team == 16) launch_adj<F64, 16>(a, s);
    else if (team == 8) launch_adj<F64, 8>(a, s);
    else if (team == 4) launch_adj<F64, 4>(a, s);
    else launch_adj<F64, 1>(a, s);
}

}  // namespace

void launch_walk_adjoint_wide(const WalkArgs& a, tc_walk mode, int team, hipStream_t s)
{
    if (a.n == 0) return;
    if (mode == TC_WALK_F64) launch_adj_team<true>(a, team, s);
    else launch_adj_team<false>(a, team, s);
}

}  // namespace tc
