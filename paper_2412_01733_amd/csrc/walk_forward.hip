// The forward walk for many particles: accelerations and potentials of Eq.(1)
// with the opening rule of the TreeCode description (section 2).
//
// Layout of the work.  One wavefront serves 64 consecutive targets of the
// target order, the particles along the Hilbert curve (spatially compact; see
// order.hip).  It walks the union of the 64 lanes' open sets: a stack in LDS
// holds groups of sibling nodes together with the 64-bit mask of lanes that
// opened their parent.  A step takes several groups off the stack and stages all
// their children at once, one lane per child; every active lane then applies
// the exact per-particle rule to each child:
//   - the node contains the target           -> open (never accepted);
//   - |X - x|^2 > (s_l / theta)^2            -> accept: one monopole term;
//   - otherwise                              -> open.
// A one-particle leaf gives the same term whether accepted or opened, so it is
// taken directly (self excluded); a multi-particle leaf (several particles
// sharing a level-21 cell) that is opened contributes its particles one by one.
// The interaction sets are therefore exactly those of the per-particle
// algorithm; only the summation order differs.
//
// What bounds it: vector instructions.  A wave64 FP32 instruction on vector
// registers issues every ~2.6 cycles of a SIMD that holds 8 wavefronts (4.5
// with a scalar operand, 8.4 for the reciprocal square root, 4.7 in FP64), and
// at 1e7 particles the walk spends ~95 % of its time issuing them.  What costs
// instructions without being arithmetic is therefore kept off the children's
// path:
//   - the box test decides most children for the whole wavefront at staging
//     (all accept, all open), without a test per target;
//   - accepted children of a group are evaluated in a straight run under the
//     group's mask.  But a third of the evaluations belong to masks of at most
//     16 lanes, 24 % to at most 8: those are transposed, 8 children x 8 targets in
//     one run, with the targets' positions passed through LDS, the sums over the
//     children taken by DPP and pulled back into the targets' lanes: ~45
//     instructions a group instead of 14 a child (LDS atomics in place of the DPP
//     sums took 19.4 ms: 8 lanes add to the same word);
//   - opened children push their groups all at once, each lane its own child, at
//     the place that a prefix count gives it; a partly opened child's mask reaches
//     its lane by v_writelane.
//
// Precision.  F32C: node and target coordinates enter as FP32 offsets from a
// per-wave FP64 anchor (the first target of the wave), formed in FP64 once
// per staged node, so differences stay small and accurate; interactions are
// FP32 (hardware reciprocal square root); plain partial sums are added every
// step into per-lane Kahan-compensated totals.  F64: absolute FP64
// coordinates, FP64 reciprocal square root refined by one third-order
// correction, plain FP64 sums.  Both walks also reduce sum_i m_i a_i and
// sum_i m_i |a_i| in FP64, one partial per wave, for the momentum diagnostic.
#include <type_traits>

#include "walk_common.h"

namespace tc {
namespace {

constexpr int kFwdWaves = 4;
constexpr int kFwdThreads = 64 * kFwdWaves;
constexpr uint32_t kXcdRun = 64;  // consecutive blocks one XCD takes at a time

// Stack bound.  An entry at position p whose nodes lie at level l is safe if
//   p + 1 + 7 + 7 (20 - l) + 1 <= kStack:
// a depth-first descent from it grows the stack by at most 7 a level.  Group j
// of a step (j = 0 the top) pushes at positions below sp - ng + 8 (j + 1), so it
// joins the step only while sp + 7 (j + 1) + 7 (20 - l) + 1 <= kStack, which
// makes its children's groups safe in turn; the top group always satisfies this,
// by being safe, and the first entry does (142).  A push beyond the stack
// therefore cannot happen; it would be refused and flagged (status bit 0).
// Shapes, measured at Plummer 1e7, theta = 0.5: sibling groups a step takes at
// most, stack entries, wavefronts per SIMD that the compiler is asked for (F32C
// compiles to 56 registers and 18.6 KB of LDS a block, which 8 share, FP64 to 68 and
// 22.7 KB, 7), and how many accepted children a sparse group must exceed to be
// transposed.
//   F32C (ms): 5 groups 12.43, 6 groups 12.11, 7 groups 12.39; never transposed
//   12.67; groups of up to 16 lanes transposed as well (4 children x 16 targets,
//   twice) 12.83.
//   FP64 (ms): 6 groups 22.55, 7 groups 22.26, 8 groups 21.97; never transposed 25.4.
// A team: the four wavefronts of a block serve the same 64 targets, share one
// stack and take a quarter of each step's groups each, so that a walk is a
// quarter as long: with fewer than ~10 wavefronts per place on the chip the
// tail and the lone chains cost more than the two barriers of a step.
constexpr int kTeamStack = 400;

template <bool F64> struct FwdShape {
    static constexpr int groups = F64 ? 8 : 6;
    static constexpr int stack = F64 ? 180 : 190;
    static constexpr int waves = F64 ? 6 : 7;
    static constexpr uint32_t min_children = F64 ? 0 : 3;
    static_assert(stack >= 142, "the root's children must be safe");
};

template <bool F64, bool COUNT, int TEAM>
__global__ __launch_bounds__(kFwdThreads) __attribute__((amdgpu_waves_per_eu(COUNT ? 1 : FwdShape<F64>::waves)))
void k_walk_fwd(WalkArgs a)
{
    using R = typename std::conditional<F64, double, float>::type;
    using Shape = FwdShape<F64>;
    constexpr int kGroups = Shape::groups, kStack = TEAM > 1 ? kTeamStack : Shape::stack, kSlots = 64;
    constexpr int kStacks = TEAM > 1 ? 1 : kFwdWaves;
    static_assert(TEAM == 1 || TEAM == kFwdWaves, "a team is a block");
    struct __align__(16) Pos { R x, y, z, m; };
    struct __align__(16) Aux { R tau; uint32_t first, count; };  // opening threshold (-1: a one-particle leaf), particle range
    struct __align__(16) Tgt { R x, y, z; };
    __shared__ uint64_t stk_m[kStacks][kStack];  // lanes that opened the parent
    __shared__ uint32_t stk_gs[kStacks][kStack]; // first node
    __shared__ uint8_t stk_b[kStacks][kStack];   // child count - 1 | level of the nodes << 3
    // staged children: slot 8 j + k holds child k of group j; after the walk a team's totals
    constexpr int kTotals = 4;
    struct __align__(16) Stage { Pos pos[kSlots]; Aux aux[kSlots]; };
    __shared__ union { Stage st[kFwdWaves]; double total[TEAM][kTotals][64]; } stage;
    __shared__ Tgt tgt[kFwdWaves][8];          // a sparse group's targets
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
    const int64_t wave_id = TEAM > 1 ? (int64_t)lb : (int64_t)lb * kFwdWaves + w;  // 64 targets
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
    R tx = 0, ty = 0, tz = 0, tp = 0;
    float cx = 0.f, cy = 0.f, cz = 0.f, cp = 0.f;
    R bx = 0, by = 0, bz = 0, bp = 0;
    uint32_t nint = 0;
    uint64_t vis_nodes = 0, vis_lanes = 0, vis_groups = 0, vis_noacc = 0, vis_allacc = 0, vis_boxopen = 0,
             vis_boxacc = 0, vis_steps = 0, vis_single = 0, vis_ovl = 0, vis_slow_acc_ovl = 0;
    int max_sp = 0;

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
    bool stack_over = false;
    uint32_t most = 0;  // children of a staged node at most (more than 8: a corrupt tree)
    int since_fold = 0, turn = 0;
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
        const uint32_t child = nd.child, meta = nd.meta;
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
        if constexpr (COUNT) {
            vis_steps += 1;
            vis_single += ng == 1;
            vis_allacc += __popcll(far_m);
            vis_boxacc += __popcll(far_m);
            vis_noacc += __popcll(near_m);
            vis_boxopen += __popcll(near_m);
            vis_ovl += __popcll(ovl_m);
        }
        wave_sync();

        for (int j = 0; j < mine; ++j) {
            const uint64_t mask = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)om_lo, 8 * j) |
                                  ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)om_hi, 8 * j) << 32);
            uint32_t fast = (uint32_t)(far_m >> (8 * j)) & 0xFFu;
            uint32_t mixed = (uint32_t)(mixed_m >> (8 * j)) & 0xFFu;
            const Pos* g8 = &stage.st[w].pos[8 * j];
            const Aux* x8 = &stage.st[w].aux[8 * j];
            uint32_t pc = (uint32_t)__popcll(mask);
            asm("" : "+s"(pc));  // keeps comparisons of it on the scalar unit, in 32 bits
            if constexpr (COUNT) {
                const uint32_t opened = (uint32_t)(near_m >> (8 * j)) & 0xFFu;
                const int nc = __popc(fast | mixed | opened);
                vis_nodes += nc;
                vis_lanes += (uint64_t)nc * (uint64_t)pc;
                vis_groups += 1;
                if (__builtin_amdgcn_inverse_ballot_w64(mask)) nint += __popc(fast);
            }
            if (pc <= 8u && (uint32_t)__popc(fast) > Shape::min_children) {
                // transposed: lane 8 r + k takes target r of the mask and child k; the sums over
                // the children go back to the target's lane
                const bool in = __builtin_amdgcn_inverse_ballot_w64(mask);
                const uint32_t r = popc_below(mask);
                if (in) tgt[w][r] = Tgt{px, py, pz};
                wave_sync();
                const uint32_t rows = fast * 0x01010101u;
                const uint64_t on = (((uint64_t)rows << 32) | rows) & (pc >= 8u ? ~0ull : (1ull << (8 * pc)) - 1ull);
                R vx = 0, vy = 0, vz = 0, vp = 0;
                if (__builtin_amdgcn_inverse_ballot_w64(on)) {
                    const Tgt q = tgt[w][lane >> 3];
                    const Pos h = g8[lane & 7];
                    const R dx = h.x - q.x, dy = h.y - q.y, dz = h.z - q.z;
                    const R ri = rsqrt_any(fma(dx, dx, fma(dy, dy, fma(dz, dz, eps2))));
                    vp = h.m * ri;
                    const R mr3 = vp * (ri * ri);
                    vx = mr3 * dx;
                    vy = mr3 * dy;
                    vz = mr3 * dz;
                }
                vx = slot_sum<8>(vx); vy = slot_sum<8>(vy); vz = slot_sum<8>(vz); vp = slot_sum<8>(vp);
                vx = lane_pull(vx, 8 * r); vy = lane_pull(vy, 8 * r); vz = lane_pull(vz, 8 * r); vp = lane_pull(vp, 8 * r);
                if (in) {
                    bx += vx; by += vy; bz += vz; bp -= vp;
                }
                wave_sync();
                fast = 0u;
            }
            if (fast && __builtin_amdgcn_inverse_ballot_w64(mask)) {
                // straight run over the accepted children; no opening test here, so the
                // softening enters the distance chain.  F32C: each slot is read while the
                // one before it is evaluated (the FP64 walk gains nothing from it).
                Pos hc = g8[0];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    Pos hn = hc;
                    if constexpr (!F64) {
                        if (k < 7) hn = g8[k + 1];
                    }
                    if ((fast >> k) & 1u) {
                        if constexpr (F64) hc = g8[k];
                        const R dx = hc.x - px, dy = hc.y - py, dz = hc.z - pz;
                        const R ri = rsqrt_any(fma(dx, dx, fma(dy, dy, fma(dz, dz, eps2))));
                        const R mr = hc.m * ri;
                        const R mr3 = mr * (ri * ri);
                        bx = fma(mr3, dx, bx);
                        by = fma(mr3, dy, by);
                        bz = fma(mr3, dz, bz);
                        bp -= mr;
                    }
                    hc = hn;
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
                if constexpr (COUNT) {
                    vis_noacc += am == 0;
                    vis_allacc += am == mask;
                    vis_slow_acc_ovl += am == mask && ((ovl_m >> slot) & 1ull);
                }
                if (__builtin_amdgcn_inverse_ballot_w64(am)) {
                    const R ri = rsqrt_any(d2 + eps2);
                    const R mr = h.m * ri;
                    const R mr3 = mr * (ri * ri);
                    bx = fma(mr3, dx, bx);
                    by = fma(mr3, dy, by);
                    bz = fma(mr3, dz, bz);
                    bp -= mr;
                    if constexpr (COUNT) ++nint;
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
            if constexpr (COUNT) max_sp = max(max_sp, sp);
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
                if (mine && i != su) {
                    const R ex = (R)(pj.x - mx), ey = (R)(pj.y - my), ez = (R)(pj.z - mz);
                    const R ri = rsqrt_any(fma(ex, ex, fma(ey, ey, ez * ez)) + eps2);
                    const R mr = (R)pj.m * ri;
                    const R mr3 = mr * (ri * ri);
                    bx = fma(mr3, ex, bx);
                    by = fma(mr3, ey, by);
                    bz = fma(mr3, ez, bz);
                    bp -= mr;
                    if constexpr (COUNT) ++nint;
                }
            }
        }
        team_sync<TEAM>();  // the next step restages the slots and rereads the stack
        // a step adds up to 8 terms a group and lane to the plain partial sums (F32C 48, folded every
        // step; FP64 64, every second), and the particles of opened leaves.  F32C: folded every step the
        // median error of acc against FP64 is 5.1e-8 at 1e6 (6.8e-8 every second step), at the same speed
        if (++since_fold == (F64 ? 2 : 1) || sp == 0) {
            since_fold = 0;
            if constexpr (F64) {
                tx += bx; ty += by; tz += bz; tp += bp;
            } else {
                kahan_add(tx, cx, bx);
                kahan_add(ty, cy, by);
                kahan_add(tz, cz, bz);
                kahan_add(tp, cp, bp);
            }
            bx = 0; by = 0; bz = 0; bp = 0;
        }
    }
    const bool any_corrupt = __ballot(most > 8u) != 0;
    if (lane == 0 && (stack_over || any_corrupt)) atomicOr(a.status, (stack_over ? 1u : 0u) | (any_corrupt ? 2u : 0u));

    R ox, oy, oz, op;
    if constexpr (F64) {
        ox = tx; oy = ty; oz = tz; op = tp;
    } else {
        ox = tx - cx; oy = ty - cy; oz = tz - cz; op = tp - cp;
    }
    if constexpr (TEAM > 1) {
        // the waves' totals, added in FP64 in the waves' order
        __syncthreads();  // the staged children are done with
        stage.total[w][0][lane] = F64 ? (double)ox : (double)tx - (double)cx;
        stage.total[w][1][lane] = F64 ? (double)oy : (double)ty - (double)cy;
        stage.total[w][2][lane] = F64 ? (double)oz : (double)tz - (double)cz;
        stage.total[w][3][lane] = F64 ? (double)op : (double)tp - (double)cp;
        __syncthreads();
        if (w > 0) return;
        double v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int u = 0; u < TEAM; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] += stage.total[u][c][lane];
        ox = (R)v[0]; oy = (R)v[1]; oz = (R)v[2]; op = (R)v[3];
    }
    write_target<R>(a, valid, su, ox, oy, oz, op, wave_id, lane);
    if constexpr (COUNT) {
        if (valid) a.counts[su] = nint;
        if (lane == 0) {
            atomicAdd(&a.visits[0], (unsigned long long)vis_nodes);
            atomicAdd(&a.visits[1], (unsigned long long)vis_lanes);
            atomicAdd(&a.visits[2], (unsigned long long)vis_groups);
            atomicAdd(&a.visits[3], (unsigned long long)vis_noacc);
            atomicAdd(&a.visits[4], (unsigned long long)vis_allacc);
            atomicAdd(&a.visits[5], (unsigned long long)vis_boxopen);
            atomicAdd(&a.visits[6], (unsigned long long)vis_boxacc);
            atomicMax(&a.visits[7], (unsigned long long)max_sp);
            atomicAdd(&a.visits[8], (unsigned long long)vis_steps);
            atomicAdd(&a.visits[9], (unsigned long long)vis_single);
            atomicAdd(&a.visits[10], (unsigned long long)vis_ovl);
            atomicAdd(&a.visits[11], (unsigned long long)vis_slow_acc_ovl);
        }
    }
}

}  // namespace

// Walk times in us, team / one wavefront (Plummer, theta = 0.5 unless said):
//   F32C  131072: 246 / 477    262144: 411 / 551    524288: 742 / 804
//         1000000: 1341 / 1396, theta = 1: 482 / 432    4000000: 5750 / 4880
//   FP64  262144: 656 / 853    1000000: 2283 / 2405    2000000: 4746 / 4549
bool walk_team(int64_t n, tc_walk mode) { return n <= (mode == TC_WALK_F64 ? 3 << 18 : 1 << 19); }

void launch_walk_forward(const WalkArgs& a, tc_walk mode, bool count, bool team, hipStream_t s)
{
    if (a.n == 0) return;
    const int64_t waves = walk_waves(a.n);
    if (count) team = false;
    const unsigned blocks = (unsigned)(team ? waves : (waves + kFwdWaves - 1) / kFwdWaves);
    if (mode == TC_WALK_F64) {
        if (count) k_walk_fwd<true, true, 1><<<blocks, kFwdThreads, 0, s>>>(a);
        else if (team) k_walk_fwd<true, false, kFwdWaves><<<blocks, kFwdThreads, 0, s>>>(a);
        else k_walk_fwd<true, false, 1><<<blocks, kFwdThreads, 0, s>>>(a);
    } else {
        if (count) k_walk_fwd<false, true, 1><<<blocks, kFwdThreads, 0, s>>>(a);
        else if (team) k_walk_fwd<false, false, kFwdWaves><<<blocks, kFwdThreads, 0, s>>>(a);
        else k_walk_fwd<false, false, 1><<<blocks, kFwdThreads, 0, s>>>(a);
    }
}

}  // namespace tc
