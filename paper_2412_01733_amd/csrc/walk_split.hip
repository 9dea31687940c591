// The walk for few particles: a wavefront serves T = 8 or 16 targets.
//
// A wavefront that serves 64 targets (walk_forward.hip) evaluates one node at a time for
// all of them.  Below ~1e5 particles there are fewer such wavefronts than the
// chip has places for, and each is a long serial chain: a lone wavefront issues
// an instruction every ~8 cycles, whatever its dependences.  Here lane
// s T + t handles target t and node slot s, so that S = 64 / T nodes are
// evaluated at once, there are 64 / T times more wavefronts, and each has a
// correspondingly shorter chain (the T targets lie closer together, so they also
// open fewer nodes between them).  The price is that a node record is staged for
// T targets instead of 64, which is why large inputs stay with walk_forward.hip.
//
// A team: 2 or 4 wavefronts, the block, serve the same T targets, share one stack
// and take an equal part of each step's groups each, so that the chain is shorter
// still (the walk at 1000 particles: 46 us alone, 24 with four); once the chip is
// full the two barriers of a step and the part-filled runs cost more than that.
//
// A step takes up to 8 sibling groups off the stack and stages their <= 64
// children, one per lane.  The box test of walk_forward.hip sorts the children into
// accepted by every target (list A, compacted in LDS), opened by every target of
// the group's mask, and undecided (list M).  The slots take the entries of A in
// one straight run; those of M with the per-target rule, which leaves each
// entry's mask of opening targets in LDS.  Then all opened children push their
// groups at once, each at the place that a prefix count gives it.
//
// Decisions are those of walk_forward.hip, bit for bit: the FP32 offsets come from the
// same anchor (the first target of the aligned 64), through the same operations.
// Only the order of the sums differs; the slots' partial sums are added in FP64.
#include <type_traits>

#include "walk_common.h"

namespace tc {
namespace {

constexpr int kSplitWaves = 4;
constexpr int block_waves(int team) { return team > 1 ? team : kSplitWaves; }  // a team is a block
// Stack bound.  An entry at position p whose nodes lie at level l is safe if
//   p + 1 + 7 + 7 (20 - l) + 1 <= kSplitStack:
// a depth-first descent from it grows the stack by at most 7 a level.  Group j
// of a step (j = 0 the top) pushes at positions below sp - ng + 8 (j + 1), so it
// joins the step only while sp + 7 (j + 1) + 7 (20 - l) + 1 <= kSplitStack, which
// makes its children's groups safe in turn; the top group always satisfies this,
// by being safe, and the first entry does (142).
constexpr int kSplitStack = 256;
constexpr int kTeamStack = 400;
static_assert(kSplitStack >= 142, "the root's children must be safe");

// group entry: first node, mask (bits 0-15) | child count (16-19) | level of the nodes (20-24)
__device__ inline uint32_t pack_group(uint32_t mask, uint32_t nchild, uint32_t level)
{
    return mask | (nchild << 16) | (level << 20);
}

template <bool F64, int T, bool ADJ, int TEAM>
__global__ __launch_bounds__(64 * block_waves(TEAM)) void k_walk_split(WalkArgs a)
{
    constexpr int kWaves = block_waves(TEAM), kStacks = TEAM > 1 ? 1 : kWaves, kStack = TEAM > 1 ? kTeamStack : kSplitStack;
    constexpr int S = 64 / T;
    constexpr uint32_t kMaskT = (1u << T) - 1u;
    using R = typename std::conditional<F64, double, float>::type;
    struct __align__(16) Rec { R x, y, z, m; };
    constexpr int kRec = 64 + 2 * S;  // lists A and M, each padded to whole runs of S
    __shared__ uint2 stk[kStacks][kStack];
    __shared__ Rec rec[kWaves][kRec];
    __shared__ uint32_t rmask[kWaves][kRec];  // targets (bits 0-15) | staging lane << 16
    __shared__ R stau[kWaves][64];            // by staging lane: opening threshold,
    __shared__ uint2 srange[kWaves][64];      // first particle and count,
    __shared__ uint32_t somask[kWaves][64];   // targets that open the child
    __shared__ uint32_t pushes[2][TEAM];
    __shared__ double total[TEAM][4][TEAM > 1 ? T : 1];
    __shared__ uint32_t rnode[ADJ ? kWaves : 1][ADJ ? kRec : 1];

    const int w = (int)(threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t t = lane % T, s = lane / T;
    const uint32_t tbit = 1u << t;
    const int sw = TEAM > 1 ? 0 : w;  // whose stack
    const int64_t wave_id = TEAM > 1 ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * kWaves + w;  // T targets
    const int64_t base = wave_id * T;
    if (base >= a.n) return;  // the whole wave; of a team, the whole block
    R tau0;
    if constexpr (F64) tau0 = a.tau0_64;
    else tau0 = a.tau0_32;

    const bool valid = base + t < a.n;
    const uint32_t first_t = uni(a.order[base]);
    const uint32_t su = valid ? a.order[base + t] : first_t;
    const Particle self = a.sp[su];
    double Ax = 0.0, Ay = 0.0, Az = 0.0;
    R px, py, pz;
    if constexpr (F64) {
        px = self.x; py = self.y; pz = self.z;
    } else {
        const Particle anchor = a.sp[uni(a.order[base & ~(int64_t)63])];
        Ax = anchor.x; Ay = anchor.y; Az = anchor.z;
        px = (float)(self.x - Ax); py = (float)(self.y - Ay); pz = (float)(self.z - Az);
    }
    const R eps2 = (R)a.eps2;
    const R Gc = (R)a.G;
    R gxl = 0, gyl = 0, gzl = 0, hl = 0;  // adjoint: G dL/da and G dL/dphi of this lane's target
    if constexpr (ADJ) {
        if (valid) {
            const uint32_t i = a.perm[su];
            const R* ga = (const R*)a.g_acc;
            gxl = Gc * ga[3 * (int64_t)i + 0];
            gyl = Gc * ga[3 * (int64_t)i + 1];
            gzl = Gc * ga[3 * (int64_t)i + 2];
            if (a.g_pot) hl = Gc * ((const R*)a.g_pot)[i];
        }
    }
    // the sorted range the targets span and their bounding box (see walk_forward.hip)
    uint32_t smin = su, smax = su;
    R bnx = px, bny = py, bnz = pz, bxx = px, bxy = py, bxz = pz;
#pragma unroll
    for (int o = T / 2; o > 0; o >>= 1) {
        smin = min(smin, (uint32_t)__shfl_xor((int)smin, o, 64));
        smax = max(smax, (uint32_t)__shfl_xor((int)smax, o, 64));
        bnx = fmin(bnx, __shfl_xor(bnx, o, 64)); bny = fmin(bny, __shfl_xor(bny, o, 64));
        bnz = fmin(bnz, __shfl_xor(bnz, o, 64)); bxx = fmax(bxx, __shfl_xor(bxx, o, 64));
        bxy = fmax(bxy, __shfl_xor(bxy, o, 64)); bxz = fmax(bxz, __shfl_xor(bxz, o, 64));
    }
    const uint32_t wave_lo = smin, wave_end = smax + 1u;

    R tx = 0, ty = 0, tz = 0, tp = 0;  // totals (F32C: with compensations), plain partial sums
    float cx = 0.f, cy = 0.f, cz = 0.f, cp = 0.f;
    R bx = 0, by = 0, bz = 0, bp = 0;
    bool stack_over = false, corrupt = false;

    // one accepted entry: the term (or its adjoint) of the active lanes
    auto term = [&](const bool on, const Rec& e, const R dx, const R dy, const R dz, const R q, const uint32_t node) {
        if constexpr (!ADJ) {
            if (on) {
                const R ri = rsqrt_any(q);
                const R mr = e.m * ri;
                const R mr3 = mr * (ri * ri);
                bx = fma(mr3, dx, bx);
                by = fma(mr3, dy, by);
                bz = fma(mr3, dz, bz);
                bp -= mr;
            }
        } else {
            R sx = 0, sy = 0, sz = 0, sm = 0;
            if (on) {
                adj_term(dx, dy, dz, q, e.m, gxl, gyl, gzl, hl, sx, sy, sz, sm);
                bx -= sx;
                by -= sy;
                bz -= sz;
            }
            // sums over the T targets of the slot; four of its lanes add one component each
            const bool any = __ballot(on) >> (s * T) & kMaskT;
            sx = slot_sum<T>(sx); sy = slot_sum<T>(sy); sz = slot_sum<T>(sz); sm = slot_sum<T>(sm);
            const R v = t == 0 ? sx : t == 1 ? sy : t == 2 ? sz : sm;
            if (any && t < 4) unsafeAtomicAdd(a.node_grad + 4 * (int64_t)node + t, (double)v);
        }
    };

    int sp = 0;
    const uint32_t rmeta = uni(a.nodes[0].meta);
    if (!meta_leaf(rmeta)) {
        const uint32_t live = (uint32_t)__ballot(valid) & kMaskT;
        if (lane == 0 && w == sw) stk[sw][0] = make_uint2(uni(a.nodes[0].child), pack_group(live, meta_nchild(rmeta), 1u));
        sp = 1;
    }
    team_sync<TEAM>();

    const uint32_t gj = lane >> 3, gk = lane & 7;
    int since_fold = 0, turn = 0;
    while (sp > 0) {
        // take the groups that the stack bound allows off the top; lanes 8 j .. 8 j + 7 stage group j
        // (of a team's groups a wavefront takes up to 8, from the j0-th off the top)
        uint2 e = make_uint2(0u, 0u);
        int ng, mine;
        if constexpr (TEAM == 1) {
            bool ok = false;
            if ((int)gj < sp) {
                e = stk[sw][sp - 1 - (int)gj];
                const int l = (int)((e.y >> 20) & 31u);
                ok = gj == 0 || sp + 7 * ((int)gj + 1) + 7 * (20 - l) + 1 <= kStack;
            }
            const uint64_t okm = __ballot(ok);
            ng = ~okm ? (int)(__builtin_ctzll(~okm) >> 3) : 8;
            mine = ng;
        } else {
            bool ok = false;
            if ((int)lane < min(sp, 8 * TEAM)) {
                const int l = (int)((stk[0][sp - 1 - (int)lane].y >> 20) & 31u);
                ok = lane == 0 || sp + 7 * ((int)lane + 1) + 7 * (20 - l) + 1 <= kStack;
            }
            const uint64_t okm = __ballot(ok);
            ng = uni(~okm ? (int)__builtin_ctzll(~okm) : 64);
            const int q = (ng + TEAM - 1) / TEAM, j0 = w * q;
            mine = max(0, min(q, ng - j0));
            if ((int)gj < mine) e = stk[0][sp - 1 - j0 - (int)gj];
        }
        sp = uni(sp - ng);
        const uint32_t nc = (e.y >> 16) & 15u, pmask = e.y & 0xFFFFu;
        const bool live = (int)gj < mine && gk < min(nc, 8u);
        if (__ballot(live && nc > 8u)) corrupt = true;
        bool far_all = false, near_all = false;
        uint32_t child = 0, meta = 0, first = 0, count = 0;
        Rec h;
        const uint32_t node = e.x + gk;
        if (live) {
            const WalkNode nd = a.nodes[node];
            if constexpr (F64) {
                h.x = nd.x; h.y = nd.y; h.z = nd.z; h.m = nd.m;
            } else {
                h.x = (float)(nd.x - Ax); h.y = (float)(nd.y - Ay); h.z = (float)(nd.z - Az);
                h.m = (float)nd.m;
            }
            first = nd.first;
            count = nd.count;
            child = nd.child;
            meta = nd.meta;
            const bool ovl = first < wave_end && first + count > wave_lo;
            const R tau = meta_single(meta) ? (R)-1 : (R)ldexp(tau0, -2 * (int)meta_level(meta));
            stau[w][lane] = tau;
            srange[w][lane] = make_uint2(first, count);
            // the box test of walk_forward.hip: decided for every target of the wavefront
            const R gx = fmax(fmax(bnx - h.x, h.x - bxx), (R)0), fx = fmax(fabs(h.x - bnx), fabs(h.x - bxx));
            const R gy = fmax(fmax(bny - h.y, h.y - bxy), (R)0), fy = fmax(fabs(h.y - bny), fabs(h.y - bxy));
            const R gz = fmax(fmax(bnz - h.z, h.z - bxz), (R)0), fz = fmax(fabs(h.z - bnz), fabs(h.z - bxz));
            far_all = !ovl && fma(gx, gx, fma(gy, gy, gz * gz)) > tau;
            near_all = !far_all && !(fma(fx, fx, fma(fy, fy, fz * fz)) > tau);
        }
        const bool mixed = live && !far_all && !near_all;
        const uint64_t fm = __ballot(far_all), mm = __ballot(mixed);
        const int na = (int)__popcll(fm), nm = (int)__popcll(mm);
        const int na_pad = (na + S - 1) & ~(S - 1), end = na_pad + ((nm + S - 1) & ~(S - 1));
        if (far_all || mixed) {
            const uint32_t at = far_all ? popc_below(fm) : (uint32_t)na_pad + popc_below(mm);
            rec[w][at] = h;
            rmask[w][at] = pmask | (lane << 16);
            if constexpr (ADJ) rnode[w][at] = node;
        }
        if ((int)lane < na_pad - na) rmask[w][na + (int)lane] = 0u;
        if ((int)lane < end - na_pad - nm) rmask[w][na_pad + nm + (int)lane] = 0u;
        wave_sync();

        // list A: accepted by every target of the entry's mask
        {
            Rec hc = rec[w][s];
            uint32_t mc = rmask[w][s];
            for (int e0 = 0; e0 < na_pad; e0 += S) {
                // the next run's entry is read while this one is evaluated (the last read may fall
                // into list M or past it, within the array, and is not used)
                const Rec hn = rec[w][e0 + S + (int)s < kRec ? e0 + S + (int)s : 0];
                const uint32_t mn = rmask[w][e0 + S + (int)s < kRec ? e0 + S + (int)s : 0];
                const R dx = hc.x - px, dy = hc.y - py, dz = hc.z - pz;
                term((mc & tbit) != 0u, hc, dx, dy, dz, fma(dx, dx, fma(dy, dy, fma(dz, dz, eps2))),
                     ADJ ? rnode[ADJ ? w : 0][ADJ ? e0 + (int)s : 0] : 0u);
                hc = hn;
                mc = mn;
            }
        }
        // list M: the per-target rule (accepted = active, not containing, far enough)
        for (int e0 = na_pad; e0 < end; e0 += S) {
            const Rec hc = rec[w][e0 + (int)s];
            const uint32_t mc = rmask[w][e0 + (int)s];
            const uint32_t src = mc >> 16;
            const uint2 fr = srange[w][src];
            const R tau = stau[w][src];
            const R dx = hc.x - px, dy = hc.y - py, dz = hc.z - pz;
            const R d2 = fma(dx, dx, fma(dy, dy, dz * dz));
            const bool active = (mc & tbit) != 0u;
            const bool take = active && d2 > tau && !((su - fr.x) < fr.y);
            term(take, hc, dx, dy, dz, d2 + eps2, ADJ ? rnode[ADJ ? w : 0][ADJ ? e0 + (int)s : 0] : 0u);
            const uint64_t om = __ballot(active && !take);
            if (t == 0 && (mc & kMaskT)) somask[w][src] = (uint32_t)(om >> (s * T)) & kMaskT;
        }
        wave_sync();

        // opened children push their groups; an opened multi-particle leaf's particles are taken one by one
        uint32_t open = 0u;
        if (near_all) open = pmask;
        else if (mixed) open = somask[w][lane];
        const bool leaf = meta_leaf(meta);
        const uint64_t pm = __ballot(open != 0u && !leaf);
        const int np = (int)__popcll(pm);
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
            turn ^= 1;
        }
        if (sp + all > kStack) {
            stack_over = true;  // cannot happen (see the bound); refused and flagged
        } else {
            if (open != 0u && !leaf)
                stk[sw][sp + before + (int)popc_below(pm)] =
                    make_uint2(child, pack_group(open, meta_nchild(meta), meta_level(meta) + 1u));
            sp = uni(sp + all);
        }
        for (uint64_t lm = __ballot(open != 0u && leaf && count > 1u); lm; lm &= lm - 1ull) {
            const int src = (int)__builtin_ctzll(lm);
            const uint32_t f = (uint32_t)__builtin_amdgcn_readlane((int)first, src);
            const uint32_t cnt = (uint32_t)__builtin_amdgcn_readlane((int)count, src);
            const uint32_t om = (uint32_t)__builtin_amdgcn_readlane((int)open, src);
            const bool lane_open = (om & tbit) != 0u;
            for (uint32_t j0 = 0; j0 < cnt; j0 += S) {
                // separations in FP64: the particles share a level-21 cell (see walk_forward.hip)
                const uint32_t j = f + j0 + s;
                const bool in = j0 + s < cnt;
                const Particle pj = a.sp[in ? j : f];
                const bool on = in && lane_open && j != su;
                R sx = 0, sy = 0, sz = 0, sm = 0;
                if (on) {
                    const Particle me = a.sp[su];
                    const R mj = (R)pj.m;
                    const R ex = (R)(pj.x - me.x), ey = (R)(pj.y - me.y), ez = (R)(pj.z - me.z);
                    const R q = fma(ex, ex, fma(ey, ey, ez * ez)) + eps2;
                    if constexpr (!ADJ) {
                        const R ri = rsqrt_any(q);
                        const R mr = mj * ri;
                        const R mr3 = mr * (ri * ri);
                        bx = fma(mr3, ex, bx);
                        by = fma(mr3, ey, by);
                        bz = fma(mr3, ez, bz);
                        bp -= mr;
                    } else {
                        adj_term(ex, ey, ez, q, mj, gxl, gyl, gzl, hl, sx, sy, sz, sm);
                        bx -= sx;
                        by -= sy;
                        bz -= sz;
                    }
                }
                if constexpr (ADJ) {
                    sx = slot_sum<T>(sx); sy = slot_sum<T>(sy); sz = slot_sum<T>(sz); sm = slot_sum<T>(sm);
                    const R v = t == 0 ? sx : t == 1 ? sy : t == 2 ? sz : sm;
                    if (in && t < 4) unsafeAtomicAdd(a.part_grad + 4 * (int64_t)j + t, (double)v);
                }
            }
        }
        team_sync<TEAM>();
        // F32C: a step adds up to 64 / S + 1 terms a lane to the plain sums (lists A and M are
        // padded apart), so up to 2 (64 / S + 1) between folds, and the particles of opened leaves
        if (++since_fold == 2 || sp == 0) {
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
    if (lane == 0 && (stack_over || corrupt)) atomicOr(a.status, (stack_over ? 1u : 0u) | (corrupt ? 2u : 0u));

    // the slots' totals, added in FP64
    double v[4];
    if constexpr (F64) {
        v[0] = tx; v[1] = ty; v[2] = tz; v[3] = tp;
    } else {
        v[0] = (double)tx - (double)cx; v[1] = (double)ty - (double)cy;
        v[2] = (double)tz - (double)cz; v[3] = (double)tp - (double)cp;
    }
#pragma unroll
    for (int o = T; o < 64; o <<= 1)
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] += __shfl_xor(v[k], o, 64);
    if constexpr (TEAM > 1) {
        // the waves' totals, added in the waves' order
        if (s == 0)
#pragma unroll
            for (int k = 0; k < 4; ++k) total[w][k][t] = v[k];
        __syncthreads();
        if (w > 0) return;
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = total[0][k][t];
#pragma unroll
        for (int u = 1; u < TEAM; ++u)
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] += total[u][k][t];
    }

    if constexpr (ADJ) {
        if (valid && s == 0) {
            double* tg = a.target_grad + 3 * (int64_t)su;
            tg[0] = v[0]; tg[1] = v[1]; tg[2] = v[2];
        }
    } else {
        write_target<R>(a, valid && s == 0, su, (R)v[0], (R)v[1], (R)v[2], (R)v[3], wave_id, lane);
    }
}

template <bool F64, int T, bool ADJ, int TEAM>
void launch_split(const WalkArgs& a, hipStream_t s)
{
    const int64_t waves = (a.n + T - 1) / T;
    const unsigned blocks = (unsigned)(TEAM > 1 ? waves : (waves + kSplitWaves - 1) / kSplitWaves);
    k_walk_split<F64, T, ADJ, TEAM><<<blocks, 64 * block_waves(TEAM), 0, s>>>(a);
}

}  // namespace

// Where the lines lie (walk times in us on one MI355X, Plummer, theta = 0.5; T targets /
// wavefronts that share them; 64 / 4: the team of walk_forward.hip):
//             8/1   8/2   8/4   8/8   16/1  16/2  16/4  64/4
//   F32C 1000   46    32    24    24    60    40    28     -
//        4096   62    43    31    33    95    62    40   106
//        8192   69    48    36    55   102    67    43     -
//       16384   77    56    63    93   113    73    52   132
//       32768   92   100   111   170   116    85    89   143
//       65536  171   180   213   342   155   151   159   180
//       98000  235   256   313   504   218   210   225     -
//      131072  300     -     -     -   262     -     -   244
//   FP64 4096   65    44    33    36    99    65    42   128
//        8192   73    51    42    66   108    72    47     -
//       16384   87    69    80   125   120    83    67   154
//       32768  123   131   146   242   139   117   120   180
//       65536  228   246   288   491   220   214   224   238
//      100000  336   366   435   758   306   317   338   318
//      131072  431   479   571   994   378   403   437   406
int walk_targets(int64_t n, tc_walk mode)
{
    if (n <= 3 << 12) return 8;
    return n <= (mode == TC_WALK_F64 ? 1 << 17 : 3 << 15) ? 16 : 64;
}

int64_t walk_rows_max(int64_t n)
{
    const int t = min(walk_targets(n, TC_WALK_F32C), walk_targets(n, TC_WALK_F64));
    return (n + t - 1) / t;
}

// The adjoint adds to a node's gradient with four atomics per wavefront and node,
// so fewer targets a wavefront mean more atomics (us; T = 8 with 1 / 2 / 4 / 8
// wavefronts, and 16 wavefronts for 64 targets, see walk_adjoint.hip):
//   F32C  1000: 68 / 47 / 36 / 33, -    4096: 107 / 80 / 63 / 66, 111    8192: 159 / 132 / 131 / 118, 124
//   FP64  1000: 75 / 50 / 38 / 36, -    4096: 122 / 85 / 70 / 67, 137    8192: 170 / 144 / 131 / 125, 153
int adjoint_targets(int64_t n) { return n <= 7 << 10 ? 8 : 64; }

void launch_walk_split(const WalkArgs& a, int targets, tc_walk mode, hipStream_t s)
{
    if (a.n == 0) return;
    const bool f64 = mode == TC_WALK_F64;
    if (targets == 8) f64 ? launch_split<true, 8, false, 4>(a, s) : launch_split<false, 8, false, 4>(a, s);
    else if (a.n <= 3 << 13) f64 ? launch_split<true, 16, false, 4>(a, s) : launch_split<false, 16, false, 4>(a, s);
    else if (!f64 || a.n <= 5 << 14) f64 ? launch_split<true, 16, false, 2>(a, s) : launch_split<false, 16, false, 2>(a, s);
    else launch_split<true, 16, false, 1>(a, s);
}

void launch_walk_split_adjoint(const WalkArgs& a, tc_walk mode, hipStream_t s)
{
    if (a.n == 0) return;
    if (mode == TC_WALK_F64) launch_split<true, 8, true, 4>(a, s);
    else launch_split<false, 8, true, 4>(a, s);
}

}  // namespace tc
