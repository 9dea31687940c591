// theta = 0: the direct sum of Eq.(1).  The opening rule never accepts a node, so
// every target takes every other particle one by one, and no tree has to be
// walked for that: the particles are read in key order and broadcast.
//
// One block serves 64 targets of the target order (a lane each) with 16
// wavefronts, each of which takes every 16th run of 64 particles: a run is
// loaded coalesced, one particle a lane, its offsets from the block's anchor are
// formed in FP64, and the 64 records are read back from LDS by all lanes.  Bound
// by the 14 vector instructions of a term; the split over 16 wavefronts fills
// the chip from ~4000 particles on (12345 particles: walk 996 -> 104 us, 1.5e12 terms a second).
//
// Precision as in walk_forward.hip: the FP32 offsets are those the walk would
// use (same anchor), the sums Kahan-compensated.  Particles that share a level-21
// cell need FP64 separations there; a set that has any takes the walk instead.
#include <type_traits>

#include "walk_common.h"

namespace tc {
namespace {

constexpr int kDirectWaves = 16;
// Terms of a plain partial sum (F32C potentials against FP64 at 5000 particles:
// 2.95e-8 with 64, 2.63e-8 with 32, as the walk (2.57e-8) with 16).
constexpr int kFold = 16;

template <bool F64>
__global__ __launch_bounds__(64 * kDirectWaves) void k_direct(WalkArgs a)
{
    using R = typename std::conditional<F64, double, float>::type;
    struct __align__(16) Pos { R x, y, z, m; };
    __shared__ Pos src[kDirectWaves][64];
    __shared__ double total[kDirectWaves][4][64];
    const int w = (int)(threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63;
    const int64_t base = (int64_t)blockIdx.x * 64;  // < n
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
    uint32_t smin = su, smax = su;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        smin = min(smin, (uint32_t)__shfl_xor((int)smin, o, 64));
        smax = max(smax, (uint32_t)__shfl_xor((int)smax, o, 64));
    }
    const int64_t own_lo = uni(smin), own_end = (int64_t)uni(smax) + 1;  // the targets lie within

    R tx = 0, ty = 0, tz = 0, tp = 0;
    float cx = 0.f, cy = 0.f, cz = 0.f, cp = 0.f;
    R bx = 0, by = 0, bz = 0, bp = 0;
    auto term = [&](const Pos& h) {
        const R dx = h.x - px, dy = h.y - py, dz = h.z - pz;
        const R ri = rsqrt_any((R)fma(dx, dx, fma(dy, dy, fma(dz, dz, eps2))));
        const R mr = h.m * ri;
        const R mr3 = mr * (ri * ri);
        bx = fma(mr3, dx, bx);
        by = fma(mr3, dy, by);
        bz = fma(mr3, dz, bz);
        bp -= mr;
    };
    for (int64_t j0 = 64 * (int64_t)w; j0 < a.n; j0 += 64 * kDirectWaves) {
        const int cnt = a.n - j0 < 64 ? (int)(a.n - j0) : 64;
        if ((int)lane < cnt) {
            const Particle q = a.sp[j0 + lane];
            Pos h;
            if constexpr (F64) {
                h.x = q.x; h.y = q.y; h.z = q.z; h.m = q.m;
            } else {
                h.x = (float)(q.x - Ax); h.y = (float)(q.y - Ay); h.z = (float)(q.z - Az);
                h.m = (float)q.m;
            }
            src[w][lane] = h;
        }
        wave_sync();
        auto fold = [&]() {
            if constexpr (F64) {
                tx += bx; ty += by; tz += bz; tp += bp;
            } else {
                kahan_add(tx, cx, bx);
                kahan_add(ty, cy, by);
                kahan_add(tz, cz, bz);
                kahan_add(tp, cp, bp);
            }
            bx = 0; by = 0; bz = 0; bp = 0;
        };
        int k = 0;
        if (j0 + cnt <= own_lo || j0 >= own_end) {
            for (; k + kFold <= cnt; k += kFold) {
#pragma unroll
                for (int v = 0; v < kFold; v += 8) {
                    Pos h[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) h[u] = src[w][k + v + u];
#pragma unroll
                    for (int u = 0; u < 8; ++u) term(h[u]);
                }
                fold();
            }
            for (; k < cnt; ++k) term(src[w][k]);
        } else {  // may hold a target: itself excluded
            for (; k < cnt; ++k) {
                const Pos h = src[w][k];
                if ((uint32_t)(j0 + k) != su) term(h);
                if (k % kFold == kFold - 1) fold();
            }
        }
        fold();
        wave_sync();
    }
    total[w][0][lane] = F64 ? (double)tx : (double)tx - (double)cx;
    total[w][1][lane] = F64 ? (double)ty : (double)ty - (double)cy;
    total[w][2][lane] = F64 ? (double)tz : (double)tz - (double)cz;
    total[w][3][lane] = F64 ? (double)tp : (double)tp - (double)cp;
    __syncthreads();
    if (w > 0) return;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (int u = 0; u < kDirectWaves; ++u)
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] += total[u][c][lane];
    write_target<R>(a, valid, su, (R)v[0], (R)v[1], (R)v[2], (R)v[3], blockIdx.x, lane);
}

}  // namespace

// Terms of a leaf that several particles share are formed in FP64 (see above).
bool direct_serves(double theta, int64_t multi_leaves) { return theta == 0.0 && multi_leaves == 0; }

void launch_direct(const WalkArgs& a, tc_walk mode, hipStream_t s)
{
    if (a.n == 0) return;
    const unsigned blocks = (unsigned)walk_waves(a.n);
    if (mode == TC_WALK_F64) k_direct<true><<<blocks, 64 * kDirectWaves, 0, s>>>(a);
    else k_direct<false><<<blocks, 64 * kDirectWaves, 0, s>>>(a);
}

}  // namespace tc
