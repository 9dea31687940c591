// Device helpers shared by the walk kernels.
#pragma once

#include "tc_internal.h"

namespace tc {
namespace {

__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// What separates a step's LDS accesses: TEAM wavefronts of a block share the stack, or one has its own.
template <int TEAM>
__device__ inline void team_sync()
{
    if constexpr (TEAM > 1) __syncthreads();
    else wave_sync();
}

__device__ inline uint32_t uni(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline float uni_r(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }
__device__ inline double uni_r(double v)
{
    const long long b = __double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b), hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// 1/sqrt(x) in FP64: with the hardware estimate y (relative error below
// 2^-24, measured) and r = 1 - x y^2, the exact value is y (1 - r)^(-1/2);
// its series truncated after the quadratic term, y (1 + r/2 + 3 r^2/8), leaves
// an error of order r^3 ~ 2^-72, below FP64 rounding (measured maximum 1.25
// ulp, the same as two Newton-Raphson steps, with 5 operations instead of 8).
__device__ inline double rsqrt64(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double r = fma(-x * y, y, 1.0);
    return fma(y * r, fma(0.375, r, 0.5), y);
}

__device__ inline float rsqrt_any(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ inline double rsqrt_any(double x) { return rsqrt64(x); }

__device__ inline void kahan_add(float& s, float& c, float v)
{
    float y = v - c;
    float t = s + y;
    c = (t - s) - y;
    s = t;
}

template <typename R>
__device__ inline R wave_sum(R v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Adjoint of one term (mass mu at offset (dx,dy,dz) from the target,
// q = d^2 + eps^2) for dL/da = (gx,gy,gz), dL/dphi = h.  With
// T = q^-3/2 I - 3 q^-5/2 Delta Delta^T the source receives
//   dL/dy  = G mu (T g + q^-3/2 Delta h)   (the target receives the negative),
//   dL/dmu = G (Delta.g q^-3/2 - h q^-1/2).
// Both are linear in (g, h): the caller passes G g and G h.
template <typename R>
__device__ inline void adj_term(R dx, R dy, R dz, R q, R mu, R gx, R gy, R gz, R h, R& sx, R& sy, R& sz, R& sm)
{
    const R ri = rsqrt_any(q);
    const R ri2 = ri * ri;
    const R ri3 = ri2 * ri;
    const R dg = fma(dx, gx, fma(dy, gy, dz * gz));
    const R c1 = mu * ri3;
    const R c2 = c1 * fma((R)-3 * ri2, dg, h);
    sx = fma(c1, gx, c2 * dx);
    sy = fma(c1, gy, c2 * dy);
    sz = fma(c1, gz, c2 * dz);
    sm = fma(dg, ri3, -h * ri);
}

// Sum over the wave of four values; the result is uniform.
template <typename R>
__device__ inline void wave_sum4(R& a0, R& a1, R& a2, R& a3)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        a0 += __shfl_xor(a0, o, 64);
        a1 += __shfl_xor(a1, o, 64);
        a2 += __shfl_xor(a2, o, 64);
        a3 += __shfl_xor(a3, o, 64);
    }
}

// Sum over each 16-lane row of the wave (DPP: xor 1, xor 2, half-row
// mirror, row mirror; every lane active, so that bound_ctrl changes nothing but
// lets the move fold into the addition); afterwards every lane holds its row's sum.
__device__ inline float dpp_f(float v, int ctrl)
{
    switch (ctrl) {  // the control word must be a constant
    case 0: return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));
    case 1: return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xF, 0xF, true));
    case 2: return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x141, 0xF, 0xF, true));
    default: return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x140, 0xF, 0xF, true));
    }
}

__device__ inline double dpp_d(double v, int ctrl)
{
    const long long b = __double_as_longlong(v);
    int lo = (int)(b & 0xFFFFFFFF), hi = (int)(b >> 32);
    switch (ctrl) {
    case 0: lo = __builtin_amdgcn_mov_dpp(lo, 0xB1, 0xF, 0xF, true); hi = __builtin_amdgcn_mov_dpp(hi, 0xB1, 0xF, 0xF, true); break;
    case 1: lo = __builtin_amdgcn_mov_dpp(lo, 0x4E, 0xF, 0xF, true); hi = __builtin_amdgcn_mov_dpp(hi, 0x4E, 0xF, 0xF, true); break;
    case 2: lo = __builtin_amdgcn_mov_dpp(lo, 0x141, 0xF, 0xF, true); hi = __builtin_amdgcn_mov_dpp(hi, 0x141, 0xF, 0xF, true); break;
    default: lo = __builtin_amdgcn_mov_dpp(lo, 0x140, 0xF, 0xF, true); hi = __builtin_amdgcn_mov_dpp(hi, 0x140, 0xF, 0xF, true); break;
    }
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

template <typename R>
__device__ inline R row_sum(R v)
{
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        if constexpr (sizeof(R) == 8) v += dpp_d(v, c);
        else v += dpp_f(v, c);
    }
    return v;
}

__device__ inline void add4(double* dst, double v0, double v1, double v2, double v3)
{
    unsafeAtomicAdd(dst + 0, v0);
    unsafeAtomicAdd(dst + 1, v1);
    unsafeAtomicAdd(dst + 2, v2);
    unsafeAtomicAdd(dst + 3, v3);
}

// Sum over aligned runs of T = 8 or 16 lanes; every lane holds its run's sum.
template <int T, typename R>
__device__ inline R slot_sum(R v)
{
#pragma unroll
    for (int c = 0; c < (T == 16 ? 4 : 3); ++c) {
        if constexpr (sizeof(R) == 8) v += dpp_d(v, c);
        else v += dpp_f(v, c);
    }
    return v;
}

// Exchanges lanes 32-63 of a with lanes 0-31 of b.
__device__ inline void half_swap(float& a, float& b)
{
    const auto r = __builtin_amdgcn_permlane32_swap((unsigned)__float_as_int(a), (unsigned)__float_as_int(b), false, false);
    a = __int_as_float((int)r[0]);
    b = __int_as_float((int)r[1]);
}

__device__ inline void half_swap(double& a, double& b)
{
    const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    a = __longlong_as_double((long long)(((uint64_t)hi[0] << 32) | lo[0]));
    b = __longlong_as_double((long long)(((uint64_t)hi[1] << 32) | lo[1]));
}

// Sum over aligned runs of N = 2, 4 or 8 lanes.
template <uint32_t N, typename R>
__device__ inline R part_sum(R v)
{
#pragma unroll
    for (int c = 0; c < (N == 8 ? 3 : N == 4 ? 2 : 1); ++c) {
        if constexpr (sizeof(R) == 8) v += dpp_d(v, c);
        else v += dpp_f(v, c);
    }
    return v;
}

// The value that lane `from` (taken modulo 64) holds.
__device__ inline float lane_pull(float v, uint32_t from)
{
    return __int_as_float(__builtin_amdgcn_ds_bpermute((int)(from << 2), __float_as_int(v)));
}

__device__ inline uint32_t lane_pull_u(uint32_t v, uint32_t from)
{
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(from << 2), (int)v);
}

__device__ inline double lane_pull(double v, uint32_t from)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_ds_bpermute((int)(from << 2), (int)(b & 0xFFFFFFFF));
    const int hi = __builtin_amdgcn_ds_bpermute((int)(from << 2), (int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Count of set bits of m strictly below this lane.
__device__ inline uint32_t popc_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// The outputs of a wavefront's targets (lanes with `valid`; su: sorted position),
// scaled by G, in the caller's order, and its row of the momentum diagnostic:
// sum m a, sum m |a| in FP64.
template <typename R>
__device__ inline void write_target(const WalkArgs& a, const bool valid, const uint32_t su, R ox, R oy, R oz, R op,
                                    const int64_t row, const uint32_t lane)
{
    const R G = (R)a.G;
    ox *= G; oy *= G; oz *= G; op *= G;
    double dm[4] = {0.0, 0.0, 0.0, 0.0};
    if (valid) {
        const uint32_t i = a.perm[su];
        R* acc = (R*)a.acc;
        acc[3 * (int64_t)i + 0] = ox;
        acc[3 * (int64_t)i + 1] = oy;
        acc[3 * (int64_t)i + 2] = oz;
        if (a.pot) ((R*)a.pot)[i] = op;
        const double m = a.sp[su].m;
        const double ex = (double)ox, ey = (double)oy, ez = (double)oz;
        dm[0] = m * ex;
        dm[1] = m * ey;
        dm[2] = m * ez;
        dm[3] = m * sqrt(ex * ex + ey * ey + ez * ez);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) dm[k] = wave_sum(dm[k]);
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) a.diag[4 * row + k] = dm[k];
    }
}

}  // namespace
}  // namespace tc
