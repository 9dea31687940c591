// Root cube, quantisation and Morton keys: device functions shared by keys.hip
// and sort_small.hip.
#pragma once

#include <float.h>
#include <math.h>

#include "tc_internal.h"

namespace tc {
namespace {

// Root cube from the minima mm[0..2] and maxima mm[3..5] of n >= 1 particles.
__device__ inline Geom make_geom(const double mm[6], uint32_t bad)
{
    Geom g;
    double E = 0.0;
    for (int k = 0; k < 3; ++k) {
        g.lo[k] = mm[k];
        const double ext = mm[3 + k] - mm[k];
        if (ext > E) E = ext;
    }
    int eL = 0;
    if (!isfinite(E)) {
        bad |= 1u;
    } else if (E > 0.0) {
        // E = f 2^e, f in [0.5, 1): a power of two iff f == 0.5
        int e;
        const double f = frexp(E, &e);
        eL = (f == 0.5) ? e - 1 : e;
    }
    g.log2L = eL;
    g.L = ldexp(1.0, eL);
    g.scale = ldexp(1.0, 21 - eL);
    g.h = ldexp(1.0, eL - 21);
    g.bad = bad;
    g.nnodes = 0;
    g.pad = 0;
    return g;
}

// Spread the low 21 bits of v so that bit b lands on bit 3b.
__device__ inline uint64_t spread3(uint64_t v)
{
    v &= 0x1FFFFFull;
    v = (v | (v << 32)) & 0x001F00000000FFFFull;
    v = (v | (v << 16)) & 0x001F0000FF0000FFull;
    v = (v | (v << 8)) & 0x100F00F00F00F00Full;
    v = (v | (v << 4)) & 0x10C30C30C30C30C3ull;
    v = (v | (v << 2)) & 0x1249249249249249ull;
    return v;
}

__device__ inline uint64_t quantise(double x, double lo, double scale)
{
    double f = floor((x - lo) * scale);
    if (!(f >= 0.0)) f = 0.0;
    if (f > (double)kQMax) return kQMax;
    return (uint64_t)f;
}

__device__ inline uint64_t morton(uint64_t qx, uint64_t qy, uint64_t qz)
{
    return (spread3(qx) << 2) | (spread3(qy) << 1) | spread3(qz);
}

// One particle's share of the bounds and input checks.
template <typename T>
__device__ inline void bounds_add(const T* __restrict__ pos, const T* __restrict__ mass, int64_t i, double mm[6],
                                  uint32_t& bad)
{
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double x = (double)pos[3 * i + k];
        if (!isfinite(x)) {
            bad |= 1u;
        } else {
            mm[k] = fmin(mm[k], x);
            mm[3 + k] = fmax(mm[3 + k], x);
        }
    }
    const double m = (double)mass[i];
    if (!(m >= 0.0) || !isfinite(m)) bad |= 2u;
}

// The wave's minima, maxima and flags, in every lane.
__device__ inline void bounds_wave(double mm[6], uint32_t& bad)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            mm[k] = fmin(mm[k], __shfl_xor(mm[k], o, 64));
            mm[3 + k] = fmax(mm[3 + k], __shfl_xor(mm[3 + k], o, 64));
        }
        bad |= (uint32_t)__shfl_xor((int)bad, o, 64);
    }
}

}  // namespace
}  // namespace tc
