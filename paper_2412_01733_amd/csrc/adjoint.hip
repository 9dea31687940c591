// Top-down half of the adjoint: node gradients to particle gradients.
//
// The walk's source-side gradients per node, dL/dX_n and dL/dM_n, reach the
// particles through the monopole moments M_n = sum_j m_j and
// X_n = sum_j m_j x_j / M_n (tree membership held fixed):
//   dL/dm_j += dL/dM_n + (dL/dX_n) . (x_j - X_n) / M_n,   dL/dx_j += (m_j / M_n) dL/dX_n.
// With u_n = (dL/dX_n) / M_n and c_n = dL/dM_n - u_n . X_n this is
//   dL/dm_j += c_n + u_n . x_j,   dL/dx_j += m_j u_n,
// summed over every node holding j, i.e. along the root-to-leaf path.  One
// thread per inner node works out its u_n and c_n; then one thread per particle
// starts with its leaf's, climbs to the root adding up those it passes, adds its
// target-side gradient and any direct-term gradient and writes the result in the
// caller's order.  A node of zero mass sits at its fixed cell centre, so u_n = 0
// for it.  All FP64.
//
// The steps of a climb wait only for the link up, not for the sums, and
// neighbouring particles climb through the same nodes: 12 us at 4096 particles, 14
// at 20000, 25 at 2^18, 89 at 1e6, 0.93 ms at 1e7, bound by HBM there.  (23, 35, 56,
// 126 us and 0.93 ms with the sums handed down level by level: a launch per
// populous level, whose nodes wait for the level above.)
#include "tc_internal.h"

namespace tc {
namespace {

// u_b and c_b of one node with mass and centre x.
__device__ inline void node_sums(int64_t b, const double4 x, const double* __restrict__ node_grad, double o[4])
{
    const double2* gn = reinterpret_cast<const double2*>(node_grad + 4 * b);
    const double2 g0 = gn[0], g1 = gn[1];
    o[0] = o[1] = o[2] = 0.0;
    if (x.w != 0.0) {
        o[0] = g0.x / x.w;
        o[1] = g0.y / x.w;
        o[2] = g1.x / x.w;
    }
    o[3] = g1.y - (o[0] * x.x + o[1] * x.y + o[2] * x.z);
}

__device__ inline double4 node_mass_point(const WalkNode* __restrict__ wn, int64_t b)
{
    const double2 xy = *reinterpret_cast<const double2*>(&wn[b].x), zm = *reinterpret_cast<const double2*>(&wn[b].z);
    return make_double4(xy.x, xy.y, zm.x, zm.y);
}

// s += v, the rounding error of it added to e (Knuth's two-sum).  Once an infinity or an
// overflow is met, s is the plain sum still, but e is not a number.
__device__ inline void two_sum(double& s, double& e, double v)
{
    const double t = s + v, b = t - s;
    e += (s - (t - b)) + (v - b);
    s = t;
}

__global__ __launch_bounds__(256) void k_adjoint_nodes(int64_t nn, const uint4* __restrict__ topo,
                                                       const WalkNode* __restrict__ wn,
                                                       const double* __restrict__ node_grad, double* __restrict__ uc)
{
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nn || meta_leaf(topo[b].z)) return;
    double o[4];
    node_sums(b, node_mass_point(wn, b), node_grad, o);
    double2* mine = reinterpret_cast<double2*>(uc + 4 * b);
    mine[0] = make_double2(o[0], o[1]);
    mine[1] = make_double2(o[2], o[3]);
}

// One particle (sorted position j) from its leaf.
template <typename R>
__global__ __launch_bounds__(256) void k_adjoint_particles(int64_t n, const uint32_t* __restrict__ leaf_of,
                                                           const WalkNode* __restrict__ wn, const uint2* __restrict__ up,
                                                           const double* __restrict__ node_grad, const double* __restrict__ uc,
                                                           const Particle* __restrict__ sp, const uint32_t* __restrict__ perm,
                                                           const double* __restrict__ target_grad,
                                                           const double* __restrict__ part_grad, R* __restrict__ g_pos,
                                                           R* __restrict__ g_mass)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const uint32_t b = leaf_of[j];
    const Particle q = sp[j];
    const double* tg = target_grad + 3 * j;
    const int64_t i = perm[j];
    // a one-particle leaf is its particle (mass and centre verbatim) and has no direct-term gradient
    const bool single = !((j > 0 && leaf_of[j - 1] == b) || (j + 1 < n && leaf_of[j + 1] == b));
    double4 x = make_double4(q.x, q.y, q.z, q.m);
    double2 p0 = make_double2(0.0, 0.0), p1 = p0;
    if (!single) {
        x = node_mass_point(wn, b);
        const double2* pg = reinterpret_cast<const double2*>(part_grad + 4 * j);
        p0 = pg[0];
        p1 = pg[1];
    }
    double o[4];
    node_sums(b, x, node_grad, o);
    // The terms grow towards the leaf, so what each addition rounds off is carried
    // along (relative error of the FP64 gradients at 20000: 8.7e-15 without, 5.6e-15
    // with it, 5.8e-15 when summed from the root down).
    double lost[4] = {0.0, 0.0, 0.0, 0.0};
    uint32_t a = b;
    for (int l = 0; l < kMaxLevel && a != 0u; ++l) {  // at most one step a level
        a = up[a].y;
        const double2* above = reinterpret_cast<const double2*>(uc + 4 * (int64_t)a);
        const double2 a0 = above[0], a1 = above[1];
        two_sum(o[0], lost[0], a0.x);
        two_sum(o[1], lost[1], a0.y);
        two_sum(o[2], lost[2], a1.x);
        two_sum(o[3], lost[3], a1.y);
    }
    for (int k = 0; k < 4; ++k)
        if (isfinite(lost[k])) o[k] += lost[k];
    if (g_pos) {
        g_pos[3 * i + 0] = (R)(tg[0] + p0.x + q.m * o[0]);
        g_pos[3 * i + 1] = (R)(tg[1] + p0.y + q.m * o[1]);
        g_pos[3 * i + 2] = (R)(tg[2] + p1.x + q.m * o[2]);
    }
    if (g_mass) g_mass[i] = (R)(p1.y + o[3] + (o[0] * q.x + o[1] * q.y + o[2] * q.z));
}

__global__ __launch_bounds__(256) void k_zero_f64(double* __restrict__ p, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0.0;
}

}  // namespace

void launch_fill_f64_zero(double* p, int64_t n, hipStream_t s)
{
    if (n <= 0) return;
    int64_t b = (n + 255) / 256;
    if (b > 8192) b = 8192;
    k_zero_f64<<<(unsigned)b, 256, 0, s>>>(p, n);
}

void launch_adjoint_down(int64_t nn, int64_t n, const uint4* topo, const WalkNode* wn, const uint2* up,
                         const double* node_grad, double* uc, const uint32_t* leaf_of, const Particle* sp,
                         const uint32_t* perm, const double* target_grad, const double* part_grad, void* g_pos,
                         void* g_mass, bool out_f64, hipStream_t s)
{
    k_adjoint_nodes<<<(unsigned)((nn + 255) / 256), 256, 0, s>>>(nn, topo, wn, node_grad, uc);
    const unsigned grid = (unsigned)((n + 255) / 256);
    if (out_f64)
        k_adjoint_particles<double><<<grid, 256, 0, s>>>(n, leaf_of, wn, up, node_grad, uc, sp, perm, target_grad, part_grad,
                                                         (double*)g_pos, (double*)g_mass);
    else
        k_adjoint_particles<float><<<grid, 256, 0, s>>>(n, leaf_of, wn, up, node_grad, uc, sp, perm, target_grad, part_grad,
                                                        (float*)g_pos, (float*)g_mass);
}

}  // namespace tc
