// FP64 pair arithmetic shared by the kick, drift, diagnostic and large-group kernels, and the
// Bulirsch-Stoer helpers shared by the one-wave and the grid-wide encounter steps.
#pragma once

#include <hip/hip_runtime.h>

#include "genga_internal.h"

namespace genga {

// separation^2 and squares without contraction: encounter decisions use exactly the rounding
// of the definition ((dx*dx + dy*dy) + dz*dz, then compare with rc*rc)
__device__ __forceinline__ double sep2_rn(double dx, double dy, double dz)
{
#pragma clang fp contract(off)
    double a = dx * dx;
    double b = dy * dy;
    double c = dz * dz;
    return (a + b) + c;
}

__device__ __forceinline__ double sq_rn(double a)
{
#pragma clang fp contract(off)
    return a * a;
}

// Changeover weight of Chambers (1999), cited in Sect. 1: K(y) = y^2 / (2y^2 - 2y + 1) on
// [0, 1], 0 below, 1 above.
__device__ __forceinline__ double changeover_k(double y)
{
    if (y <= 0.0) return 0.0;
    if (y >= 1.0) return 1.0;
    double y2 = y * y;
    return y2 / (2.0 * y2 - 2.0 * y + 1.0);
}

// 1/sqrt(q) in FP64: v_rsq_f64 (about 2^-24) and one third-order correction
__device__ __forceinline__ double inv_sqrt64(double q)
{
    const double y0 = __builtin_amdgcn_rsq(q);
    const double t = q * y0;
    const double e = fma(-t, y0, 1.0);
    const double p = fma(0.375, e, 0.5);
    return fma(y0 * e, p, y0);
}

// 1/x in FP64 for normal x well inside the range: v_rcp_f64 (about 2^-24) and one third-order
// correction; within an ulp of the quotient, at a third of the instructions of a division
__device__ __forceinline__ double inv64(double x)
{
    const double r = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, r, 1.0);
    return fma(r, fma(e, e, e), r);
}

// The changeover at separation r of a pair with i09 = 1 / (0.9 r_crit), without a division or a
// branch: y = (r - 0.1 r_crit) i09 = r i09 - 1/9 cut to [0, 1] and u = 1 - y give K = y^2 / d and
// 1 - K = u^2 / d with d = y^2 + u^2 (= 2 y^2 - 2 y + 1).  Outside r_crit u is 0, so 1 - K
// vanishes by itself.  For the larger of two radii take the smaller i09.
struct Changeover {
    double y, u, d;
};
__device__ __forceinline__ Changeover changeover_parts(double r, double i09)
{
    Changeover c;
    c.y = fmin(fmax(fma(r, i09, -1.0 / 9.0), 0.0), 1.0);
    c.u = 1.0 - c.y;
    c.d = fma(c.u, c.u, c.y * c.y);
    return c;
}

// Step reduction after a rejected step: 0.9 (tol/err)^(1/15) from the last column's error,
// kept within [1/50, 1/2].
__device__ __forceinline__ double shrink_factor(double err, double tol)
{
    const double f = 0.9 * pow(tol / err, 1.0 / (2 * BS_KMAX - 1));
    return fmax(0.02, fmin(0.5, f));
}

// Polynomial extrapolation in h^2 to h = 0 over the nodes n_0..n_k (n_j = 2(j+1)) has the
// Lagrange weights w_j = prod_{m != j} n_j^2 / (n_j^2 - n_m^2); it is the value Neville's
// scheme computes, T(k, k), and the same over the nodes 1..k gives T(k, k-1).  Both sets of
// weights sum to one, so the sums are formed relative to T(0, 0), which keeps their rounding
// at the size of the differences.
struct LagrangeTable {
    double w[BS_KMAX][BS_KMAX]; // w[k][j]: weight of T(j, 0) in T(k, k)
    double d[BS_KMAX][BS_KMAX]; // d[k][j]: weight of T(j, 0) in T(k, k) - T(k, k-1)
    constexpr LagrangeTable() : w(), d()
    {
        for (int k = 0; k < BS_KMAX; ++k)
            for (int j = 0; j <= k; ++j) {
                const double nj2 = 4.0 * (j + 1) * (j + 1);
                double a = 1.0, b = 1.0;
                for (int m = 0; m <= k; ++m) {
                    if (m == j) continue;
                    const double nm2 = 4.0 * (m + 1) * (m + 1);
                    a *= nj2 / (nj2 - nm2);
                    if (m >= 1) b *= nj2 / (nj2 - nm2);
                }
                w[k][j] = a;
                d[k][j] = j >= 1 ? a - b : a;
            }
    }
};
__constant__ constexpr LagrangeTable LAGRANGE{};

// Minimum / maximum over the 64 lanes of a wave.
__device__ __forceinline__ double wave_minv(double v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ double wave_maxv(double v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

// Bounding box of the positions held by the lanes with v = true, into
// out[t * 8 + 0..5] = (min x, y, z, max x, y, z).  Every lane of the wave calls it.
__device__ __forceinline__ void tile_box(bool v, double x, double y, double z, double *out, int t)
{
    const int lane = threadIdx.x & 63;
    const double lo[3] = {wave_minv(v ? x : INFINITY), wave_minv(v ? y : INFINITY), wave_minv(v ? z : INFINITY)};
    const double hi[3] = {wave_maxv(v ? x : -INFINITY), wave_maxv(v ? y : -INFINITY), wave_maxv(v ? z : -INFINITY)};
    if (lane < 3) {
        out[t * 8 + lane] = lo[lane];
        out[t * 8 + 3 + lane] = hi[lane];
    }
}

// Body i's acceleration: out, checked, and v += tau a.
__device__ __forceinline__ void store_accel(const KickArgs &a, int i, double tx, double ty, double tz)
{
    a.ax[i] = tx;
    a.ay[i] = ty;
    a.az[i] = tz;
    if (!(isfinite(tx) && isfinite(ty) && isfinite(tz))) atomicOr(a.flags, FLAG_NONFINITE);
    if (a.update_v) {
        a.vx[i] += a.tau * tx;
        a.vy[i] += a.tau * ty;
        a.vz[i] += a.tau * tz;
    }
}

// The tasks' shares of body `lane` (below w.ni) of item `it`, added in task order; with parts > 1
// those of part `part` of its tasks.
__device__ __forceinline__ void item_shares(const KickArgs &a, int it, const WorkItem &w, int lane, double t[3],
                                            int part = 0, int parts = 1)
{
    const int first = a.tasks ? a.task_first[it] : it * a.split;
    const uint32_t row = a.tasks ? a.item_row[it] : (uint32_t)a.split * (uint32_t)w.i0;
    int t0 = first, t1 = a.tasks ? a.task_first[it + 1] : first + a.split;
    if (parts > 1) {
        const int n = t1 - t0;
        t0 = first + n * part / parts;
        t1 = first + n * (part + 1) / parts;
    }
    t[0] = t[1] = t[2] = 0.0;
    const int ni = w.ni, stride = 3 * ni;
    const double *p = a.part + 3 * (size_t)row + (size_t)(t0 - first) * stride + lane;
    int k = t0;
    for (; k + 8 <= t1; k += 8, p += 8 * stride) { // eight tasks' loads in flight
        double v[8][3];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            for (int q = 0; q < 3; ++q) v[u][q] = p[u * stride + q * ni];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            for (int q = 0; q < 3; ++q) t[q] += v[u][q];
    }
    if (k + 4 <= t1) {
        double v[4][3];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            for (int q = 0; q < 3; ++q) v[u][q] = p[u * stride + q * ni];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            for (int q = 0; q < 3; ++q) t[q] += v[u][q];
        k += 4;
        p += 4 * stride;
    }
    for (; k < t1; ++k, p += stride)
        for (int q = 0; q < 3; ++q) t[q] += p[q * ni];
}

} // namespace genga
