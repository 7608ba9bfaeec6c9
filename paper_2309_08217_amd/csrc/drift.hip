// Drift part of the hybrid symplectic step (Brasser et al. 2023, Sect. 1), all FP64:
//  * Sun drift: r_i += tau * (sum_j m_j v_j) / Mstar (democratic heliocentric split);
//  * Kepler drift of every body not in a close encounter, by universal variables (Stumpff
//    functions; Halley's method on the universal Kepler equation, a bracketed solver where it
//    does not settle);
//  * close-encounter step: the encounter pairs are joined into groups (connected components,
//    one workgroup, in LDS for up to 1024 pairs), and each group is integrated over dt by
//    Gragg-Bulirsch-Stoer under the Sun's force plus the (1 - K) share of the members' mutual
//    forces, in the same launch as the Kepler drift (groups of 9-64 in one beside or after it).
#include "genga_internal.h"
#include "pair_math.h"
#include "union_find.h"

namespace genga {

namespace {

// ------------------------------------------------------------------------------------------
// Sun drift in two launches over chunks of one system: partial momenta per chunk (fixed-order
// block reduction), then every chunk adds its system's partials in chunk order and shifts
// its positions.  Deterministic.
// ------------------------------------------------------------------------------------------
constexpr int SUN_THREADS = CHUNK;

__global__ __launch_bounds__(SUN_THREADS) void momentum_kernel(const Chunk *chunks, const double *m,
                                                               const double *vx, const double *vy,
                                                               const double *vz, double *mom_part)
{
    __shared__ double red[3][SUN_THREADS / 64];
    const Chunk c = chunks[blockIdx.x];
    double px = 0.0, py = 0.0, pz = 0.0;
    for (int i = c.b + threadIdx.x; i < c.e; i += SUN_THREADS) {
        px += m[i] * vx[i];
        py += m[i] * vy[i];
        pz += m[i] * vz[i];
    }
    for (int o = 32; o > 0; o >>= 1) {
        px += __shfl_xor(px, o, 64);
        py += __shfl_xor(py, o, 64);
        pz += __shfl_xor(pz, o, 64);
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0) {
        red[0][wave] = px;
        red[1][wave] = py;
        red[2][wave] = pz;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double P[3] = {0.0, 0.0, 0.0};
        for (int w = 0; w < SUN_THREADS / 64; ++w)
            for (int q = 0; q < 3; ++q) P[q] += red[q][w];
        for (int q = 0; q < 3; ++q) mom_part[3 * (size_t)blockIdx.x + q] = P[q];
    }
}

// Momentum of system s for a block of SUN_THREADS threads: the chunk partials summed with a
// stride, then a fixed tree, so every block of the system gets the same value.
__device__ __forceinline__ void system_momentum(const int32_t *chunk_first, const double *mom_part, int s,
                                                double (*red)[SUN_THREADS / 64], double P[3])
{
    double Px = 0.0, Py = 0.0, Pz = 0.0;
    for (int k = chunk_first[s] + threadIdx.x; k < chunk_first[s + 1]; k += SUN_THREADS) {
        Px += mom_part[3 * (size_t)k];
        Py += mom_part[3 * (size_t)k + 1];
        Pz += mom_part[3 * (size_t)k + 2];
    }
    for (int o = 32; o > 0; o >>= 1) {
        Px += __shfl_xor(Px, o, 64);
        Py += __shfl_xor(Py, o, 64);
        Pz += __shfl_xor(Pz, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = Px;
        red[1][threadIdx.x >> 6] = Py;
        red[2][threadIdx.x >> 6] = Pz;
    }
    __syncthreads();
    P[0] = P[1] = P[2] = 0.0;
    for (int w = 0; w < SUN_THREADS / 64; ++w)
        for (int q = 0; q < 3; ++q) P[q] += red[q][w];
    __syncthreads();
}

__global__ __launch_bounds__(SUN_THREADS) void sun_shift_kernel(const Chunk *chunks,
                                                                const int32_t *chunk_first,
                                                                const double *mstar,
                                                                const double *mom_part, double tau,
                                                                double *x, double *y, double *z)
{
    __shared__ double red[3][SUN_THREADS / 64];
    const Chunk c = chunks[blockIdx.x];
    double P[3];
    system_momentum(chunk_first, mom_part, c.sys, red, P);
    const double f = tau / mstar[c.sys];
    const double sx = f * P[0], sy = f * P[1], sz = f * P[2];
    for (int i = c.b + threadIdx.x; i < c.e; i += SUN_THREADS) {
        x[i] += sx;
        y[i] += sy;
        z[i] += sz;
    }
}

// ------------------------------------------------------------------------------------------
// Kepler drift by universal variables.
// ------------------------------------------------------------------------------------------

// Stumpff functions c2(z) = (1 - cos sqrt z)/z, c3(z) = (sqrt z - sin sqrt z)/z^(3/2)
// (hyperbolic forms for z < 0); series for |z| < 1.
__device__ void stumpff(double zz, double &c2, double &c3)
{
    if (fabs(zz) < 1.0) {
        // c2 = sum (-z)^k / (2k+2)!, c3 = sum (-z)^k / (2k+3)!
        double t2 = 0.5, t3 = 1.0 / 6.0;
        double s2 = t2, s3 = t3;
        for (int k = 1; k < 14; ++k) {
            t2 *= -zz / ((2.0 * k + 1.0) * (2.0 * k + 2.0));
            t3 *= -zz / ((2.0 * k + 2.0) * (2.0 * k + 3.0));
            s2 += t2;
            s3 += t3;
        }
        c2 = s2;
        c3 = s3;
    } else if (zz > 0.0) {
        double sz = sqrt(zz);
        double h = sin(0.5 * sz);
        c2 = 2.0 * h * h / zz;
        c3 = (sz - sin(sz)) / (zz * sz);
    } else {
        double sz = sqrt(-zz);
        double h = sinh(0.5 * sz);
        c2 = 2.0 * h * h / (-zz);
        c3 = (sinh(sz) - sz) / (-zz * sz);
    }
}

// (r, v) advanced on the two-body orbit about mu by dt; ok false if not converged.  Any orbit and
// step: the root of the universal Kepler equation is bracketed first.
struct KeplerState {
    double x, y, z, vx, vy, vz;
    bool ok;
};
__device__ __noinline__ KeplerState kepler_bracketed(double x, double y, double z, double vx, double vy, double vz,
                                                     double mu, double dt)
{
    const double r0 = sqrt(x * x + y * y + z * z);
    const double v2 = vx * vx + vy * vy + vz * vz;
    const double sig = (x * vx + y * vy + z * vz) / sqrt(mu); // r0 . v0 / sqrt(mu)
    const double alpha = 2.0 / r0 - v2 / mu;                   // 1 / a
    const double smu = sqrt(mu);
    // universal Kepler equation F(chi) = sig chi^2 c2 + (1 - alpha r0) chi^3 c3 + r0 chi - sqrt(mu) dt
    // F'(chi) = r(chi) > 0.  Bracket the root, then safeguarded Newton.
    double chi = (alpha > 0.0) ? smu * dt * alpha : smu * dt / r0;
    double lo, hi;
    {
        // expand a bracket around the first guess
        double step = fabs(chi) + (alpha > 0.0 ? 1.0 / sqrt(alpha) : r0);
        lo = chi - step;
        hi = chi + step;
        for (int k = 0; k < 200; ++k) {
            double c2, c3, zz = alpha * lo * lo;
            stumpff(zz, c2, c3);
            double F = sig * lo * lo * c2 + (1.0 - alpha * r0) * lo * lo * lo * c3 + r0 * lo - smu * dt;
            if (F <= 0.0) break;
            lo -= step;
            step *= 2.0;
        }
        step = fabs(hi - chi) + 1e-300;
        for (int k = 0; k < 200; ++k) {
            double c2, c3, zz = alpha * hi * hi;
            stumpff(zz, c2, c3);
            double F = sig * hi * hi * c2 + (1.0 - alpha * r0) * hi * hi * hi * c3 + r0 * hi - smu * dt;
            if (F >= 0.0) break;
            hi += step;
            step *= 2.0;
        }
    }
    bool ok = false;
    double c2 = 0.5, c3 = 1.0 / 6.0, rr = r0;
    for (int it = 0; it < 100; ++it) {
        const double zz = alpha * chi * chi;
        stumpff(zz, c2, c3);
        const double chi2 = chi * chi;
        const double F = sig * chi2 * c2 + (1.0 - alpha * r0) * chi2 * chi * c3 + r0 * chi - smu * dt;
        rr = sig * chi * (1.0 - zz * c3) + (1.0 - alpha * r0) * chi2 * c2 + r0;
        if (F > 0.0) hi = chi; else lo = chi;
        const double step = F / rr;
        if (fabs(step) <= 1e-15 * fabs(chi) || hi - lo <= 4e-16 * fabs(chi)) {
            // converged: take the last Newton correction (it may sit on the bracket edge)
            chi -= step;
            ok = true;
            break;
        }
        double nx = chi - step;
        if (!(nx > lo && nx < hi)) nx = 0.5 * (lo + hi);
        chi = nx;
    }
    const double zz = alpha * chi * chi;
    stumpff(zz, c2, c3);
    const double chi2 = chi * chi;
    const double f = 1.0 - chi2 / r0 * c2;
    const double g = dt - chi2 * chi / smu * c3;
    const double nxp = f * x + g * vx, nyp = f * y + g * vy, nzp = f * z + g * vz;
    const double r = sqrt(nxp * nxp + nyp * nyp + nzp * nzp);
    const double fd = smu / (r * r0) * chi * (zz * c3 - 1.0);
    const double gd = 1.0 - chi2 / r * c2;
    return KeplerState{nxp, nyp, nzp, fd * x + gd * vx, fd * y + gd * vy, fd * z + gd * vz, ok};
}

// c2 and c3 for |z| < 1 by Horner's rule: the first dropped terms are 1/22! and 1/23!
__device__ __forceinline__ void stumpff_series(double z, double &c2, double &c3)
{
    constexpr double f[20] = {// 1 / (n + 2)!
                              1.0 / 2, 1.0 / 6, 1.0 / 24, 1.0 / 120, 1.0 / 720, 1.0 / 5040, 1.0 / 40320, 1.0 / 362880,
                              1.0 / 3628800, 1.0 / 39916800, 1.0 / 479001600, 1.0 / 6227020800.0,
                              1.0 / 87178291200.0, 1.0 / 1307674368000.0, 1.0 / 20922789888000.0,
                              1.0 / 355687428096000.0, 1.0 / 6402373705728000.0, 1.0 / 121645100408832000.0,
                              1.0 / 2432902008176640000.0, 1.0 / 51090942171709440000.0};
    c2 = f[18];
    c3 = f[19];
#pragma unroll
    for (int k = 8; k >= 0; --k) {
        c2 = fma(-z, c2, f[2 * k]);
        c3 = fma(-z, c3, f[2 * k + 1]);
    }
}

// The same for the steps a run takes, a fraction of an orbit (|alpha| chi^2 < 1): from the guess
// of the third-order expansion in dt by Halley steps, whose error falls with its cube, so that a
// correction below 1e-6 of chi is the last.  Latency bound (one wave per SIMD at most for a
// disc): the bracketing and the Stumpff series' divisions took three times as long.  Whatever
// does not converge goes to the bracketed solver.
__device__ bool kepler_universal(double &x, double &y, double &z, double &vx, double &vy, double &vz, double mu,
                                 double dt)
{
    if (dt == 0.0) return true;
    const double q0 = fma(x, x, fma(y, y, z * z)), ir0 = inv_sqrt64(q0), r0 = q0 * ir0;
    const double v2 = fma(vx, vx, fma(vy, vy, vz * vz));
    const double ismu = inv_sqrt64(mu), smu = mu * ismu;
    const double sig = fma(x, vx, fma(y, vy, z * vz)) * ismu; // r0 . v0 / sqrt(mu)
    const double alpha = fma(2.0, ir0, -v2 * (ismu * ismu));  // 1 / a
    const double beta = fma(-alpha, r0, 1.0);
    const double M = smu * dt;
    // r0 chi + sig chi^2 / 2 + beta chi^3 / 6 = M to third order in M / r0
    const double w = M * ir0, p = 0.5 * sig * ir0, b = beta * ir0 * (1.0 / 6.0);
    double chi = w * fma(w, fma(w, fma(2.0 * p, p, -b), -p), 1.0);
    bool ok = false;
    double c2, c3;
    for (int it = 0; it < 8 && !ok; ++it) {
        const double c = chi * chi, zz = alpha * c;
        if (!(fabs(zz) < 1.0)) break;
        stumpff_series(zz, c2, c3);
        const double g1 = chi * fma(-zz, c3, 1.0), g2 = c * c2, g3 = c * chi * c3;
        const double F = fma(sig, g2, fma(beta, g3, fma(r0, chi, -M)));
        const double r = fma(sig, g1, fma(beta, g2, r0));       // dF / dchi
        const double rp = fma(sig, fma(-zz, c2, 1.0), beta * g1); // d2F / dchi2
        // Halley: F / (r - F r' / (2 r))
        const double n = F * inv64(r);
        const double step = n * inv64(fma(-0.5 * n, rp * inv64(r), 1.0));
        chi -= step;
        ok = fabs(step) <= 1e-6 * fabs(chi);
    }
    const double c = chi * chi, zz = alpha * c;
    if (!ok || !(fabs(zz) < 1.0)) {
        const KeplerState k = kepler_bracketed(x, y, z, vx, vy, vz, mu, dt);
        x = k.x;
        y = k.y;
        z = k.z;
        vx = k.vx;
        vy = k.vy;
        vz = k.vz;
        return k.ok;
    }
    stumpff_series(zz, c2, c3);
    const double g2 = c * c2;
    const double f = fma(-g2, ir0, 1.0), g = fma(-c * chi * c3, ismu, dt);
    const double nx = fma(f, x, g * vx), ny = fma(f, y, g * vy), nz = fma(f, z, g * vz);
    const double ir = inv_sqrt64(fma(nx, nx, fma(ny, ny, nz * nz)));
    const double fd = smu * (ir * ir0) * chi * fma(zz, c3, -1.0);
    const double gd = fma(-g2, ir, 1.0);
    const double nvx = fma(fd, x, gd * vx), nvy = fma(fd, y, gd * vy), nvz = fma(fd, z, gd * vz);
    x = nx;
    y = ny;
    z = nz;
    vx = nvx;
    vy = nvy;
    vz = nvz;
    return true;
}

__device__ __forceinline__ void store_state(double *x, double *y, double *z, double *vx, double *vy,
                                            double *vz, int b, const double *Y)
{
    x[b] = Y[0];
    y[b] = Y[1];
    z[b] = Y[2];
    vx[b] = Y[3];
    vy[b] = Y[4];
    vz[b] = Y[5];
}

// ------------------------------------------------------------------------------------------
// Encounter groups: one workgroup.  lab[] (init -1) and mark[] (init 0) are global arrays
// over all bodies that this kernel leaves clean again for the next step, and for uf_union_kernel,
// which takes every label that is not -1 as a link of its own.
// Output: members[] sorted by (group root, body), group_start[g] (g < n_groups, plus an end
// sentinel), member_slot[body] = position in members[] (-1: in no group that is integrated).
// ------------------------------------------------------------------------------------------
constexpr int CE_THREADS = 1024;
constexpr int BS_LANES = 64;
constexpr int CP_MEM = 8; // largest group whose extrapolation columns run side by side
static_assert(CP_MEM * BS_KMAX == BS_LANES, "one lane per (column, member)");

__device__ __forceinline__ double wave_sum(double v)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Grid-wide union-find of the encounter pairs in one launch, for the large-group mode and the
// levels: afterwards every body of a pair leads to its component's smallest body.  A thread joins
// its pair's roots, the larger under the smaller, by compare-and-swap; one that finds the root
// taken meanwhile goes on from where it now leads.  Every failure is another thread's success, so
// the loops end.  (Rounds of hooking, each of which could lose to another's, and of compressing
// were up to 13 launches; 40322 bodies in one group: 290 -> 200 us.)
__global__ __launch_bounds__(256) void uf_union_kernel(const int32_t *pairs, const int32_t *pair_count,
                                                       int32_t pair_cap, int32_t *lab)
{
    const int np = min(*pair_count, pair_cap);
    for (int p = blockIdx.x * 256 + threadIdx.x; p < np; p += gridDim.x * 256) {
        int a = pairs[2 * p], b = pairs[2 * p + 1];
        const int la = uf_load(lab, a), lb = uf_load(lab, b);
        if (la >= 0 && la == lb) continue; // most pairs of a large tree by then
        if (la < 0) atomicCAS(&lab[a], -1, a);
        if (lb < 0) atomicCAS(&lab[b], -1, b);
        a = uf_find(lab, a);
        b = uf_find(lab, b);
        while (a != b) {
            const int lo = min(a, b), hi = max(a, b);
            // (a root that is no longer one costs no compare-and-swap: pairs of two large trees
            // all try the same root, and they would queue on that address)
            if (uf_load(lab, hi) == hi && atomicCAS(&lab[hi], hi, lo) == hi) break;
            a = uf_find(lab, hi);
            b = uf_find(lab, lo);
        }
    }
}

// A list of up to GF_PAIRS pairs (a disc whose r_crit is a few Hill radii has tens to hundreds)
// is joined in LDS: a thread per pair, a hash table of the bodies, union-find over its slots; the
// rounds' dependent loads were most of the builder's 6-14 us when the labels were in global memory.
constexpr int GF_PAIRS = CE_THREADS;
constexpr int GF_SLOTS = 4096, GF_RANK = 256;
static_assert(GF_SLOTS >= 2 * 2 * GF_PAIRS, "hash table at most half full");

struct GroupFast {
    int32_t body[GF_SLOTS], par[GF_SLOTS]; // a slot's body and its parent slot (a smaller body)
    uint64_t keys[2 * GF_PAIRS];
};
struct GroupLds {
    union {
        uint64_t keys[CE_MAX_MEMBERS];
        GroupFast f;
        uint64_t sorted[2 * GF_PAIRS]; // over the hash table, which is then no longer used
    };
    int32_t nmem, changed, ng, cnt[CE_THREADS / 64];
};
static_assert(sizeof(GroupFast) <= CE_MAX_MEMBERS * sizeof(uint64_t), "the fast path's tables fit");
static_assert(2 * GF_PAIRS * sizeof(uint64_t) <= 2 * GF_SLOTS * sizeof(int32_t), "sorted keys end before the keys");

__device__ __forceinline__ int slot_root(const int32_t *par, int a)
{
    int r = ((volatile const int32_t *)par)[a];
    while (r != a) {
        a = r;
        r = ((volatile const int32_t *)par)[a];
    }
    return r;
}

__device__ __forceinline__ int slot_of(GroupLds &S, int b)
{
    int h = (int)(((uint32_t)b * 2654435761u) >> 20);
    for (;;) {
        const int32_t old = atomicCAS(&S.f.body[h], -1, b);
        if (old == b) return h;
        if (old == -1) {
            S.f.par[h] = h;
            S.f.keys[atomicAdd(&S.nmem, 1)] = (uint64_t)h;
            return h;
        }
        h = (h + 1) & (GF_SLOTS - 1);
    }
}

// Bitonic sort of keys[0..n), padded with all-ones to a power of two.
__device__ __forceinline__ void sort_keys(uint64_t *keys, int n)
{
    const int tid = threadIdx.x;
    int npow = 1;
    while (npow < n) npow <<= 1;
    for (int k = n + tid; k < npow; k += CE_THREADS) keys[k] = ~0ull;
    __syncthreads();
    for (int size = 2; size <= npow; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int k = tid; k < npow; k += CE_THREADS) {
                const int partner = k ^ stride;
                if (partner > k) {
                    const bool up = (k & size) == 0;
                    const uint64_t a = keys[k], b = keys[partner];
                    if ((a > b) == up) {
                        keys[k] = b;
                        keys[partner] = a;
                    }
                }
            }
            __syncthreads();
        }
    }
}

// Members of the groups of np pairs as sorted keys (root body << 32 | body), their number.
__device__ const uint64_t *group_keys_fast(const GroupBuild &g, GroupLds &S, int np, int &nmem)
{
    const int tid = threadIdx.x;
    for (int k = tid; k < GF_SLOTS; k += CE_THREADS) S.f.body[k] = -1;
    __syncthreads();
    int sa = 0, sb = 0;
    if (tid < np) {
        sa = slot_of(S, g.pairs[2 * tid]);
        sb = slot_of(S, g.pairs[2 * tid + 1]);
    }
    __syncthreads();
    // the larger root's body hooks under the smaller; a hook that another thread's overwrites
    // is made again in the next round
    for (;;) {
        if (tid == 0) S.changed = 0;
        __syncthreads();
        if (tid < np) {
            const int a = slot_root(S.f.par, sa), b = slot_root(S.f.par, sb);
            if (a != b) {
                const bool less = S.f.body[a] < S.f.body[b];
                S.f.par[less ? b : a] = less ? a : b;
                S.changed = 1;
            }
        }
        __syncthreads();
        if (!S.changed) break;
        __syncthreads();
    }
    nmem = S.nmem;
    for (int k = tid; k < nmem; k += CE_THREADS) {
        const int h = (int)S.f.keys[k], r = slot_root(S.f.par, h);
        S.f.keys[k] = ((uint64_t)(uint32_t)S.f.body[r] << 32) | (uint32_t)S.f.body[h];
    }
    __syncthreads();
    if (nmem > GF_RANK) {
        sort_keys(S.f.keys, nmem);
        return S.f.keys;
    }
    // few members: a key's place is the number of smaller ones
    if (tid < nmem) {
        const uint64_t key = S.f.keys[tid];
        int rank = 0;
        for (int k = 0; k < nmem; ++k) rank += S.f.keys[k] < key;
        S.sorted[rank] = key;
    }
    __syncthreads();
    return S.sorted;
}

__device__ const uint64_t *group_keys_global(const GroupBuild &g, GroupLds &S, int np, int &nmem)
{
    uint64_t *keys = S.keys;
    const int tid = threadIdx.x;
    int32_t *lab = g.lab, *mark = g.mark;
    const int32_t *pairs = g.pairs;
    // collect distinct member bodies; each becomes its own root
    for (int p = tid; p < np; p += CE_THREADS) {
        for (int e = 0; e < 2; ++e) {
            const int b = pairs[2 * p + e];
            if (atomicCAS(&mark[b], 0, 1) == 0) {
                const int k = atomicAdd(&S.nmem, 1);
                if (k < CE_MAX_MEMBERS) keys[k] = (uint64_t)(uint32_t)b;
                __hip_atomic_store(&lab[b], b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    __syncthreads();
    const int nmem_all = S.nmem;
    nmem = min(nmem_all, CE_MAX_MEMBERS);
    if (nmem_all > CE_MAX_MEMBERS) {
        if (tid == 0) atomicOr(g.flags, FLAG_CAPACITY);
    }
    // union by hooking the larger root under the smaller until no pair spans two roots
    for (int round = 0; round < 4096; ++round) {
        if (tid == 0) S.changed = 0;
        __syncthreads();
        for (int p = tid; p < np; p += CE_THREADS) {
            int a = uf_root(lab, pairs[2 * p]);
            int b = uf_root(lab, pairs[2 * p + 1]);
            if (a != b) {
                const int lo = min(a, b), hi = max(a, b);
                if (uf_load(lab, hi) > lo) atomicMin(&lab[hi], lo);
                S.changed = 1;
            }
        }
        __syncthreads();
        if (!S.changed) break;
        __syncthreads();
    }
    // sort members by (root, body) so each group is contiguous and in ascending order
    for (int k = tid; k < nmem; k += CE_THREADS) {
        const int b = (int)(keys[k] & 0xffffffffu);
        const int r = uf_root(lab, b);
        keys[k] = ((uint64_t)(uint32_t)r << 32) | (uint32_t)b;
    }
    sort_keys(keys, nmem);
    // every root has been read (sort_keys has barriers): labels and marks are left as they were found
    for (int p = tid; p < np; p += CE_THREADS)
        for (int e = 0; e < 2; ++e) {
            const int b = pairs[2 * p + e];
            mark[b] = 0;
            __hip_atomic_store(&lab[b], -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    return keys;
}

// The groups of CP_MEM + 1 .. BS_LANES members in group order, by one workgroup (a ballot and a
// scan per round of 1024 groups): list[0] their number, list[1 + i] the groups.
__device__ __forceinline__ void list_wg_groups(const int32_t *group_start, int G, int32_t *list, int32_t *wsum)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int base = 0;
    for (int c = 0; c < G; c += CE_THREADS) {
        const int g = c + (int)threadIdx.x;
        const int nb = g < G ? group_start[g + 1] - group_start[g] : 0;
        const bool med = nb > CP_MEM && nb <= BS_LANES;
        const unsigned long long bal = __ballot(med);
        if (lane == 0) wsum[wave] = __popcll(bal);
        __syncthreads();
        int off = 0, tot = 0;
        for (int w = 0; w < CE_THREADS / 64; ++w) {
            off += w < wave ? wsum[w] : 0;
            tot += wsum[w];
        }
        if (med) list[1 + base + off + __popcll(bal & ((1ull << lane) - 1))] = g;
        base += tot;
        __syncthreads(); // wsum is rewritten by the next round
    }
    if (threadIdx.x == 0) list[0] = base;
}

// One workgroup of CE_THREADS: members, group_start, n_groups, member_slot and wg_list.
__device__ void build_groups(const GroupBuild &g, GroupLds &S)
{
    const int tid = threadIdx.x;
    const int np = min(*g.pair_count, g.pair_cap);
    if (tid == 0) {
        S.nmem = 0;
        S.ng = 0;
    }
    __syncthreads();
    if (np <= 0) {
        if (tid == 0) {
            *g.n_groups = 0;
            g.wg_list[0] = 0;
        }
        return;
    }
    int nmem = 0;
    const uint64_t *keys = np <= GF_PAIRS ? group_keys_fast(g, S, np, nmem) : group_keys_global(g, S, np, nmem);
    // write members; number the groups with a chunked scan of the start flags
    const int per = (nmem + CE_THREADS - 1) / CE_THREADS;
    const int kb = min(tid * per, nmem), ke = min(kb + per, nmem);
    int nstart = 0;
    for (int k = kb; k < ke; ++k) {
        g.members[k] = (int)(keys[k] & 0xffffffffu);
        if (k == 0 || (keys[k - 1] >> 32) != (keys[k] >> 32)) ++nstart;
    }
    // exclusive scan of the per-thread start counts: in-wave shuffles, then the wave totals
    const int lane = tid & 63, wave = tid >> 6;
    int incl = nstart;
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
    }
    if (lane == 63) S.cnt[wave] = incl;
    __syncthreads();
    int gi = incl - nstart, ng = 0;
    for (int w = 0; w < CE_THREADS / 64; ++w) {
        gi += w < wave ? S.cnt[w] : 0;
        ng += S.cnt[w];
    }
    // Members beyond CE_MAX_MEMBERS (flagged) can leave groups of one, and so more groups than the
    // drift has blocks and sums for: the members of those get no slot and are Kepler-drifted.
    for (int k = kb; k < ke; ++k) {
        if (k == 0 || (keys[k - 1] >> 32) != (keys[k] >> 32)) {
            if (gi <= CE_MAX_GROUPS) g.group_start[gi] = k;
            ++gi;
        }
        if (gi <= CE_MAX_GROUPS) g.member_slot[(int)(keys[k] & 0xffffffffu)] = k; // in group gi - 1
    }
    if (ng <= CE_MAX_GROUPS && tid == 0) g.group_start[ng] = nmem;
    ng = min(ng, CE_MAX_GROUPS);
    if (tid == 0) *g.n_groups = ng;
    __threadfence_block();
    __syncthreads(); // group_start is read back by other threads
    list_wg_groups(g.group_start, ng, g.wg_list, S.cnt);
}

// The end of a list's import: its length, or 0 with FLAG_BADPAIR when a pair was invalid.
__device__ __forceinline__ void import_finish(const PairImport &p)
{
    const int c = *p.src_count;
    const bool good = !*p.bad && c >= 0;
    *p.dst_count = good ? c : 0;
    if (!good) atomicOr(p.flags, FLAG_BADPAIR);
    else if (c > p.cap) atomicOr(p.flags, FLAG_CAPACITY);
    *p.bad = 0;
}

__global__ __launch_bounds__(64) void import_finish_kernel(PairImport p)
{
    if (threadIdx.x == 0) import_finish(p);
}

__global__ __launch_bounds__(CE_THREADS) void ce_groups_kernel(GroupBuild g, PairImport p)
{
    __shared__ GroupLds S;
    if (p.src) {
        if (threadIdx.x == 0) import_finish(p);
        __syncthreads();
    }
    build_groups(g, S);
}

// What a wave of a CloseBlock works on: an item of a system (item < 0: none), or a part of its tasks.
struct CloseWave {
    int sys, item, part, parts;
    int f0, f1;     // the system's items
    int w0, waves;  // the system's waves
    double mstar;
};

// SMALL: the layout has blocks of several systems.  (Looked up in every block, they cost layouts without
// any 0.5 to 1 us a launch.)
template <bool SMALL>
__device__ __forceinline__ CloseWave close_wave(const CloseBlock &blk, const StepMomentum &pm, int wave)
{
    if (SMALL && blk.waves != CLOSE_WAVES) {
        const int k = wave / blk.waves, s = blk.sys + min(k, blk.n - 1);
        const int f0 = pm.item_first[s], f1 = pm.item_first[s + 1], it = f0 + wave % blk.waves;
        return CloseWave{s, k < blk.n && it < f1 ? it : -1, 0, 1, f0, f1, k * blk.waves, blk.waves, pm.mstar[s]};
    }
    const int k = wave / pm.parts;
    return CloseWave{blk.sys, k < blk.n ? blk.item + k : -1, wave % pm.parts, pm.parts, blk.f0, blk.f1, 0, CLOSE_WAVES,
                     blk.mstar};
}

// The rows of a block's sums from its waves' (red), once every wave has stored its own.
template <bool SMALL>
__device__ __forceinline__ void store_rows(const CloseBlock &blk, const double (*red)[CLOSE_WAVES], double *rows)
{
    const int tid = threadIdx.x;
    if (SMALL && blk.waves != CLOSE_WAVES) {
        const int i = tid / 3, q = tid % 3;
        if (i >= blk.n) return;
        double s = 0.0;
        for (int k = 0; k < blk.waves; ++k) s += red[q][i * blk.waves + k];
        rows[3 * (size_t)(blk.row + i) + q] = s;
    } else if (tid < 3) {
        double s = 0.0;
        for (int k = 0; k < CLOSE_WAVES; ++k) s += red[tid][k];
        rows[3 * (size_t)blk.row + tid] = s;
    }
}

// What a drift outside a step starts from, in one launch: the momentum sums of the items' blocks,
// and, from the workgroups after them, the check and copy of a caller's pair list.
template <bool SMALL>
__global__ __launch_bounds__(CE_THREADS) void drift_open_kernel(const WorkItem *items, const double *vx,
                                                                const double *vy, const double *vz, const double *m,
                                                                StepMomentum pm, PairImport im)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if ((int)blockIdx.x >= pm.n_blocks) {
        const int n = min(*im.src_count, im.cap), first = (blockIdx.x - pm.n_blocks) * CE_THREADS + tid;
        bool ok = true;
        for (int p = first; p < n; p += (gridDim.x - pm.n_blocks) * CE_THREADS) {
            const int i = im.src[2 * p], j = im.src[2 * p + 1];
            const bool good = i >= 0 && i < j && j < im.n_total && im.sys_of[i] == im.sys_of[j];
            ok = ok && good;
            im.dst[2 * p] = good ? i : 0;
            im.dst[2 * p + 1] = good ? j : 0;
        }
        if (!ok) atomicOr(im.bad, 1);
        return;
    }
    __shared__ double red[3][CLOSE_WAVES];
    const CloseBlock blk = pm.blocks[blockIdx.x];
    double p[3] = {0.0, 0.0, 0.0};
    const CloseWave c = close_wave<SMALL>(blk, pm, wave);
    if (c.item >= 0 && c.part == 0) {
        const WorkItem w = items[c.item];
        if (lane < w.ni) {
            const int i = w.i0 + lane;
            const double mi = m[i];
            p[0] = mi * vx[i];
            p[1] = mi * vy[i];
            p[2] = mi * vz[i];
        }
    }
    for (int q = 0; q < 3; ++q) {
        p[q] = wave_sum(p[q]);
        if (lane == 0) red[q][wave] = p[q];
    }
    __syncthreads();
    store_rows<SMALL>(blk, red, pm.kick);
}

// The first of the G groups (in system order) whose system is not below s, by a wave in two rounds of
// loads.
__device__ __forceinline__ int first_group(const int32_t *group_sys, int G, int s)
{
    static_assert(CE_MAX_GROUPS <= 64 * 64, "two rounds of 64");
    const int lane = threadIdx.x & 63, step = (G + 63) / 64;
    const auto below = [&](int k, bool on) { return __popcll(__ballot(on && k < G && group_sys[k] < s)); };
    const int n = below(lane * step, true);
    if (n == 0) return 0;
    return (n - 1) * step + below((n - 1) * step + lane, lane < step);
}

// The second half of a Sun drift, tau P / Mstar of the wave's system, P summed after the drift by item
// and by group from the system's first group on, so that the order of the sum depends on the system
// alone (groups are in system order).  Every thread of the workgroup calls it.  G: the drift's groups;
// gs: the system of group tid, loaded ahead; red: LDS; first: a word of LDS.
template <bool SMALL>
__device__ __forceinline__ void close_shift(const StepMomentum &pm, const CloseWave &c, int G, int gs, int *first,
                                            double (*red)[CLOSE_WAVES], double sh[3])
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double P[3] = {0.0, 0.0, 0.0};
    const auto add = [&](const double *part, int k) {
        for (int q = 0; q < 3; ++q) P[q] += part[3 * (size_t)k + q];
    };
    if (!SMALL || c.waves == CLOSE_WAVES) { // the whole workgroup
        if (pm.n_large && c.f1 - c.f0 > LARGE_ROWS * CLOSE_WAVES) { // (runs of CLOSE_WAVES items there)
            if (tid == 0) add(pm.sys_kepler, c.sys);
        } else {
            for (int k = c.f0 + tid; k < c.f1; k += CE_THREADS) add(pm.kepler, k);
        }
        if (tid == 0) *first = G;
        __syncthreads();
        for (int k = tid; k < G; k += CE_THREADS) {
            if (k != tid) gs = pm.group_sys[k];
            if (gs == c.sys) {
                atomicMin(first, k);
                break;
            }
        }
        __syncthreads();
        for (int k = *first + tid; k < G && pm.group_sys[k] == c.sys; k += CE_THREADS) add(pm.group, k);
    } else if (wave == c.w0) { // the system's first wave: as many items as lanes at most
        if (c.f0 + lane < c.f1) add(pm.kepler, c.f0 + lane);
        if (G > 0)
            for (int k = first_group(pm.group_sys, G, c.sys) + lane; k < G && pm.group_sys[k] == c.sys; k += 64)
                add(pm.group, k);
    }
    for (int q = 0; q < 3; ++q) {
        P[q] = wave_sum(P[q]);
        if (lane == 0) red[q][wave] = P[q];
    }
    __syncthreads();
    const double f = pm.tau / c.mstar;
    for (int q = 0; q < 3; ++q) {
        double s = 0.0;
        if (SMALL)
            for (int k = 0; k < c.waves; ++k) s += red[q][c.w0 + k];
        else
            for (int k = 0; k < CLOSE_WAVES; ++k) s += red[q][k];
        sh[q] = f * s;
    }
}

// The second half of the Sun drift after a drift outside a step: positions + tau P / Mstar.
template <bool SMALL>
__global__ __launch_bounds__(CE_THREADS) void drift_close_kernel(const WorkItem *items, double *x, double *y, double *z,
                                                                 StepMomentum pm)
{
    __shared__ double red[3][CLOSE_WAVES];
    __shared__ int first;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const CloseBlock blk = pm.blocks[blockIdx.x];
    const int G = *pm.group_n, gs = pm.group_sys[tid];
    const CloseWave c = close_wave<SMALL>(blk, pm, wave);
    const WorkItem w = c.item >= 0 && c.part == 0 ? items[c.item] : WorkItem{0, 0, 0, 0};
    const bool on = lane < w.ni;
    const int i = w.i0 + lane;
    double X[3] = {0.0, 0.0, 0.0}, sh[3];
    if (on) {
        X[0] = x[i];
        X[1] = y[i];
        X[2] = z[i];
    }
    close_shift<SMALL>(pm, c, G, gs, &first, red, sh);
    if (on) {
        x[i] = X[0] + sh[0];
        y[i] = X[1] + sh[1];
        z[i] = X[2] + sh[2];
    }
}

// A system's sum over part[3 first[s] ..), by every lane of a wave.
__device__ __forceinline__ void wave_momentum(const int32_t *first, const double *part, int s, double P[3])
{
    P[0] = P[1] = P[2] = 0.0;
    for (int k = first[s] + (int)(threadIdx.x & 63); k < first[s + 1]; k += 64)
        for (int q = 0; q < 3; ++q) P[q] += part[3 * (size_t)k + q];
    for (int q = 0; q < 3; ++q) P[q] = wave_sum(P[q]);
}

// The sums of part[3 first[s] ..) of the large systems s, a workgroup each.
__global__ __launch_bounds__(CE_THREADS) void large_sums_kernel(const int32_t *large, const int32_t *first,
                                                                const double *part, double *sums)
{
    __shared__ double red[3][CE_THREADS / 64];
    const int s = large[blockIdx.x], tid = threadIdx.x, k1 = first[s + 1];
    double P[3] = {0.0, 0.0, 0.0};
    for (int k = first[s] + tid; k < k1; k += 4 * CE_THREADS) { // four rows in flight
        double v[4][3];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            for (int q = 0; q < 3; ++q) v[u][q] = part[3 * (size_t)min(k + u * CE_THREADS, k1 - 1) + q];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            for (int q = 0; q < 3; ++q) P[q] += k + u * CE_THREADS < k1 ? v[u][q] : 0.0;
    }
    for (int q = 0; q < 3; ++q) {
        P[q] = wave_sum(P[q]);
        if ((tid & 63) == 0) red[q][tid >> 6] = P[q];
    }
    __syncthreads();
    if (tid < 3) {
        double t = 0.0;
        for (int w = 0; w < CE_THREADS / 64; ++w) t += red[tid][w];
        sums[3 * (size_t)s + tid] = t;
    }
}

// The end of a kick inside a step (launch_kick_close).  Workgroup 0 builds the groups, the others
// take a block of items each, of which those of a large system have up to four waves an item, which
// share its tasks (20040 bodies in FP64, 39 tasks an item: 14 us with four waves, 26 with one).
// Latency bound, a chain of loads of what other launches wrote: everything a wave needs is loaded before
// the first barrier, in three rounds.
template <bool SMALL>
__global__ __launch_bounds__(CE_THREADS) void kick_close_kernel(KickArgs a, double *x, double *y, double *z,
                                                                StepMomentum pm, GroupBuild g, int with_groups)
{
    __shared__ GroupLds S;
    constexpr int NW = CLOSE_WAVES;
    static_assert(NW == CE_THREADS / 64, "the block's waves");
    if (blockIdx.x == 0) {
        if (with_groups) build_groups(g, S);
        return;
    }
    double(*red)[NW] = reinterpret_cast<double(*)[NW]>(S.keys);                     // [6][NW]
    double(*share)[NW][64] = reinterpret_cast<double(*)[NW][64]>(S.keys + 6 * NW); // [3][NW][64]
    static_assert((6 + 3 * 64) * NW <= CE_MAX_MEMBERS, "the sums fit");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool shift = pm.tau != 0.0;
    // first round: the block, the drift's groups (one per thread; more below)
    const CloseBlock blk = pm.blocks[blockIdx.x - 1];
    const int G = shift ? *pm.group_n : 0;
    const int gs = shift ? pm.group_sys[tid] : -1;
    // second round: the item, its tasks
    const CloseWave c = close_wave<SMALL>(blk, pm, wave);
    const WorkItem w = c.item >= 0 ? a.items[c.item] : WorkItem{0, 0, 0, 0};
    const bool on = lane < w.ni, lead = on && c.part == 0;
    const int i = w.i0 + lane;
    // third: the shares and the body
    double t[3] = {0.0, 0.0, 0.0}, X[3] = {0.0, 0.0, 0.0}, V[3] = {0.0, 0.0, 0.0}, sh[3] = {0.0, 0.0, 0.0}, mi = 0.0;
    if (lead) {
        mi = a.m[i];
        V[0] = a.vx[i];
        V[1] = a.vy[i];
        V[2] = a.vz[i];
        if (shift) {
            X[0] = x[i];
            X[1] = y[i];
            X[2] = z[i];
        }
    }
    if (on) item_shares(a, c.item, w, lane, t, c.part, c.parts);
    for (int q = 0; q < 3; ++q) share[q][wave][lane] = t[q];
    if (shift) close_shift<SMALL>(pm, c, G, gs, &S.ng, red, sh);
    __syncthreads();
    double p[3] = {0.0, 0.0, 0.0};
    if (lead) {
        for (int k = 1; k < c.parts; ++k)
            for (int q = 0; q < 3; ++q) t[q] += share[q][wave + k][lane];
        a.ax[i] = t[0];
        a.ay[i] = t[1];
        a.az[i] = t[2];
        if (!(isfinite(t[0]) && isfinite(t[1]) && isfinite(t[2]))) atomicOr(a.flags, FLAG_NONFINITE);
        for (int q = 0; q < 3; ++q) {
            V[q] += a.tau * t[q];
            p[q] = mi * V[q];
        }
        a.vx[i] = V[0];
        a.vy[i] = V[1];
        a.vz[i] = V[2];
        if (shift) {
            x[i] = X[0] + sh[0];
            y[i] = X[1] + sh[1];
            z[i] = X[2] + sh[2];
        }
    }
    for (int q = 0; q < 3; ++q) {
        p[q] = wave_sum(p[q]);
        if (lane == 0) red[3 + q][wave] = p[q];
    }
    __syncthreads();
    store_rows<SMALL>(blk, red + 3, pm.kick);
}

// ------------------------------------------------------------------------------------------
// Bulirsch-Stoer over dt for the close-encounter groups (FP64): one wavefront per group.
// Same method as the oracle: modified midpoint with n_k = 2(k+1) sub-steps (k = 0..7),
// polynomial extrapolation in h^2 by Neville's scheme, and the step accepted at the first
// column k >= 1 whose last two entries agree to tol on the group's position and velocity
// scales.  After a step accepted at column k the next one is doubled (k <= 4), kept
// (k = 5, 6) or halved (k = 7); a rejected step shrinks by shrink_factor.  Step decisions use
// wave-wide values, so control flow stays uniform.
//
// Everything per lane lives in registers except what other lanes read: the positions
// published for the pair forces and the tableau rows, both in LDS.  Force evaluations are
// plain loops over the members, so the code stays small and nothing spills.
// ------------------------------------------------------------------------------------------

__device__ __forceinline__ double wave_max(double v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

// Neville factor 1 / ((n_k / n_(k-l))^2 - 1) for n_k = 2(k+1), written as p^2 / (q^2 - p^2)
// with q = k + 1, p = k + 1 - l: exact small integers and one rounding.
__device__ __forceinline__ double neville_c(int k, int l)
{
    const double q = (double)(k + 1), p = (double)(k + 1 - l);
    return (p * p) / (q * q - p * p);
}

// Members' data shared by the lanes of the group's wave.
struct BsShared {
    double pos[2][BS_LANES][4];                // positions published for the pair forces
    double m[BS_LANES];                        // member masses
    double i09[BS_LANES];                      // 1 / (0.9 r_crit)
    double i9l[LEVELS_MAX - 1][BS_LANES];      // hierarchical levels 1..nlev-1: the same of each
    int32_t test[BS_LANES];                    // member is a test body (TP2)
    int32_t nlev;                              // symplectic levels (1: the plain step)
};

// This lane's member: its constants and which lanes hold its partners' positions.
struct BsMember {
    int a, nb, base; // member index, group size, lane of member 0 in pos[]
    bool act, test;
    double mstar, i09;
};

template <int CTRL>
__device__ __forceinline__ double dpp64(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_MIRROR8 = 0x141; // quad_perm, row_half_mirror

// m (1 - K) / r^3 of a pair at squared separation q: the factor of its difference vector in the
// encounter force, zero outside r_crit,ab.  With LV (hierarchical levels) the weight is the
// product over levels 0..nlev-1 of (1 - K_k), so zero beyond the deepest level's radius (the
// radii do not grow with the level); ia / ib give the two members' 1 / (0.9 r_crit) of levels
// 1.. with the given stride.
//
// ALL (ia and ib in registers): every level there can be, those above nlev with 1 / (0.9 r_crit) = 0,
// which leaves the product as it is; a loop to nlev would index the arrays, that is, keep them in
// scratch memory (drifts in the levels of 40322
// bodies 108 -> 88 us).
template <bool LV, bool ALL = false>
__device__ __forceinline__ double encounter_factor(double q, double m, double i09, int nlev, const double *ia,
                                                   const double *ib, int stride)
{
    const double rq = inv_sqrt64(q), r = q * rq;
    const Changeover c = changeover_parts(r, i09);
    double u = c.u, d = c.d;
    if constexpr (LV)
#pragma unroll
        for (int k = 1; k < (ALL ? LEVELS_MAX : nlev); ++k) {
            const Changeover ck = changeover_parts(r, fmin(ia[(k - 1) * stride], ib[(k - 1) * stride]));
            u *= ck.u;
            d *= ck.d;
        }
    return m * (u * u) * inv64(d) * ((rq * rq) * rq);
}

// The forces at the positions z: the Kepler term about the Sun plus the (1 - K) share of the
// Newtonian forces from the other members (K of Chambers 1999 over [0.1, 1] r_crit,ab; two test
// bodies do not interact).  Every lane of the wave calls it.
template <bool LV, int NZ>
__device__ __forceinline__ void bs_forces(const BsMember &me, BsShared &S, int slot, const double (&z)[NZ][3],
                                          double (&f)[NZ][3])
{
#pragma unroll
    for (int s = 0; s < NZ; ++s)
        for (int q = 0; q < 3; ++q) S.pos[s][slot][q] = z[s][q];
    __syncthreads();
#pragma unroll
    for (int s = 0; s < NZ; ++s) {
        const double ri = inv_sqrt64(z[s][0] * z[s][0] + z[s][1] * z[s][1] + z[s][2] * z[s][2]);
        const double w = -me.mstar * (ri * ri) * ri;
        for (int q = 0; q < 3; ++q) f[s][q] = w * z[s][q];
    }
    // two independent terms at a time; the member itself and a second test body get mass zero
#pragma unroll(3 - NZ)
    for (int b = 0; b < me.nb; ++b) {
        const bool skip = b == me.a || (me.test && S.test[b]);
        const double mb = skip ? 0.0 : S.m[b], ib = fmin(me.i09, S.i09[b]);
#pragma unroll
        for (int s = 0; s < NZ; ++s) {
            const double dx = S.pos[s][me.base + b][0] - z[s][0];
            const double dy = S.pos[s][me.base + b][1] - z[s][1];
            const double dz = S.pos[s][me.base + b][2] - z[s][2];
            const double q = skip ? 1.0 : fma(dx, dx, fma(dy, dy, dz * dz));
            const double t = encounter_factor<LV>(q, mb, ib, S.nlev, &S.i9l[0][me.a], &S.i9l[0][b], BS_LANES);
            f[s][0] = fma(t, dx, f[s][0]);
            f[s][1] = fma(t, dy, f[s][1]);
            f[s][2] = fma(t, dz, f[s][2]);
        }
    }
    __syncthreads(); // the next call overwrites pos
}

// Groups of 3 to CP_MEM: lane (k, a) runs member a in extrapolation column k, two sub-steps a round
// (as in bs_pair).  When column k ends, its T(k, 0) go to LDS, and the wave forms T(k, k) -
// T(k, k-1) with one lane per state element, from the Lagrange form of the extrapolation
// (LAGRANGE).  tcol: LDS [BS_KMAX][6 CP_MEM]; ybuf: [6 CP_MEM].  (With a Neville row per column and
// one sub-step a round, and groups of three on a lane per column, the drift of 20040 bodies in TP2
// mode took 19.6 us, now 14.9; drifts in the levels of 40322 bodies 84 and 76.)
template <bool LV>
__device__ bool bs_columns(const BsMember &me, int k, int lane, BsShared &S, double *tcol, double *ybuf, double Y[6],
                           double dt, double tol)
{
    constexpr int E = 6 * CP_MEM;
    static_assert(E <= BS_LANES && CP_MEM == 8, "an element per lane, a member per lane of eight");
    const int slot = me.base + me.a, nsub = 2 * (k + 1);
    const int e = lane < 6 * me.nb ? lane : 0; // this lane's state element in the extrapolation
    const auto column = [&](int kk, const double *c) { // sum over columns 1..kk of c[j] (T(j, 0) - T(0, 0))
        double v[BS_KMAX], s = 0.0;
#pragma unroll
        for (int j = 0; j < BS_KMAX; ++j) v[j] = tcol[E * j + e];
#pragma unroll
        for (int j = 1; j < BS_KMAX; ++j)
            if (j <= kk) s = fma(c[j], v[j] - v[0], s);
        return s;
    };
    const auto members_max = [](double v) { // over the eight lanes of a column
        v = fmax(v, dpp64<DPP_XOR1>(v));
        v = fmax(v, dpp64<DPP_XOR2>(v));
        return fmax(v, dpp64<DPP_MIRROR8>(v));
    };
    double t = 0.0, H = dt;
    int attempts = 0;
    while (t < dt) {
        const bool last = H >= (dt - t) * (1.0 - 0x1p-30); // ends the interval (exactly)
        if (last) H = dt - t;
        if (H < dt * 0x1p-40 || ++attempts > 20000) return false;
        const double sr = members_max(me.act ? sqrt(Y[0] * Y[0] + Y[1] * Y[1] + Y[2] * Y[2]) : 0.0);
        const double sv = members_max(me.act ? sqrt(Y[3] * Y[3] + Y[4] * Y[4] + Y[5] * Y[5]) : 0.0);
        const double scale = e % 6 < 3 ? sr : sv;
        const double h = H / nsub, h2 = 2.0 * h;
        // z_i and z_i+1, u_i, u_i-1, i = 2 kk + 1
        double z[2][3], f[2][3], ui[3], up[3];
        {
            const double y0[1][3] = {{Y[0], Y[1], Y[2]}};
            double f0[1][3];
            bs_forces<LV, 1>(me, S, slot, y0, f0);
            for (int q = 0; q < 3; ++q) {
                up[q] = Y[3 + q];
                ui[q] = up[q] + h * f0[0][q];
                z[0][q] = Y[q] + h * up[q];
                z[1][q] = Y[q] + h2 * ui[q];
            }
        }
        int kstar = -1;
        double err_last = 0.0;
#pragma unroll 1
        for (int kk = 0; kk < BS_KMAX; ++kk) {
            bs_forces<LV, 2>(me, S, slot, z, f);
            double un[3]; // u_i+1
            for (int q = 0; q < 3; ++q) un[q] = up[q] + h2 * f[0][q];
            if (kk == k && me.act)
                for (int q = 0; q < 3; ++q) { // T(k, 0)
                    tcol[E * k + 6 * me.a + q] = 0.5 * (z[0][q] + z[1][q] + h * un[q]);
                    tcol[E * k + 6 * me.a + 3 + q] = 0.5 * (ui[q] + un[q] + h * f[1][q]);
                }
            for (int q = 0; q < 3; ++q) { // unused once kk >= k
                up[q] = un[q];
                ui[q] = ui[q] + h2 * f[1][q];
                z[0][q] = z[0][q] + h2 * un[q];
                z[1][q] = z[1][q] + h2 * ui[q];
            }
            if (kk == 0) continue;
            __syncthreads();
            const double diff = fabs(column(kk, LAGRANGE.d[kk]));
            if (!__ballot(!(diff <= tol * scale))) {
                kstar = kk;
                break;
            }
            if (kk == BS_KMAX - 1) err_last = wave_max(diff / scale);
        }
        if (kstar >= 0) {
            const double y = tcol[e] + column(kstar, LAGRANGE.w[kstar]);
            if (lane < 6 * me.nb) ybuf[lane] = y;
            __syncthreads(); // (tcol has been read, too)
            for (int q = 0; q < 6; ++q) Y[q] = ybuf[6 * (me.act ? me.a : 0) + q];
            t = last ? dt : t + H;
            if (kstar <= 4) H = 2.0 * H;
            else if (kstar == BS_KMAX - 1) H = 0.5 * H;
        } else {
            H = H * shrink_factor(err_last, tol);
        }
        __syncthreads(); // ybuf and tcol are rewritten
    }
    return true;
}

// Groups of CP_MEM + 1 .. BS_LANES members: one workgroup of BS_KMAX waves, wave k running
// extrapolation column k for every member, so the columns advance side by side, two sub-steps a
// round (as in bs_pair), and an attempt takes at most BS_KMAX + 1 rounds.  A member has P
// lanes (4 for groups of up to 16, 2 up to 32, else 1) that share its sources, sum every
// P-th one and add the parts in a fixed tree.  Column k completes with round k and
// extends each member's Neville row in place in LDS: it reads row k - 1, which column k - 1
// wrote the round before, and replaces it by row k, which column k + 1 reads the round
// after.  The tableau arithmetic and the accepted column (the first converged one) are those
// of the sequential scheme.  Latency bound: the barriers, and the chain of a round's forces (the
// launch of a dense annulus of 1000 bodies 137 us with one sub-step a round, 104 with two).
constexpr int WG_THREADS = BS_KMAX * BS_LANES;

struct BsWgShared {
    double pos[2][BS_KMAX][BS_LANES][3];       // each column's positions, for its pair forces
    double m[BS_LANES], i09[BS_LANES];
    double i9l[LEVELS_MAX - 1][BS_LANES];      // hierarchical levels 1..nlev-1
    double tab[BS_KMAX][6][BS_LANES];          // Neville rows, extended in place
    double err_last;                           // column BS_KMAX - 1's estimate
    int32_t test[BS_LANES];
    int32_t nlev;
    int32_t kstar, kstar_att;                  // converged column and the attempt it ended
};

// The forces of column k on part `part` of member a's P lanes at the positions z (when `on`), after
// a barrier that every thread of the workgroup reaches; the caller has another before the next call
// overwrites pos.
template <bool LV, int NZ>
__device__ void wg_forces(bool on, int k, int a, int part, int P, int nb, bool test, double mstar, double i09,
                          BsWgShared &S, const double (&z)[NZ][3], double (&f)[NZ][3])
{
    if (part == 0)
#pragma unroll
        for (int s = 0; s < NZ; ++s)
            for (int q = 0; q < 3; ++q) S.pos[s][k][a][q] = z[s][q];
    __syncthreads();
    if (!on) return;
#pragma unroll
    for (int s = 0; s < NZ; ++s) {
        const double ri = inv_sqrt64(z[s][0] * z[s][0] + z[s][1] * z[s][1] + z[s][2] * z[s][2]);
        const double w = part == 0 ? -mstar * (ri * ri) * ri : 0.0;
        for (int q = 0; q < 3; ++q) f[s][q] = w * z[s][q];
    }
    // first the partners inside r_crit,ab at either position, a bit each (in a chain of encounters
    // most members are farther apart), then only their terms, every lane its own (outside r_crit,ab
    // a term is zero)
    unsigned long long near = 0;
    for (int b = part, n = 0; b < nb; b += P, ++n) {
        const double i = fmin(i09, S.i09[b]);
        bool in = false;
#pragma unroll
        for (int s = 0; s < NZ; ++s) {
            const double dx = S.pos[s][k][b][0] - z[s][0];
            const double dy = S.pos[s][k][b][1] - z[s][1];
            const double dz = S.pos[s][k][b][2] - z[s][2];
            const double q = fma(dx, dx, fma(dy, dy, dz * dz));
            // r / (0.9 r_crit) < 10/9, with a margin for the rounding
            in |= (q * i) * i < 100.0 / 81.0 * (1.0 + 0x1p-40);
        }
        near |= (unsigned long long)(in && b != a && !(test && S.test[b])) << n;
    }
    while (near) {
        const int b = part + P * __builtin_ctzll(near);
        near &= near - 1;
        const double mb = S.m[b], ib = fmin(i09, S.i09[b]);
#pragma unroll
        for (int s = 0; s < NZ; ++s) {
            const double dx = S.pos[s][k][b][0] - z[s][0];
            const double dy = S.pos[s][k][b][1] - z[s][1];
            const double dz = S.pos[s][k][b][2] - z[s][2];
            const double q = fma(dx, dx, fma(dy, dy, dz * dz));
            const double t = encounter_factor<LV>(q, mb, ib, S.nlev, &S.i9l[0][a], &S.i9l[0][b], BS_LANES);
            f[s][0] = fma(t, dx, f[s][0]);
            f[s][1] = fma(t, dy, f[s][1]);
            f[s][2] = fma(t, dz, f[s][2]);
        }
    }
    for (int o = 1; o < P; o <<= 1)
#pragma unroll
        for (int s = 0; s < NZ; ++s)
            for (int q = 0; q < 3; ++q) f[s][q] += __shfl_xor(f[s][q], o, 64);
}

template <bool LV>
__device__ bool bs_workgroup(int k, int a, int part, int P, int nb, bool act, bool test, double mstar, double i09,
                             BsWgShared &S, double Y[6], double dt, double tol)
{
    const int nsub = 2 * (k + 1);
    const int lane = threadIdx.x & (BS_LANES - 1);
    double t = 0.0, H = dt;
    int attempts = 0;
    while (t < dt) {
        const bool last = H >= (dt - t) * (1.0 - 0x1p-30); // ends the interval (exactly)
        if (last) H = dt - t;
        if (H < dt * 0x1p-40 || ++attempts > 20000) return false;
        const double sr = wave_max(act ? sqrt(Y[0] * Y[0] + Y[1] * Y[1] + Y[2] * Y[2]) : 0.0);
        const double sv = wave_max(act ? sqrt(Y[3] * Y[3] + Y[4] * Y[4] + Y[5] * Y[5]) : 0.0);
        const double h = H / nsub, h2 = 2.0 * h;
        // z_i and z_i+1, u_i, u_i-1, i = 2 kk + 1 (as in bs_pair)
        double z[2][3], f[2][3] = {}, ui[3], up[3], T[6];
        {
            const double y0[1][3] = {{Y[0], Y[1], Y[2]}};
            double f0[1][3] = {};
            wg_forces<LV, 1>(act, k, a, part, P, nb, test, mstar, i09, S, y0, f0);
            for (int q = 0; q < 3; ++q) {
                up[q] = Y[3 + q];
                ui[q] = up[q] + h * f0[0][q];
                z[0][q] = Y[q] + h * up[q];
                z[1][q] = Y[q] + h2 * ui[q];
            }
            __syncthreads(); // the first round overwrites pos
        }
        int kstar = -1;
#pragma unroll 1
        for (int kk = 0; kk < BS_KMAX; ++kk) {
            wg_forces<LV, 2>(act && kk <= k, k, a, part, P, nb, test, mstar, i09, S, z, f);
            double un[3]; // u_i+1
            for (int q = 0; q < 3; ++q) un[q] = up[q] + h2 * f[0][q];
            if (kk < k) {
                for (int q = 0; q < 3; ++q) {
                    up[q] = un[q];
                    ui[q] = ui[q] + h2 * f[1][q];
                    z[0][q] = z[0][q] + h2 * un[q];
                    z[1][q] = z[1][q] + h2 * ui[q];
                }
            } else if (kk == k) {
                for (int q = 0; q < 3; ++q) { // T(k, 0)
                    T[q] = 0.5 * (z[0][q] + z[1][q] + h * un[q]);
                    T[3 + q] = 0.5 * (ui[q] + un[q] + h * f[1][q]);
                }
                // Neville: row k - 1 is replaced by row k in place (T(k, l-1) goes into slot
                // l-1 once T(k-1, l-1) has been read from it)
                double dp = 0.0, dv = 0.0;
#pragma unroll 1
                for (int l = 1; l <= k; ++l) {
                    const double c = neville_c(k, l);
                    double old[6];
                    for (int q = 0; q < 6; ++q) old[q] = S.tab[l - 1][q][a];
                    if (part == 0)
                        for (int q = 0; q < 6; ++q) S.tab[l - 1][q][a] = T[q];
                    for (int q = 0; q < 6; ++q) {
                        const double nx = T[q] + (T[q] - old[q]) * c;
                        if (l == k) {
                            if (q < 3) dp = fmax(dp, fabs(nx - T[q]));
                            else dv = fmax(dv, fabs(nx - T[q]));
                        }
                        T[q] = nx;
                    }
                }
                if (part == 0)
                    for (int q = 0; q < 6; ++q) S.tab[k][q][a] = T[q];
                if (k > 0) {
                    const double err = wave_max(act ? fmax(dp / sr, dv / sv) : 0.0);
                    if (lane == 0) {
                        if (err <= tol) {
                            S.kstar = k;
                            S.kstar_att = attempts;
                        }
                        if (k == BS_KMAX - 1) S.err_last = err;
                    }
                }
            }
            __syncthreads(); // the completed column's verdict; the next round overwrites pos
            if (S.kstar_att == attempts) {
                kstar = S.kstar;
                break;
            }
        }
        if (kstar >= 0) {
            for (int q = 0; q < 6; ++q) Y[q] = S.tab[kstar][q][a];
            t = last ? dt : t + H;
            if (kstar <= 4) H = 2.0 * H;
            else if (kstar == BS_KMAX - 1) H = 0.5 * H;
        } else {
            H = H * shrink_factor(S.err_last, tol);
        }
        __syncthreads(); // tab[kstar] and err_last are read before the next attempt writes them
    }
    return true;
}

// Groups of two (almost all groups when r_crit is a few Hill radii): lane 8k + s runs column k for
// one coordinate of one body, s = 0..3 the x, y, z and nothing of the first, 7..4 of the second,
// so that a coordinate's partner is the lane mirrored within its eight and a body's coordinates
// are a quad.  What a lane holds is a position and a velocity; a force evaluation is about 60
// instructions, of which the sums over a quad and the partner's coordinate are DPP moves.
// Latency bound (one wave per group, the slowest group sets the launch): with a column's whole
// state in one lane a pass was about 200 instructions and 1.1 us.
// (a + b) + (c + d) over the quad's lanes, the same in each of them
__device__ __forceinline__ double quad_sum(double v)
{
    v += dpp64<DPP_XOR1>(v);
    return v + dpp64<DPP_XOR2>(v);
}

struct PairGroup {
    double mstar, mp, i09;      // mp: the partner's mass, 0 between two test bodies
    double i9l[LEVELS_MAX - 1]; // hierarchical levels 1.., 0 above nlev - 1
};

template <bool LV>
__device__ __forceinline__ double pair_accel(const PairGroup &g, double z)
{
    const double dz = dpp64<DPP_MIRROR8>(z) - z;
    const double q0 = quad_sum(z * z), q1 = quad_sum(dz * dz);
    const double ri = inv_sqrt64(q0);
    // (two test bodies: a mass of zero at any separation; a branch here would keep the forces of a
    // round from running side by side)
    const double f = encounter_factor<LV, true>(g.mp != 0.0 ? q1 : 1.0, g.mp, g.i09, LEVELS_MAX, g.i9l, g.i9l, 1);
    return fma(f, dz, -g.mstar * (ri * ri) * ri * z);
}

// Sum over columns 1..k of c[j] (T(j, 0) - T(0, 0)) for one element (k wave-uniform): every
// load is issued before the first use.
__device__ __forceinline__ double pair_sum(const double *T, const double *c, int k)
{
    const double t0 = T[0];
    double v[BS_KMAX], s = 0.0;
#pragma unroll
    for (int j = 1; j < BS_KMAX; ++j) v[j] = T[16 * j];
#pragma unroll
    for (int j = 1; j < BS_KMAX; ++j)
        if (j <= k) s = fma(c[j], v[j] - t0, s);
    return s;
}

// x, v: this lane's coordinate, in every column's lanes; tcol: LDS [BS_KMAX][16], T(j, 0) of the
// positions (lanes 0..7) and velocities (8..15).
//
// A wave with a chain of some 25 dependent FP64 operations per force.  The midpoint rule is two
// leapfrogs that meet only at the end: positions at even sub-steps take the velocities at odd
// ones, and those the forces at even ones, so the forces at z_i and z_i+1, i = 2 j + 1, are
// independent and run side by side: after f(x) eight rounds an attempt instead of 16 (a drift of 40000
// bodies, set by a pair of 12 attempts: 57 -> 47 us).
template <bool LV>
__device__ bool bs_pair(const PairGroup &g, int lane, double &x, double &v, double *tcol, double dt, double tol)
{
    const int k = lane >> 3, nsub = 2 * (k + 1);
    double t = 0.0, H = dt;
    int attempts = 0;
    while (t < dt) {
        const bool last = H >= (dt - t) * (1.0 - 0x1p-30); // ends the interval (exactly)
        if (last) H = dt - t;
        if (H < dt * 0x1p-40 || ++attempts > 20000) return false;
        const double r1 = sqrt(quad_sum(x * x)), v1 = sqrt(quad_sum(v * v));
        const double sr = fmax(r1, dpp64<DPP_MIRROR8>(r1)), sv = fmax(v1, dpp64<DPP_MIRROR8>(v1));
        const double scale = lane & 8 ? sv : sr;
        const double h = H / nsub, h2 = 2.0 * h;
        // z_i, z_i+1, u_i, u_i-1 of every column
        double ui = fma(h, pair_accel<LV>(g, x), v), up = v;
        double zi = fma(h, v, x), zn = fma(h2, ui, x);
        int kstar = -1;
        double err_last = 0.0;
#pragma unroll 1
        for (int kk = 0; kk < BS_KMAX; ++kk) {
            const double ai = pair_accel<LV>(g, zi), an = pair_accel<LV>(g, zn);
            const double un = fma(h2, ai, up); // u_i+1
            if (kk == k) { // the column's last round
                tcol[16 * k + (lane & 7)] = 0.5 * (zi + zn + h * un); // T(k, 0)
                tcol[16 * k + 8 + (lane & 7)] = 0.5 * (ui + un + h * an);
            }
            ui = fma(h2, an, ui);
            up = un;
            zi = fma(h2, un, zi);
            zn = fma(h2, ui, zn);
            if (kk == 0) continue;
            __syncthreads();
            const double diff = fabs(pair_sum(tcol + (lane & 15), LAGRANGE.d[kk], kk));
            if (!__ballot(!(diff <= tol * scale))) {
                kstar = kk;
                break;
            }
            if (kk == BS_KMAX - 1) err_last = wave_max(diff / scale);
        }
        if (kstar >= 0) {
            x = tcol[lane & 7] + pair_sum(tcol + (lane & 7), LAGRANGE.w[kstar], kstar);
            v = tcol[8 + (lane & 7)] + pair_sum(tcol + 8 + (lane & 7), LAGRANGE.w[kstar], kstar);
            t = last ? dt : t + H;
            if (kstar <= 4) H = 2.0 * H;
            else if (kstar == BS_KMAX - 1) H = 0.5 * H;
        } else {
            H = H * shrink_factor(err_last, tol);
        }
        __syncthreads(); // every lane has read tcol
    }
    return true;
}

template <bool LV>
__device__ bool run_pair(const BsShared &S, int lane, double ms, double *x, double *y, double *z, double *vx,
                         double *vy, double *vz, const int32_t *mem, double *tcol, double dt, const double sh[3],
                         double p[3])
{
    const int s = lane & 7, body = s >> 2, c = body ? 7 - s : s; // coordinate c (3: none)
    PairGroup g;
    g.mstar = ms;
    g.mp = S.test[0] && S.test[1] ? 0.0 : S.m[1 - body];
    g.i09 = fmin(S.i09[0], S.i09[1]);
    if constexpr (LV)
#pragma unroll
        for (int l = 0; l + 1 < LEVELS_MAX; ++l) g.i9l[l] = l + 1 < S.nlev ? fmin(S.i9l[l][0], S.i9l[l][1]) : 0.0;
    const int b = mem[body];
    double *px = c == 0 ? x : c == 1 ? y : z, *pv = c == 0 ? vx : c == 1 ? vy : vz;
    double X = c < 3 ? px[b] + (c == 0 ? sh[0] : c == 1 ? sh[1] : sh[2]) : 0.0, V = c < 3 ? pv[b] : 0.0;
    const bool ok = bs_pair<LV>(g, lane, X, V, tcol, dt, 1e-12);
    const double mv = lane < 8 ? S.m[body] * V : 0.0;
    for (int q = 0; q < 3; ++q) p[q] = c == q ? mv : 0.0;
    if (lane < 8 && c < 3) {
        px[b] = X;
        pv[b] = V;
    }
    return ok;
}

// The first half of a Sun drift in the drift launches: tau P / Mstar of system s (zero without pm).
__device__ __forceinline__ void sun_shift_of(const StepMomentum &pm, const double *mstar, int s, double sh[3])
{
    sh[0] = sh[1] = sh[2] = 0.0;
    if (!pm.kick) return;
    double P[3];
    if (pm.n_large && pm.row_first[s + 1] - pm.row_first[s] > LARGE_ROWS)
        for (int q = 0; q < 3; ++q) P[q] = pm.sys_kick[3 * (size_t)s + q];
    else
        wave_momentum(pm.row_first, pm.kick, s, P);
    const double f = pm.tau / mstar[s];
    for (int q = 0; q < 3; ++q) sh[q] = f * P[q];
}

// A wave's lanes' momenta p summed into out[3 k ..].
__device__ __forceinline__ void store_momentum(double *out, int k, const double p[3])
{
    for (int q = 0; q < 3; ++q) {
        const double t = wave_sum(p[q]);
        if ((threadIdx.x & 63) == 0) out[3 * (size_t)k + q] = t;
    }
}

// The Sun drift's halves around a drift in parts: the shift from the sums that the kick left, and
// the sums for the shift after it, a wave per item.
__global__ __launch_bounds__(64) void sun_shift_items_kernel(const WorkItem *items, const double *mstar, double *x,
                                                             double *y, double *z, StepMomentum pm)
{
    const WorkItem w = items[blockIdx.x];
    const int lane = threadIdx.x, i = w.i0 + lane;
    double sh[3];
    sun_shift_of(pm, mstar, w.sys, sh);
    if (lane >= w.ni) return;
    x[i] += sh[0];
    y[i] += sh[1];
    z[i] += sh[2];
}

__global__ __launch_bounds__(64) void drifted_kernel(const WorkItem *items, const double *vx, const double *vy,
                                                     const double *vz, const double *m, StepMomentum pm)
{
    const WorkItem w = items[blockIdx.x];
    const int lane = threadIdx.x, i = w.i0 + lane;
    double p[3] = {0.0, 0.0, 0.0};
    if (lane < w.ni) {
        const double mi = m[i];
        p[0] = mi * vx[i];
        p[1] = mi * vy[i];
        p[2] = mi * vz[i];
    }
    store_momentum(pm.kepler, blockIdx.x, p);
    if (blockIdx.x == 0 && lane == 0) {
        *pm.clear = 0;
        *pm.group_n = 0;
    }
}

// The drift over dt: blocks [0, bs_blocks) integrate the encounter groups with Bulirsch-Stoer, the blocks after them Kepler-drift an item of up to 64 bodies each and skip the group
// members.  Each body is read and written by one block only.
template <bool LV>
__global__ __launch_bounds__(BS_LANES) __attribute__((amdgpu_waves_per_eu(2))) void drift_kernel(const int32_t *sys_of, const int32_t *sys_off,
                                                         const int32_t *n_massive, const double *mstar,
                                                         const WorkItem *items, int n_total, double *x, double *y,
                                                         double *z, double *vx, double *vy, double *vz,
                                                         const double *m, const double *rc, double dt,
                                                         const int32_t *members,
                                                         const int32_t *group_start,
                                                         const int32_t *n_groups, int32_t *member_slot,
                                                         int32_t *flags, int big_groups, int bs_blocks,
                                                         const double *rc_lv, int nlev, StepMomentum pm, int one_sys)
{
    // T(k, 0) of a group's state elements, and its state.  The block's LDS sets how many share a CU.
    __shared__ BsShared S;
    __shared__ double tab[BS_KMAX * CP_MEM * 6];
    __shared__ double ybuf[CP_MEM * 6];
    const int lane = threadIdx.x;
    double sh[3], p[3] = {0.0, 0.0, 0.0};
    if ((int)blockIdx.x >= bs_blocks) {
        const int it = blockIdx.x - bs_blocks;
        if (it == 0 && pm.group_n && lane == 0) {
            if (pm.clear) *pm.clear = 0;
            *pm.group_n = *n_groups;
        }
        const WorkItem w = items[it];
        const int i = w.i0 + lane;
        const bool on = lane < w.ni;
        const bool group = on && member_slot[i] >= 0;
        double Y[6] = {};
        if (on)
            for (int q = 0; q < 6; ++q) Y[q] = (q == 0 ? x : q == 1 ? y : q == 2 ? z : q == 3 ? vx : q == 4 ? vy : vz)[i];
        sun_shift_of(pm, mstar, w.sys, sh);
        if (group) member_slot[i] = -1; // integrated by its group's block; leave the slot clear
        if (on && !group) {
            for (int q = 0; q < 3; ++q) Y[q] += sh[q];
            if (!kepler_universal(Y[0], Y[1], Y[2], Y[3], Y[4], Y[5], mstar[w.sys], dt)) atomicOr(flags, FLAG_KEPLER);
            store_state(x, y, z, vx, vy, vz, i, Y);
            const double mi = m[i];
            for (int q = 0; q < 3; ++q) p[q] = mi * Y[3 + q];
        }
        if (pm.kepler) store_momentum(pm.kepler, it, p);
        return;
    }
    // the group's bounds are loaded beside the count (the array has room for every block's), and a
    // layout of one system looks up none
    const int g = blockIdx.x, k0 = group_start[g], k1 = group_start[g + 1];
    if (g >= *n_groups) return;
    const int nb = k1 - k0;
    const int sys = one_sys ? 0 : sys_of[members[k0]];
    const double ms = mstar[sys];
    if (pm.group && lane == 0) pm.group_sys[g] = sys;
    if (nb > BS_LANES && big_groups) return;       // integrated by the grid-wide path
    if (nb > CP_MEM && nb <= BS_LANES) return;     // a workgroup of drift_wg_kernel integrates it
    sun_shift_of(pm, mstar, sys, sh);
    p[0] = p[1] = p[2] = 0.0;
    if (nb > BS_LANES) {
        // larger than one wave: Kepler-drift the members instead and flag it
        if (lane == 0) atomicOr(flags, FLAG_CAPACITY);
        for (int k = lane; k < nb; k += BS_LANES) {
            const int b = members[k0 + k];
            double Y[6] = {x[b] + sh[0], y[b] + sh[1], z[b] + sh[2], vx[b], vy[b], vz[b]};
            if (!kepler_universal(Y[0], Y[1], Y[2], Y[3], Y[4], Y[5], ms, dt)) atomicOr(flags, FLAG_KEPLER);
            store_state(x, y, z, vx, vy, vz, b, Y);
            for (int q = 0; q < 3; ++q) p[q] += m[b] * Y[3 + q];
        }
        if (pm.group) store_momentum(pm.group, g, p);
        return;
    }
    if (lane < nb) {
        const int b = members[k0 + lane];
        S.m[lane] = m[b];
        S.i09[lane] = 1.0 / (0.9 * rc[b]);
        S.test[lane] = b - sys_off[sys] >= n_massive[sys];
        if constexpr (LV)
            for (int l = 1; l < nlev; ++l) S.i9l[l - 1][lane] = 1.0 / (0.9 * rc_lv[(size_t)(l - 1) * n_total + b]);
    }
    if (lane == 0) S.nlev = nlev;
    __syncthreads();
    bool ok;
    if (nb == 2) {
        ok = run_pair<LV>(S, lane, ms, x, y, z, vx, vy, vz, members + k0, tab, dt, sh, p);
    } else {
        const int k = lane / CP_MEM;
        BsMember me;
        me.a = lane % CP_MEM;
        me.nb = nb;
        me.base = k * CP_MEM;
        me.act = me.a < nb;
        const int ai = me.act ? me.a : 0;
        me.test = S.test[ai] != 0;
        me.mstar = ms;
        me.i09 = S.i09[ai];
        const int b = members[k0 + ai];
        double Y[6] = {x[b] + sh[0], y[b] + sh[1], z[b] + sh[2], vx[b], vy[b], vz[b]};
        ok = bs_columns<LV>(me, k, lane, S, tab, ybuf, Y, dt, 1e-12);
        // every lane has read its member's state before the first force evaluation's barrier
        if (me.act && k == 0) {
            store_state(x, y, z, vx, vy, vz, b, Y);
            for (int q = 0; q < 3; ++q) p[q] = S.m[ai] * Y[3 + q];
        }
    }
    if (!ok && lane == 0) atomicOr(flags, FLAG_NOCONVERGE);
    if (pm.group) store_momentum(pm.group, g, p);
}

__global__ __launch_bounds__(CE_THREADS) void wg_list_kernel(const int32_t *group_start, const int32_t *n_groups,
                                                             int32_t *list)
{
    __shared__ int32_t wsum[CE_THREADS / 64];
    list_wg_groups(group_start, *n_groups, list, wsum);
}

// The listed groups of CP_MEM + 1 .. BS_LANES members, one workgroup at a time each
// (bs_workgroup).
template <bool LV>
__global__ __launch_bounds__(WG_THREADS) void drift_wg_kernel(const int32_t *sys_of, const int32_t *sys_off,
                                                              const int32_t *n_massive, const double *mstar,
                                                              int n_total, double *x, double *y, double *z,
                                                              double *vx, double *vy, double *vz, const double *m,
                                                              const double *rc, double dt, const int32_t *members,
                                                              const int32_t *group_start, const int32_t *list,
                                                              int32_t *flags, const double *rc_lv, int nlev,
                                                              StepMomentum pm)
{
    __shared__ BsWgShared S;
    const int n_list = list[0];
    for (int li = blockIdx.x; li < n_list; li += gridDim.x) {
        const int g = list[1 + li];
        const int k0 = group_start[g], nb = group_start[g + 1] - k0;
        const int k = threadIdx.x / BS_LANES;
        const int P = nb <= 16 ? 4 : (nb <= 32 ? 2 : 1);
        const int a = (threadIdx.x % BS_LANES) / P, part = (threadIdx.x % BS_LANES) % P;
        const int sys = sys_of[members[k0]];
        const double ms = mstar[sys];
        double sh[3];
        sun_shift_of(pm, mstar, sys, sh);
        __syncthreads(); // the previous group's LDS is no longer read
        if (k == 0 && part == 0 && a < nb) {
            const int b = members[k0 + a];
            S.m[a] = m[b];
            S.i09[a] = 1.0 / (0.9 * rc[b]);
            S.test[a] = b - sys_off[sys] >= n_massive[sys];
            if constexpr (LV)
                for (int l = 1; l < nlev; ++l) S.i9l[l - 1][a] = 1.0 / (0.9 * rc_lv[(size_t)(l - 1) * n_total + b]);
        }
        if (threadIdx.x == 0) {
            S.nlev = nlev;
            S.kstar_att = 0;
        }
        __syncthreads();
        const bool act = a < nb;
        const int ai = act ? a : 0;
        const int b = members[k0 + ai];
        double Y[6] = {x[b] + sh[0], y[b] + sh[1], z[b] + sh[2], vx[b], vy[b], vz[b]};
        const bool ok = bs_workgroup<LV>(k, a, part, P, nb, act, S.test[ai] != 0, ms, S.i09[ai], S, Y, dt, 1e-12);
        // every thread has read its member's state before the first force evaluation's barrier
        const bool mine = act && k == 0 && part == 0;
        if (mine) store_state(x, y, z, vx, vy, vz, b, Y);
        if (!ok && threadIdx.x == 0) atomicOr(flags, FLAG_NOCONVERGE);
        if (pm.group && k == 0) {
            double p[3];
            for (int q = 0; q < 3; ++q) p[q] = mine ? S.m[a] * Y[3 + q] : 0.0;
            store_momentum(pm.group, g, p);
        }
    }
}

// skip: labels read, then reset to -1 (the list holds every body whose label is set)
__global__ __launch_bounds__(256) void kepler_list_kernel(const int32_t *sys_of, const double *mstar,
                                                          const int32_t *list, int n, int32_t *skip,
                                                          double *x, double *y, double *z, double *vx,
                                                          double *vy, double *vz, double dt, int32_t *flags)
{
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= n) return;
    const int i = list[k];
    if (skip) {
        const int s = skip[i];
        skip[i] = -1;
        if (s >= 0) return;
    }
    double Y[6] = {x[i], y[i], z[i], vx[i], vy[i], vz[i]};
    if (!kepler_universal(Y[0], Y[1], Y[2], Y[3], Y[4], Y[5], mstar[sys_of[i]], dt)) atomicOr(flags, FLAG_KEPLER);
    store_state(x, y, z, vx, vy, vz, i, Y);
}

} // namespace

hipError_t launch_kepler_list(const Layout &L, const int32_t *list, int32_t n, double *x, double *y,
                              double *z, double *vx, double *vy, double *vz, double dt, int32_t *flags,
                              hipStream_t stream, int32_t *skip)
{
    if (n <= 0) return hipSuccess;
    kepler_list_kernel<<<(n + 255) / 256, 256, 0, stream>>>(L.sys_of, L.mstar, list, n, skip, x, y, z, vx, vy, vz,
                                                            dt, flags);
    return hipGetLastError();
}

hipError_t launch_sun_drift(const Layout &L, double *x, double *y, double *z, const double *vx,
                            const double *vy, const double *vz, const double *m, double tau,
                            double *mom_part, hipStream_t stream)
{
    if (L.n_chunks == 0) return hipSuccess;
    momentum_kernel<<<L.n_chunks, SUN_THREADS, 0, stream>>>(L.chunks, m, vx, vy, vz, mom_part);
    sun_shift_kernel<<<L.n_chunks, SUN_THREADS, 0, stream>>>(L.chunks, L.chunk_first, L.mstar, mom_part,
                                                             tau, x, y, z);
    return hipGetLastError();
}

hipError_t launch_uf_union(const int32_t *pairs, const int32_t *pair_count, int32_t pair_cap, int32_t *lab,
                           hipStream_t stream)
{
    // (more threads lose more of their attempts to each other: the levels of a dense annulus of 40322
    // bodies 6.75 ms a step with 256 workgroups, 7.00 with 1024, 7.32 with 64)
    uf_union_kernel<<<256, 256, 0, stream>>>(pairs, pair_count, pair_cap, lab);
    return hipGetLastError();
}

// What a launch left in pm.kick or pm.kepler summed for the large systems.
static hipError_t large_sums(const StepMomentum &pm, bool kick, hipStream_t stream)
{
    if (pm.n_large > 0)
        large_sums_kernel<<<pm.n_large, CE_THREADS, 0, stream>>>(pm.large, kick ? pm.row_first : pm.item_first,
                                                                 kick ? pm.kick : pm.kepler,
                                                                 kick ? pm.sys_kick : pm.sys_kepler);
    return hipGetLastError();
}

static int import_blocks(const PairImport &p) { return std::max(1, std::min(256, (p.cap + CE_THREADS - 1) / CE_THREADS)); }

hipError_t launch_import_pairs(const PairImport &p, hipStream_t stream)
{
    drift_open_kernel<false><<<import_blocks(p), CE_THREADS, 0, stream>>>(nullptr, nullptr, nullptr, nullptr, nullptr,
                                                                   StepMomentum{}, p);
    import_finish_kernel<<<1, 64, 0, stream>>>(p);
    return hipGetLastError();
}

hipError_t launch_ce_groups(const GroupBuild &g, hipStream_t stream, const PairImport *import)
{
    ce_groups_kernel<<<1, CE_THREADS, 0, stream>>>(g, import ? *import : PairImport{});
    return hipGetLastError();
}

hipError_t launch_drift_open(const WorkItem *items, const double *vx, const double *vy, const double *vz,
                             const double *m, const StepMomentum &pm, const PairImport *import, hipStream_t stream)
{
    const int grid = pm.n_blocks + (import ? import_blocks(*import) : 0);
    (pm.small ? drift_open_kernel<true> : drift_open_kernel<false>)<<<grid, CE_THREADS, 0, stream>>>(
        items, vx, vy, vz, m, pm, import ? *import : PairImport{});
    return large_sums(pm, true, stream);
}

hipError_t launch_sun_shift(const WorkItem *items, int n_items, const double *mstar, double *x, double *y, double *z,
                            const StepMomentum &pm, hipStream_t stream)
{
    sun_shift_items_kernel<<<n_items, 64, 0, stream>>>(items, mstar, x, y, z, pm);
    return hipGetLastError();
}

hipError_t launch_drifted(const WorkItem *items, int n_items, const double *vx, const double *vy, const double *vz,
                          const double *m, const StepMomentum &pm, hipStream_t stream)
{
    drifted_kernel<<<n_items, 64, 0, stream>>>(items, vx, vy, vz, m, pm);
    return large_sums(pm, false, stream);
}

hipError_t launch_drift_close(const WorkItem *items, double *x, double *y, double *z, const StepMomentum &pm,
                              hipStream_t stream)
{
    (pm.small ? drift_close_kernel<true> : drift_close_kernel<false>)<<<pm.n_blocks, CE_THREADS, 0, stream>>>(
        items, x, y, z, pm);
    return hipGetLastError();
}

hipError_t launch_kick_close(const KickArgs &a, double *x, double *y, double *z, const StepMomentum &pm,
                             const GroupBuild *groups, hipStream_t stream)
{
    (pm.small ? kick_close_kernel<true> : kick_close_kernel<false>)<<<1 + pm.n_blocks, CE_THREADS, 0, stream>>>(
        a, x, y, z, pm, groups ? *groups : GroupBuild{}, groups != nullptr);
    return large_sums(pm, true, stream);
}

hipError_t launch_drift(const Layout &L, const WorkItem *items, int n_items, double *x, double *y, double *z,
                        double *vx, double *vy, double *vz, const double *m, const double *rc, double dt,
                        const int32_t *members, const int32_t *group_start, const int32_t *n_groups,
                        int32_t *member_slot, int32_t *flags, int big_groups, int bs_blocks, int32_t *wg_list,
                        hipStream_t stream, const double *rc_lv, int nlev, bool kepler, const DriftSide *side,
                        const StepMomentum *pm_in, bool wg_listed)
{
    if (L.n_total == 0) return hipSuccess;
    const StepMomentum pm = pm_in ? *pm_in : StepMomentum{};
    // bs_blocks 0: what the one-workgroup builder makes at most; < 0: no group blocks (the groups
    // are integrated elsewhere), only the Kepler drift of non-members.
    if (bs_blocks == 0) bs_blocks = CE_MAX_GROUPS;
    if (bs_blocks < 0) bs_blocks = 0;
    const int grid = bs_blocks + (kepler ? n_items : 0);
    if (grid == 0) return hipSuccess;
    auto kern = nlev > 1 ? drift_kernel<true> : drift_kernel<false>;
    auto wg = nlev > 1 ? drift_wg_kernel<true> : drift_wg_kernel<false>;
    // the groups of 9..64 members: listed, then one workgroup each (1024 workgroups, or the
    // largest number such groups can reach, walk the list); they run beside the launch of the
    // smaller groups on the side stream when there is one and nothing is being captured
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (side && side->stream && bs_blocks > 0) {
        const hipError_t e = hipStreamIsCapturing(stream, &cs);
        if (e != hipSuccess) return e;
    }
    const bool fork = side && side->stream && bs_blocks > 0 && cs == hipStreamCaptureStatusNone;
    const int wg_grid = std::max(1, std::min(1024, bs_blocks));
    hipError_t e = hipSuccess;
    if (bs_blocks > 0 && !wg_listed) wg_list_kernel<<<1, CE_THREADS, 0, stream>>>(group_start, n_groups, wg_list);
    if (fork) {
        if ((e = hipEventRecord(side->fork, stream)) != hipSuccess) return e;
        if ((e = hipStreamWaitEvent(side->stream, side->fork, 0)) != hipSuccess) return e;
        wg<<<wg_grid, WG_THREADS, 0, side->stream>>>(L.sys_of, L.sys_off, L.n_massive, L.mstar, L.n_total, x, y, z, vx,
                                                     vy, vz, m, rc, dt, members, group_start, wg_list, flags, rc_lv,
                                                     nlev, pm);
        if ((e = hipEventRecord(side->join, side->stream)) != hipSuccess) return e;
    }
    kern<<<grid, BS_LANES, 0, stream>>>(L.sys_of, L.sys_off, L.n_massive, L.mstar, items, L.n_total, x, y, z, vx, vy, vz,
                                        m, rc, dt, members, group_start, n_groups, member_slot, flags, big_groups,
                                        bs_blocks, rc_lv, nlev, pm, L.n_sys == 1);
    if (bs_blocks > 0 && !fork)
        wg<<<wg_grid, WG_THREADS, 0, stream>>>(L.sys_of, L.sys_off, L.n_massive, L.mstar, L.n_total, x, y, z, vx, vy, vz,
                                               m, rc, dt, members, group_start, wg_list, flags, rc_lv, nlev, pm);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (fork && (e = hipStreamWaitEvent(stream, side->join, 0)) != hipSuccess) return e;
    return large_sums(pm, false, stream);
}

} // namespace genga
