// Bulirsch-Stoer over dt for encounter groups larger than one wavefront.  In the
// encounter-dominated phase (Sect. 3.5: many planetesimals form almost one large close-encounter
// group and the run is bound by the Bulirsch-Stoer step) a group can hold most of a disc, so
// its state is spread over the whole GPU.  Method, tolerance and step control are those of
// the one-wave path and the oracle: modified midpoint with n_k = 2(k+1) sub-steps, polynomial
// extrapolation in h^2 (here in Lagrange form, relative to T(0,0)), acceptance at the first
// column k >= 1 whose estimate meets tol on the group's position / velocity scales, next step
// doubled / kept / halved, rejected steps shrunk by shrink_factor.
//
// One attempt is a fixed sequence of launches over all large groups at once: a force
// evaluation and midpoint update per sub-step (64 targets per workgroup), on the list path of
// several columns side by side, on the tile path of one column after another.  A group that has
// accepted a column, or reached dt, skips the rest.  The host repeats attempts until no group is
// active.
//
// The members of a group are ordered by ring and azimuth about the star (on the device, once per
// step), so a tile of 64 consecutive members is compact in space.  Each state buffer carries the
// bounding box of every tile, written by the launch that wrote the positions; a wave skips a
// source tile whose box is farther than the group's largest r_crit from the target tile's
// box, since no pair across the two can lie inside r_crit,ab.  The order only decides how
// much is skipped, never the result beyond rounding.
#include "genga_internal.h"
#include "pair_math.h"

namespace genga {

namespace {

using CD = const __attribute__((address_space(4))) double;
using CI = const __attribute__((address_space(4))) int32_t;

constexpr int GB_TILE = 64;
constexpr int GB_THREADS = 256;
// Up to this launch grid all eight columns of an attempt run side by side, above it the first six:
// 6600 bodies (104 tiles) 25.7 against 27.7 ms for two steps of some 40 attempts, 40322 bodies (631
// tiles) 16.4 against 15.4 ms a step (five first: 16.1).
constexpr int BIG_SIDE_TILES = 256;

__device__ __forceinline__ unsigned long long dbits(double v) { return (unsigned long long)__double_as_longlong(v); }
__device__ __forceinline__ double bitsd(unsigned long long b) { return __longlong_as_double((long long)b); }

// max into slot[g] for every lane with use = true: the lanes of the wave's first group
// combine first and one of them updates the slot; lanes of another group update their own.
// Every lane of the wave must call it.
__device__ __forceinline__ void wave_atomic_max(unsigned long long *slot, int g, bool use,
                                                unsigned long long v)
{
    const unsigned long long any = __ballot(use);
    if (!any) return;
    const int leader = __ffsll((long long)any) - 1;
    const int g0 = __shfl(g, leader, 64);
    const bool same = use && g == g0;
    unsigned long long m = same ? v : 0ull;
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long w = __shfl_xor(m, o, 64);
        m = w > m ? w : m;
    }
    if ((int)(threadIdx.x & 63) == leader) atomicMax(&slot[g0], m);
    if (use && !same) atomicMax(&slot[g], v);
}

// Per group: the step's start (t = 0, H = dt) and the star's mass; the largest squared
// candidate radius starts at 0 for big_setup_kernel's maxima.
__global__ __launch_bounds__(64) void big_setup_groups_kernel(BigBs b, const int32_t *sys_of, const double *mstar,
                                                              const int32_t *members, double dt)
{
    const int g = blockIdx.x * 64 + threadIdx.x;
    if (g >= b.dims[0]) return;
    if (g == 0) b.dtp[0] = dt;
    b.rcmax2[g] = 0.0;
    b.mstar[g] = mstar[sys_of[members[b.k0[g]]]];
    b.t[g] = 0.0;
    b.H[g] = dt;
    b.attempts[g] = 0;
    b.done[g] = 0;
    if (b.skin) {
        b.stale[g] = 0;
        b.keep[g] = 0;
    }
}

// Flat member f of large group g (one wave per tile): body index, constants, state
// Y[q * M + f], and the group's largest squared candidate radius (a maximum of bit patterns,
// which order non-negative doubles, so the result does not depend on the order of arrival).
__global__ __launch_bounds__(64) void big_setup_kernel(BigBs b, const int32_t *sys_of, const int32_t *sys_off,
                                                       const int32_t *n_massive, const double *x, const double *y,
                                                       const double *z, const double *vx, const double *vy,
                                                       const double *vz, const double *m, const double *rc,
                                                       const double *rc_lv, int n_total)
{
    const int4 tile = b.tiles[blockIdx.x];
    const int g = tile.x;
    const size_t M = (size_t)b.dims[1];
    double mx = 0.0;
    if ((int)threadIdx.x < tile.z) {
        const int f = tile.y + threadIdx.x, body = b.body[f], s = sys_of[body];
        b.grp[f] = g;
        b.rc[f] = rc[body];
        b.i09[f] = 1.0 / (0.9 * rc[body]);
        b.mass[f] = m[body];
        b.test[f] = body - sys_off[s] >= n_massive[s];
        b.Y[0 * M + f] = x[body];
        b.Y[1 * M + f] = y[body];
        b.Y[2 * M + f] = z[body];
        b.Y[3 * M + f] = vx[body];
        b.Y[4 * M + f] = vy[body];
        b.Y[5 * M + f] = vz[body];
        if (b.skin) {
            // every step starts from twice the bound's estimate, so a step's lists depend on its
            // starting state only (a run resumed from a saved state repeats them bit for bit)
            b.skin[body] = 2.0;
            b.crossed[f] = 0;
            b.amut[f] = 0.0;
            b.P[f].w = m[body];
        }
        // candidate radius: the deepest level's r_crit
        double rd = rc[body];
        for (int k = 1; k < b.nlev; ++k) {
            rd = rc_lv[(size_t)(k - 1) * n_total + body];
            b.rcl[(size_t)(k - 1) * b.cap_M + f] = rd;
            b.i9l[(size_t)(k - 1) * b.cap_M + f] = 1.0 / (0.9 * rd);
        }
        mx = sq_rn(rd);
    }
    for (int s = 32; s > 0; s >>= 1) mx = fmax(mx, __shfl_xor(mx, s, 64));
    if (threadIdx.x == 0) atomicMax(reinterpret_cast<unsigned long long *>(b.rcmax2) + g, dbits(mx));
}

// Start of an attempt, per group.
__global__ __launch_bounds__(64) void big_begin_kernel(BigBs b, int32_t *flags)
{
    const double dt = b.dtp[0];
    const int g = blockIdx.x * 64 + threadIdx.x;
    if (g >= b.dims[0] || b.done[g]) return;
    double H = b.H[g];
    const double t = b.t[g];
    const bool last = H >= (dt - t) * (1.0 - 0x1p-30); // ends the interval (exactly)
    if (last) H = dt - t;
    const int att = b.attempts[g] + 1;
    b.attempts[g] = att;
    if (b.skin) b.stale[g] = 0; // a void attempt is repeated with wider margins where they were crossed
    if (H < dt * 0x1p-40 || att > 20000) {
        atomicOr(flags, FLAG_NOCONVERGE);
        b.done[g] = 1;
        return;
    }
    b.H[g] = H;
    b.last[g] = last;
    b.acc[g] = -1;
    b.sr[g] = 0;
    b.sv[g] = 0;
    for (int k = 0; k < BS_KMAX; ++k) b.err[g * BS_KMAX + k] = 0;
}

// Position and velocity scales of each group: max |r|, max |v| over its members (max of
// non-negative doubles through their bit patterns, so the order of updates does not matter).
__global__ __launch_bounds__(GB_THREADS) void big_scale_kernel(BigBs b)
{
    const int f0 = blockIdx.x * GB_THREADS + threadIdx.x;
    const bool in = f0 < b.dims[1];
    const int f = in ? f0 : 0;
    const int g = b.grp[f];
    const bool use = in && !b.done[g];
    const size_t M = (size_t)b.dims[1];
    const double *Y = b.Y;
    const double rr = sqrt(sep2_rn(Y[f], Y[M + f], Y[2 * M + f]));
    const double vv = sqrt(sep2_rn(Y[3 * M + f], Y[4 * M + f], Y[5 * M + f]));
    wave_atomic_max(b.sr, g, use, dbits(rr));
    wave_atomic_max(b.sv, g, use, dbits(vv));
}

// Tile boxes of the attempt's starting state Y.
__global__ __launch_bounds__(64) void big_box_kernel(BigBs b)
{
    for (int me = blockIdx.x; me < b.dims[2]; me += gridDim.x) {
        const int4 tile = b.tiles[me];
        if (b.done[tile.x]) continue;
        const size_t M = (size_t)b.dims[1];
        const bool v = (int)threadIdx.x < tile.z;
        const int f = tile.y + (v ? (int)threadIdx.x : 0);
        tile_box(v, b.Y[f], b.Y[M + f], b.Y[2 * M + f], b.bb, me);
    }
}

// One sub-step of column k for the targets of a tile (one workgroup per tile): the (1 - K)
// share of the Newtonian forces from the group's other members at state Z, then
//   mode 0: OUT = Z + h f(Z)            (first sub-step, Z = Y)
//   mode 1: OUT = ZM + 2 h f(Z)         (OUT may be ZM's buffer: each lane rewrites its own)
//   mode 2: T(k, 0) = (ZM + Z + h f(Z)) / 2, into tcol[k]
// and, in modes 0 and 1, the tile's box in OUT's box array.  The workgroup first lists the
// source tiles in reach of the target tile (box gap within the largest r_crit); their
// quarters (16 members) are dealt out to the waves, so the few near tiles are spread over
// many waves.  Source positions and boxes come through scalar loads: neither is written by
// this launch.
template <bool LV, int W>
__device__ __forceinline__ void substep_tile(const BigBs &b, int me, int k, int mode, const double *Z,
                                             const double *ZM, double *OUT, const double *bbZ, double *bbOUT)
{
    __shared__ double red[3][W][GB_TILE];
    const int4 tile = b.tiles[me]; // (group, first member, count, -)
    const int g = tile.x;
    if (b.done[g] || b.acc[g] >= 0) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const size_t M = (size_t)b.dims[1];
    const int o = b.off[g], nb = b.off[g + 1] - o;
    const int tf = b.tfirst[g], nt = b.tfirst[g + 1] - tf;
    const bool valid = lane < tile.z;
    const int fa = tile.y + (valid ? lane : 0);
    const double xa = Z[fa], ya = Z[M + fa], za = Z[2 * M + fa];
    const bool testa = b.test[fa] != 0;
    // candidate radius: the group's largest r_crit^2, with a margin for the contracted r^2;
    // a source tile is skipped when the gap between the boxes exceeds it
    const double T = b.rcmax2[g] * (1.0 + 0x1p-40);
    const double Tcull = b.rcmax2[g] * (1.0 + 0x1p-30);
    CD *ZX = (CD *)Z;
    CD *ZY = (CD *)(Z + M);
    CD *ZZ = (CD *)(Z + 2 * M);
    CD *MS = (CD *)b.mass;
    CI *TS = (CI *)b.test;
    CD *BB = (CD *)bbZ;
    const double tlx = BB[me * 8 + 0], tly = BB[me * 8 + 1], tlz = BB[me * 8 + 2];
    const double thx = BB[me * 8 + 3], thy = BB[me * 8 + 4], thz = BB[me * 8 + 5];
    double ax = 0.0, ay = 0.0, az = 0.0;
    const double i09a = b.i09[fa];
    CD *I9 = (CD *)b.i09;
    // levels 1..nlev-1: the target's 1 / (0.9 radius), the sources' through scalar loads
    double i9al[LEVELS_MAX - 1] = {};
    CD *I9L = (CD *)b.i9l;
    if constexpr (LV)
        for (int l = 1; l < b.nlev; ++l) i9al[l - 1] = b.i9l[(size_t)(l - 1) * b.cap_M + fa];
    // the (1 - K) Newtonian terms of sources j .. j + cnt - 1 (cnt <= 4), side by side and
    // without branches: a pair outside r_crit,ab, the target itself and a test-test pair get
    // weight zero; the terms are added in source order
    auto pairs4 = [&](int j, int cnt, const double (&dx)[4], const double (&dy)[4], const double (&dz)[4],
                      const double (&q)[4]) {
        double t[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int jj = min(j + u, j + cnt - 1);
            const bool skip = u >= cnt || j + u == fa || (testa && TS[jj] != 0);
            const double qs = skip ? 1.0 : q[u];
            const double rq = inv_sqrt64(qs), r = qs * rq;
            const Changeover c0 = changeover_parts(r, fmin(i09a, I9[jj]));
            double uu = c0.u, dd = c0.d;
            if constexpr (LV) {
                // prod over the deeper levels of (1 - K_l): zero beyond the deepest radius
                for (int l = 1; l < b.nlev; ++l) {
                    const Changeover cl =
                        changeover_parts(r, fmin(i9al[l - 1], I9L[(size_t)(l - 1) * b.cap_M + jj]));
                    uu *= cl.u;
                    dd *= cl.d;
                }
            }
            t[u] = (skip ? 0.0 : MS[jj]) * (uu * uu) * inv64(dd) * ((rq * rq) * rq);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            ax = fma(t[u], dx[u], ax);
            ay = fma(t[u], dy[u], ay);
            az = fma(t[u], dz[u], az);
        }
    };
    // the source tiles in reach of this target tile, in tile order: one test per thread (in
    // passes of W * 64 tiles), then an ordered compaction (ballots within a wave, wave offsets
    // through LDS)
    __shared__ int near_tile[BIG_TILES_PER_GROUP];
    __shared__ int wave_cnt[W];
    int n_near = 0;
    for (int t0 = 0; t0 < nt; t0 += W * GB_TILE) {
        bool near = false;
        const int tt = t0 + (int)threadIdx.x;
        if (tt < nt) {
            const double *bs = bbZ + (size_t)(tf + tt) * 8;
            const double gx = fmax(0.0, fmax(bs[0] - thx, tlx - bs[3]));
            const double gy = fmax(0.0, fmax(bs[1] - thy, tly - bs[4]));
            const double gz = fmax(0.0, fmax(bs[2] - thz, tlz - bs[5]));
            near = (gx * gx + gy * gy) + gz * gz <= Tcull; // else no pair of the two tiles is close
        }
        const unsigned long long bal = __ballot(near);
        if (lane == 0) wave_cnt[wave] = __popcll(bal);
        __syncthreads();
        int base = n_near;
        for (int w = 0; w < W; ++w) {
            if (w < wave) base += wave_cnt[w];
            n_near += wave_cnt[w];
        }
        if (near) near_tile[base + __popcll(bal & ((1ull << lane) - 1))] = tt;
        __syncthreads();
    }
    // units of 16 sources (quarters of the near tiles), dealt out to the waves; whole quads
    // index the sources directly, so the four sources' words come in one scalar load per array
    for (int u = wave; u < 4 * n_near; u += W) {
        const int st = near_tile[u >> 2];
        const int jb = o + GB_TILE * st + 16 * (u & 3), je = min(jb + 16, o + nb);
        int j = jb;
        for (; j + 4 <= je; j += 4) {
            double dx[4], dy[4], dz[4], q[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                dx[v] = ZX[j + v] - xa;
                dy[v] = ZY[j + v] - ya;
                dz[v] = ZZ[j + v] - za;
                q[v] = fma(dx[v], dx[v], fma(dy[v], dy[v], dz[v] * dz[v]));
            }
            if (fmin(fmin(q[0], q[1]), fmin(q[2], q[3])) < T) pairs4(j, 4, dx, dy, dz, q);
        }
        if (j < je) {
            const int cnt = je - j;
            double dx[4], dy[4], dz[4], q[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int jj = min(j + v, je - 1);
                dx[v] = ZX[jj] - xa;
                dy[v] = ZY[jj] - ya;
                dz[v] = ZZ[jj] - za;
                q[v] = v < cnt ? fma(dx[v], dx[v], fma(dy[v], dy[v], dz[v] * dz[v])) : INFINITY;
            }
            if (fmin(fmin(q[0], q[1]), fmin(q[2], q[3])) < T) pairs4(j, cnt, dx, dy, dz, q);
        }
    }
    red[0][wave][lane] = ax;
    red[1][wave][lane] = ay;
    red[2][wave][lane] = az;
    __syncthreads();
    if (wave != 0) return;
    const double ri = inv_sqrt64(sep2_rn(xa, ya, za));
    const double s = -b.mstar[g] * (ri * ri) * ri;
    double d[6] = {Z[3 * M + fa], Z[4 * M + fa], Z[5 * M + fa], s * xa, s * ya, s * za};
    for (int w = 0; w < W; ++w) {
        d[3] += red[0][w][lane];
        d[4] += red[1][w][lane];
        d[5] += red[2][w][lane];
    }
    if (mode == 0 && k == 0 && valid && b.amut) {
        // the pair acceleration at the attempt's start, for the list path's bounds
        double px = 0.0, py = 0.0, pz = 0.0;
        for (int w = 0; w < W; ++w) {
            px += red[0][w][lane];
            py += red[1][w][lane];
            pz += red[2][w][lane];
        }
        b.amut[fa] = sqrt(sep2_rn(px, py, pz));
    }
    const double h = b.H[g] / (2 * (k + 1));
    if (mode == 2) {
        double tk[6];
        for (int q = 0; q < 6; ++q) tk[q] = 0.5 * (ZM[q * M + fa] + Z[q * M + fa] + h * d[q]);
        if (valid) {
            double *T0 = b.tcol + (size_t)k * 6 * M;
            for (int q = 0; q < 6; ++q) T0[q * M + fa] = tk[q];
        }
        if (k == 0) return;
        // the column's error estimate for this member (Lagrange form of T(k, k) - T(k, k-1),
        // relative to T(0, 0)) into the group's maximum: per position / velocity element over
        // the group's scales; a non-finite estimate is kept as the all-ones pattern
        double dp = 0.0, dv = 0.0;
        bool bad = false;
        for (int q = 0; q < 6; ++q) {
            const double t0 = b.tcol[q * M + fa];
            double sum = 0.0;
            for (int jj = 1; jj <= k; ++jj) {
                const double v = jj == k ? tk[q] : b.tcol[((size_t)jj * 6 + q) * M + fa];
                sum = fma(LAGRANGE.d[k][jj], v - t0, sum);
            }
            if (q < 3) dp = fmax(dp, fabs(sum));
            else dv = fmax(dv, fabs(sum));
            bad |= !(sum == sum);
        }
        const double e = fmax(dp / bitsd(b.sr[g]), dv / bitsd(b.sv[g]));
        wave_atomic_max(b.err + k, g * BS_KMAX, valid, (bad || !(e == e)) ? ~0ull : dbits(e));
        return;
    }
    double nx[6];
    for (int q = 0; q < 6; ++q) nx[q] = (mode == 0 ? Z[q * M + fa] : ZM[q * M + fa]) + (mode == 0 ? h : 2.0 * h) * d[q];
    if (valid)
        for (int q = 0; q < 6; ++q) OUT[q * M + fa] = nx[q];
    tile_box(valid, nx[0], nx[1], nx[2], bbOUT, me);
}

// The tiles are visited grid-stride, so that a launch can be sized to the layout at hand
// (the captured attempt is kept per grid size) rather than to the largest one.
template <bool LV, int W>
__global__ __launch_bounds__(GB_TILE *W) void big_substep_kernel(BigBs b, int k, int mode, const double *Z,
                                                                const double *ZM, double *OUT, const double *bbZ,
                                                                double *bbOUT)
{
    for (int me = blockIdx.x; me < b.dims[2]; me += gridDim.x) {
        if (me != (int)blockIdx.x) __syncthreads(); // the previous tile's LDS is free again
        substep_tile<LV, W>(b, me, k, mode, Z, ZM, OUT, bbZ, bbOUT);
    }
}


// ---------------------------------------------------------------------------------------------
// The list path.  At an attempt's start each member lists the sources that can come within
// r_crit,ab during the attempt.  The sub-step states of the modified midpoint method with step h
// under a constant pull A lie at Y + V tau + A (tau^2 - h^2) / 2 for odd j (tau = j h) and at
// Y + V tau + A tau^2 / 2 for even j; with A the star's pull at Y that is each member's
// prediction P_j, and S bounds its departure from it (the change of the star's pull along the
// path, the jerk 3 Mstar |V| / |Y|^3 over H^3 / 6, and the members' mutual pull a_mut over
// H^2 / 2, a_mut as the last force evaluation at an attempt's start found it (0 before the
// step's first), times the body's skin factor, at least 2).  A source is listed when the
// straight lines Y + V t of the two members come within
// r_crit,ab + S_a + S_b + |A_a - A_b| H^2 / 2 over [0, H]: then no unlisted pair can be inside
// r_crit,ab at a state where every member is within S of its prediction.  Every sub-step state
// checks |Z - P_j| <= S for every member; a crossed bound marks the group stale: the attempt is
// neither accepted nor counted as rejected, and the next one lists again, with four times the
// skin of each member that crossed its bound (bodies in close encounters, whose mutual pull the
// prediction leaves out, get wider margins for the rest of the step; every step starts at 2).
// The lists are in a fixed order, so the sums are deterministic.
// ---------------------------------------------------------------------------------------------

// The member's prediction constants: the star's pull A at Y and the bound S for step H.
struct ListMember {
    double ax, ay, az, s;
};

__device__ __forceinline__ ListMember list_member(double skin, double ms, double H, double x, double y, double z,
                                                  double u, double v, double w, double amut)
{
    const double r2 = sep2_rn(x, y, z);
    const double ri = inv_sqrt64(r2);
    const double a = ms / r2;                 // |A|
    const double c = -a * ri;                 // A = -Mstar Y / |Y|^3
    const double vv = sqrt(sep2_rn(u, v, w));
    ListMember m;
    m.ax = c * x;
    m.ay = c * y;
    m.az = c * z;
    m.s = skin * 0.5 * (a * ri * vv * H + amut) * (H * H);
    return m;
}

// Start of an attempt on the list path, one wave per tile: the positions of Y for the first round,
// the group's position and velocity scales (max |r|, max |v|: one atomic per workgroup whose
// tiles share a group, as 631 tiles' atomics on one address took 10 us), and, unless the lists
// still hold, the tile's boxes in position, velocity and A and the largest S of its members.
__global__ __launch_bounds__(GB_THREADS) void big_prepare_kernel(BigBs b)
{
    constexpr int NW = GB_THREADS / 64;
    __shared__ unsigned long long red[2][NW];
    __shared__ int grp[NW];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const size_t M = (size_t)b.dims[1];
    for (int m0 = blockIdx.x * NW; m0 < b.dims[2]; m0 += gridDim.x * NW) {
        const int me = m0 + wave;
        const bool tile_on = me < b.dims[2];
        const int4 tile = tile_on ? b.tiles[me] : make_int4(0, 0, 0, 0);
        const int g = tile.x;
        const bool on = tile_on && !b.done[g];
        const bool v = on && lane < tile.z;
        const int f = tile.y + (v ? lane : 0);
        const double H = b.H[g];
        const double x = b.Y[f], y = b.Y[M + f], z = b.Y[2 * M + f];
        const double u = b.Y[3 * M + f], vy = b.Y[4 * M + f], w = b.Y[5 * M + f];
        if (v) {
            double *p = reinterpret_cast<double *>(b.P + f);
            p[0] = x;
            p[1] = y;
            p[2] = z;
        }
        const double sr = wave_maxv(v ? sqrt(sep2_rn(x, y, z)) : 0.0);
        const double sv = wave_maxv(v ? sqrt(sep2_rn(u, vy, w)) : 0.0);
        if (lane == 0) {
            grp[wave] = on ? g : -1;
            red[0][wave] = dbits(sr);
            red[1][wave] = dbits(sv);
        }
        __syncthreads();
        if (threadIdx.x < 2) {
            // waves of one group in a row combine before the atomic
            unsigned long long *slot = threadIdx.x == 0 ? b.sr : b.sv;
            unsigned long long mx = 0;
            for (int k = 0; k < NW; ++k) {
                if (grp[k] < 0) continue;
                const unsigned long long t = red[threadIdx.x][k];
                mx = t > mx ? t : mx;
                if (k + 1 == NW || grp[k + 1] != grp[k]) {
                    atomicMax(&slot[grp[k]], mx);
                    mx = 0;
                }
            }
        }
        if (on && !b.keep[g]) {
            double sk = 2.0;
            if (v) {
                const int body = b.body[f];
                sk = b.skin[body];
                if (b.crossed[f]) { // the member left its bound in the last attempt: four times wider
                    sk *= 4.0;
                    b.skin[body] = sk;
                    b.crossed[f] = 0;
                }
            }
            const ListMember lm = list_member(sk, b.mstar[g], H, x, y, z, u, vy, w, v ? b.amut[f] : 0.0);
            if (v) b.pred[f] = make_double4(lm.ax, lm.ay, lm.az, lm.s);
            const double c[9] = {x, y, z, u, vy, w, lm.ax, lm.ay, lm.az};
            double lo[9], hi[9];
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                lo[q] = v ? c[q] : INFINITY;
                hi[q] = v ? c[q] : -INFINITY;
            }
            double ext = v ? lm.s : 0.0;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
                for (int q = 0; q < 9; ++q) {
                    lo[q] = fmin(lo[q], __shfl_xor(lo[q], off, 64));
                    hi[q] = fmax(hi[q], __shfl_xor(hi[q], off, 64));
                }
                ext = fmax(ext, __shfl_xor(ext, off, 64));
            }
            double *B = b.sbb + (size_t)me * BIG_BOX;
            if (lane == 0) {
#pragma unroll
                for (int q = 0; q < 9; ++q) {
                    B[q] = lo[q];
                    B[9 + q] = hi[q];
                }
                B[18] = ext;
            }
        }
        __syncthreads(); // red is rewritten by the next tiles
    }
}

// A body's words for the lists: the line from its state at the attempt's start, (A, S), the
// deepest level's radius.
struct ListBody {
    double x, y, z, u, v, w, r;
    double4 p;
};

// Whether the lines of target a and source j come within r = r_crit,ab + S_a + S_j
// + |A_a - A_j|_1 H^2 / 2 over [0, H] (the 1-norm bounds the length of the difference).  The
// minimum of |d + v t|^2 over [0, H] is taken without a division: at t = 0 when d.v >= 0, at t = H
// when -d.v >= |v|^2 H, else it is |d|^2 - (d.v)^2 / |v|^2, compared as
// (|d|^2 - r^2) |v|^2 < (d.v)^2.
__device__ __forceinline__ bool list_close(const ListBody &a, const ListBody &j, double H)
{
    const double dx = j.x - a.x, dy = j.y - a.y, dz = j.z - a.z;
    const double du = j.u - a.u, dv = j.v - a.v, dw = j.w - a.w;
    const double dd = sep2_rn(dx, dy, dz), vv = sep2_rn(du, dv, dw);
    const double dp = (dx * du + dy * dv) + dz * dw;
    const double r = fmax(a.r, j.r) + a.p.w + j.p.w +
                     0.5 * (fabs(j.p.x - a.p.x) + fabs(j.p.y - a.p.y) + fabs(j.p.z - a.p.z)) * (H * H);
    // a margin of 2^-30 covers the rounding of the distance
    const double r2 = r * r * (1.0 + 0x1p-30);
    if (dp >= 0.0 || vv == 0.0) return dd < r2;
    if (-dp >= vv * H) return sep2_rn(fma(du, H, dx), fma(dv, H, dy), fma(dw, H, dz)) < r2;
    return (dd - r2) * vv < dp * dp;
}

// A component of the separation of what lies in box B from what lies in box A, over [0, H], when
// both follow position + velocity t + A t^2 / 2: zero if the intervals meet, else their gap.
// lo / hi: bounds in position (p), velocity (v) and A (w).
__device__ __forceinline__ double gap_of(double alop, double ahip, double alov, double ahiv, double alow, double ahiw,
                                         double blop, double bhip, double blov, double bhiv, double blow, double bhiw,
                                         double H, double h2)
{
    const double lo = fma(fmin(blow - ahiw, 0.0), h2, fma(fmin(blov - ahiv, 0.0), H, blop - ahip));
    const double hi = fma(fmax(bhiw - alow, 0.0), h2, fma(fmax(bhiv - alov, 0.0), H, bhip - alop));
    return fmax(0.0, fmax(lo, -hi));
}

// The lists of a target tile's members, one workgroup of W waves per tile, in three passes that
// each leave the next one little: the source tiles (a thread each) whose boxes come within the
// largest radius and both largest S of the target tile's; of those, LIST_CAND at a time, the
// sources (a lane each) that do; and these, four at a time per wave through scalar loads, against
// the 64 members, as bits per member and tile in LDS.  The boxes bound the relative motion
// (neighbours move together: boxes swept by either tile alone let three times the tiles through).
// Then the source tiles with a bit become the tile's slots, in tile order (more than BIG_LIST_SLOTS
// void the attempt and send the step to the tile path), and the bits the members' lists, in order,
// as slot * 64 + the source's position in its tile.
//
// Bound by the arithmetic of the third pass (45 FP64 instructions a pair) on as many CUs as there
// are target tiles.  With one wave per tile and eighth of the source tiles, and a second launch
// that turned body lists into slot positions, 6600 bodies took 55 + 9 us an attempt and 40322
// bodies 136 + 19 (mean over attempts); now 27 and 76.  W = 16 up to BIG_SIDE_TILES target tiles, where only more
// waves per CU help; 8 beyond, two workgroups a CU.
constexpr int LIST_CAND = 32;

template <bool LV, int W>
__global__ __launch_bounds__(64 * W) void big_list_kernel(BigBs b)
{
    static_assert(BIG_LIST_SLOTS * 64 <= 65536, "16-bit slot positions");
    static_assert(LIST_CAND == 32 && LIST_CAND % W == 0, "a word of marks, whole shares per wave");
    constexpr int SH = LIST_CAND / W; // candidate tiles per wave
    __shared__ uint16_t cand[BIG_TILES_PER_GROUP];
    __shared__ unsigned long long bits[LIST_CAND][64]; // sources of a candidate tile that a member lists
    __shared__ uint16_t live[LIST_CAND * 64];          // (candidate, source) of the third pass
    __shared__ int cnt[W][64];                         // a member's entries, by wave
    __shared__ int wsum[W];
    __shared__ uint32_t used;
    CD *YA = (CD *)b.Y;
    CI *TS = (CI *)b.test;
    CD *PR = (CD *)b.pred; // (A, S) of member j at PR[4 j .. 4 j + 3]
    const int me = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (me >= b.dims[2]) return;
    const int4 tile = b.tiles[me];
    const int g = tile.x;
    if (b.done[g] || b.keep[g]) return; // the whole workgroup
    const size_t M = (size_t)b.dims[1];
    CD *RC = LV ? (CD *)(b.rcl + (size_t)(b.nlev - 2) * b.cap_M) : (CD *)b.rc; // the deepest level's radii
    const int o = b.off[g], nb = b.off[g + 1] - o;
    const int tf = b.tfirst[g], nt = b.tfirst[g + 1] - tf;
    const double H = b.H[g], h2 = 0.5 * H * H;
    CD *TB = (CD *)b.sbb + (size_t)me * BIG_BOX; // the target tile's boxes
    const bool valid = lane < tile.z;
    const int fa = tile.y + (valid ? lane : 0);
    const ListBody A = {b.Y[fa], b.Y[M + fa], b.Y[2 * M + fa], b.Y[3 * M + fa], b.Y[4 * M + fa], b.Y[5 * M + fa],
                        RC[fa], b.pred[fa]};
    const bool testa = b.test[fa] != 0;
    const double rmax = sqrt(b.rcmax2[g]) + TB[18];
    const auto near = [&](const double *lo, const double *hi, double ext) {
        double q = 0.0;
        for (int c = 0; c < 3; ++c) {
            const double gp = gap_of(TB[c], TB[9 + c], TB[3 + c], TB[12 + c], TB[6 + c], TB[15 + c], lo[c], hi[c],
                                     lo[3 + c], hi[3 + c], lo[6 + c], hi[6 + c], H, h2);
            q = fma(gp, gp, q);
        }
        const double cut = rmax + ext;
        return !(q > cut * cut * (1.0 + 0x1p-30));
    };
    // the positions of this thread's item in the order of waves and lanes, and the number of all
    const auto place = [&](bool is, int &n_all) {
        const unsigned long long bal = __ballot(is);
        if (lane == 0) wsum[wave] = __popcll(bal);
        __syncthreads();
        int pos = n_all + __popcll(bal & ((1ull << lane) - 1));
        for (int w = 0; w < W; ++w) {
            pos += w < wave ? wsum[w] : 0;
            n_all += wsum[w];
        }
        __syncthreads(); // wsum is rewritten by the next call
        return pos;
    };
    int n_cand = 0;
    for (int t0 = 0; t0 < nt; t0 += 64 * W) {
        const int tt = t0 + tid;
        bool is = false;
        if (tt < nt) {
            const double *B = b.sbb + (size_t)(tf + tt) * BIG_BOX;
            double w[19];
            for (int q = 0; q < 19; ++q) w[q] = B[q];
            is = near(w, w + 9, w[18]);
        }
        const int pos = place(is, n_cand);
        if (is) cand[pos] = (uint16_t)tt;
    }
    __syncthreads();
    int n_slots = 0, total = 0; // total: this lane's member's entries so far
    uint16_t *out = b.ll + (size_t)fa * BIG_LIST_CAP;
    for (int c0 = 0; c0 < n_cand; c0 += LIST_CAND) {
        const int nc = min(LIST_CAND, n_cand - c0);
        if (tid == 0) used = 0;
        int n_live = 0;
        for (int k = 0; k < SH; ++k) { // candidate k W + wave, source `lane`
            const int c = k * W + wave;
            bool is = false;
            if (c < nc) {
                bits[c][lane] = 0;
                const int s = 64 * cand[c0 + c] + lane;
                if (s < nb) {
                    const int j = o + s;
                    const double4 p = b.pred[j];
                    const double w[9] = {b.Y[j], b.Y[M + j], b.Y[2 * M + j], b.Y[3 * M + j], b.Y[4 * M + j], b.Y[5 * M + j],
                                         p.x, p.y, p.z};
                    is = near(w, w, p.w);
                }
            }
            const int pos = place(is, n_live);
            if (is) live[pos] = (uint16_t)(c * 64 + lane);
        }
        __syncthreads();
        for (int u = 4 * wave; u < n_live; u += 4 * W) {
            int e[4], j[4];
            ListBody S[4];
            bool T[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) { // (the last quad repeats its last source)
                e[q] = __builtin_amdgcn_readfirstlane(live[min(u + q, n_live - 1)]);
                j[q] = o + 64 * __builtin_amdgcn_readfirstlane(cand[c0 + (e[q] >> 6)]) + (e[q] & 63);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int jq = j[q];
                S[q] = {YA[jq], YA[M + jq], YA[2 * M + jq], YA[3 * M + jq], YA[4 * M + jq], YA[5 * M + jq], RC[jq],
                        make_double4(PR[4 * jq], PR[4 * jq + 1], PR[4 * jq + 2], PR[4 * jq + 3])};
                T[q] = TS[jq] != 0;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (valid && list_close(A, S[q], H) && j[q] != fa && !(testa && T[q]))
                    atomicOr(&bits[e[q] >> 6][lane], 1ull << (e[q] & 63));
        }
        __syncthreads();
        // this wave's share of the candidates: c = SH wave .. SH wave + SH - 1
        unsigned long long mine[SH];
        int n = 0;
        for (int k = 0; k < SH; ++k) {
            const int c = SH * wave + k;
            mine[k] = c < nc ? bits[c][lane] : 0;
            n += __popcll(mine[k]);
            if (__ballot(mine[k] != 0) && lane == 0) atomicOr(&used, 1u << c);
        }
        cnt[wave][lane] = n;
        __syncthreads();
        const uint32_t in = used;
        int at = total;
        for (int w = 0; w < W; ++w) {
            at += w < wave ? cnt[w][lane] : 0;
            total += cnt[w][lane];
        }
        for (int k = 0; k < SH; ++k) {
            const int c = SH * wave + k, slot = n_slots + __popc(in & ((1u << c) - 1));
            if (!(in >> c & 1) || slot >= BIG_LIST_SLOTS) continue;
            const int tt = cand[c0 + c];
            if (lane == 0) b.slot[me * BIG_LIST_SLOTS + slot] = make_int2(o + 64 * tt, min(64, nb - 64 * tt));
            for (unsigned long long q = mine[k]; q; q &= q - 1, ++at)
                if (at < BIG_LIST_CAP) out[at] = (uint16_t)(slot * 64 + __builtin_ctzll(q));
        }
        n_slots += __popc(in);
        __syncthreads(); // bits, cnt and used are rewritten by the next candidates
    }
    // a tile beyond the slots lists nothing (its attempt is void)
    if (wave == 0) {
        if (valid) b.ltot[fa] = n_slots <= BIG_LIST_SLOTS ? min(total, BIG_LIST_CAP) : 0;
        if ((__ballot(valid && total > BIG_LIST_CAP) || n_slots > BIG_LIST_SLOTS) && lane == 0) {
            atomicOr(b.ovf, 1);
            b.stale[g] = 1;
        }
        if (lane == 0) b.nslot[me] = min(n_slots, BIG_LIST_SLOTS);
    }
}

// Group g's acceptance once column k (>= 1) has been decided: its column if it is the first
// whose estimate meets tol, unless the attempt is void (a sub-step left the lists' bound).  On
// the list path every launch that needs the verdict takes it itself, from the same words, and
// one thread per group stores it in acc for the launches after it.
__device__ __forceinline__ int decided(const BigBs &b, int g, int k, double tol)
{
    const int a = b.acc[g];
    if (a >= 0 || k < 1 || b.done[g] || (b.skin && b.stale[g])) return a;
    const unsigned long long e = b.err[g * BS_KMAX + k];
    return (e != ~0ull && bitsd(e) <= tol) ? k : -1;
}

// Column kv's verdict for the launches after its last sub-step: true when the group has
// accepted it (or an earlier column), from the same words in every workgroup.  No workgroup of an
// accepted group goes on to write stale, so all of them agree; the group's first one stores acc.
__device__ __forceinline__ bool group_accepted(const BigBs &b, int g, int kv, double tol, bool store)
{
    const int a = b.acc[g], ka = kv < 0 ? a : decided(b, g, kv, tol);
    if (store && ka != a) b.acc[g] = ka;
    return ka >= 0;
}

// The list path's force at one position: the share (1 - K) of a source's pull, in parts.
struct BigPull {
    double x = 0.0, y = 0.0, z = 0.0;
};

// Round j of the columns k0, k0 + 1, .. (blockIdx.y) on the list path, one workgroup per target
// tile (blockIdx.x).  The midpoint rule is two leapfrogs that meet only at the end: positions at
// even sub-steps take the velocities at odd ones, and those the forces at even ones.  So with the
// state z_i, z_i+1, u_i, u_i-1 (i = 2 j + 1) the forces at z_i and z_i+1 are evaluated together:
//   u_i+1 = u_i-1 + 2 h f(z_i), u_i+2 = u_i + 2 h f(z_i+1), z_i+2 = z_i + 2 h u_i+1, z_i+3 = ..,
// or, in a column's last round (j = k), T(k, 0) and the group's error estimate.  The launch before
// the first round (FIRST) evaluates f(Y) once and writes z_1, u_1, z_2 of every column.  Positions
// are read by other tiles, so they alternate between two pairs of buffers; velocities are the
// member's own.  The records of the tile's slots are staged in LDS, then BIG_LIST_LANES lanes share
// a member, each summing every BIG_LIST_LANES-th entry of its list in order; the parts are added in
// a fixed tree whose result every lane has, so that the update's components (before the first
// round the columns) go to one lane each.
//
// Latency bound: two rounds of loads, a barrier, the list's chain of terms.  A launch per sub-step
// and column ran 104 tiles (6600 bodies) on 104 CUs for 6.6 us each, 72 of them an attempt; side by
// side the columns fill the chip, 17 launches of 9.2 us; two sub-steps a launch make it 9 of
// 13 us.  64 bytes per staged source: two workgroups fit a CU.
template <bool LV, bool FIRST>
__global__ __launch_bounds__(64 * BIG_LIST_LANES) __attribute__((amdgpu_waves_per_eu(4))) void big_round_kernel(
    BigBs b, int j, int k0, int kv, double tol)
{
    constexpr int P = BIG_LIST_LANES, NZ = FIRST ? 1 : 2; // positions evaluated
    constexpr int NS = BIG_LIST_SLOTS * 64;
    static_assert(P == BS_KMAX && P >= 6, "one lane per column, and per component");
    __shared__ double2 sxy[NZ][NS], szm[NZ][NS]; // (x, y), (z, mass or 1 / (0.9 r_crit))
    __shared__ double si9[FIRST ? NS : 1];
    __shared__ int sgi[LV ? NS : 1];               // member index, for the levels' radii
    __shared__ unsigned long long ered[P];         // the waves' error maxima
    constexpr int PER = NS / (64 * P); // staged sources per thread
    static_assert(NS % (64 * P) == 0, "whole rounds of staging");
    const size_t M = (size_t)b.dims[1], cm = (size_t)b.cap_M;
    const int me = blockIdx.x, k = k0 + (int)blockIdx.y, nsub = 2 * (k + 1);
    if (me >= b.dims[2]) return;
    // first round of loads: the tile, its slots
    const int4 tile = b.tiles[me];
    const int ns = b.nslot[me];
    int2 si[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) si[u] = b.slot[me * BIG_LIST_SLOTS + ((int)threadIdx.x + u * 64 * P) / 64];
    const int g = tile.x;
    const int m = (int)threadIdx.x / P, part = (int)threadIdx.x % P;
    const bool act = m < tile.z;
    const int fa = tile.y + (act ? m : 0);
    // second round: the group's state, the sources to stage and the member's own words
    if (b.done[g]) return; // the whole workgroup
    if (group_accepted(b, g, kv, tol, blockIdx.y == 0 && threadIdx.x == 0 && me == b.tfirst[g])) return;
    // z_i and z_i+1 of this round, and where the next round's go
    double4 *const Z0 = b.P + (FIRST ? 0 : 1 + 4 * k + 2 * (j & 1)) * cm, *const Z1 = Z0 + cm;
    double4 *const N0 = b.P + (1 + 4 * k + 2 * ((j + 1) & 1)) * cm, *const N1 = N0 + cm;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int e = (int)threadIdx.x + u * 64 * P;
        if (e < ns * 64 && (e & 63) < si[u].y) {
            const size_t f = (size_t)(si[u].x + (e & 63));
            const double4 p = Z0[f];
            sxy[0][e] = make_double2(p.x, p.y);
            szm[0][e] = make_double2(p.z, p.w);
            if constexpr (FIRST) {
                si9[e] = b.i09[f];
            } else {
                const double4 q = Z1[f];
                sxy[NZ - 1][e] = make_double2(q.x, q.y);
                szm[NZ - 1][e] = make_double2(q.z, q.w);
            }
            if constexpr (LV) sgi[e] = (int)f;
        }
    }
    double4 pa[NZ];
    pa[0] = Z0[fa];
    if constexpr (!FIRST) pa[NZ - 1] = Z1[fa];
    const double i09a = FIRST ? b.i09[fa] : pa[NZ - 1].w;
    const int tot = b.ltot[fa];
    const uint16_t *L = b.ll + (size_t)fa * BIG_LIST_CAP;
    int l0 = L[part], l1 = L[part + P]; // the first two positions (used only below tot)
    // this lane's component (part < 6: x, y, z of the positions, then of the velocities): u_i, u_i-1
    const int c = part % 3;
    double *const U0 = b.V + ((size_t)(2 * k) * 3 + c) * cm + fa, *const U1 = U0 + 3 * cm;
    const double ui = FIRST ? 0.0 : *U0, up = FIRST ? 0.0 : j == 0 ? b.Y[(3 + c) * M + fa] : *U1;
    __syncthreads();
    BigPull f[NZ];
    const double H = b.H[g], h = H / nsub;
    if (act) {
        // the bound of the lists: every member stays within S of its prediction
        if (!FIRST && part >= P - 2) {
            const int z = part - (P - 2), i = 2 * j + 1 + z;
            const double tau = h * i;
            const double4 pm = b.pred[fa];
            const double h2 = 0.5 * (tau * tau - ((i & 1) ? h * h : 0.0));
            const double px = fma(pm.x, h2, fma(b.Y[3 * M + fa], tau, b.Y[fa]));
            const double py = fma(pm.y, h2, fma(b.Y[4 * M + fa], tau, b.Y[M + fa]));
            const double pz = fma(pm.z, h2, fma(b.Y[5 * M + fa], tau, b.Y[2 * M + fa]));
            const double4 at = z ? pa[NZ - 1] : pa[0];
            if (!(sep2_rn(at.x - px, at.y - py, at.z - pz) <= pm.w * pm.w * (1.0 - 0x1p-30))) {
                b.stale[g] = 1;
                b.crossed[fa] = 1;
            }
        }
        const auto term = [&](int l) {
            double2 xy[NZ], zw[NZ];
#pragma unroll
            for (int z = 0; z < NZ; ++z) {
                xy[z] = sxy[z][l];
                zw[z] = szm[z][l];
            }
            const double mj = zw[0].y, i9 = fmin(i09a, FIRST ? si9[l] : zw[NZ - 1].y);
#pragma unroll
            for (int z = 0; z < NZ; ++z) {
                const double dx = xy[z].x - pa[z].x, dy = xy[z].y - pa[z].y, dz = zw[z].x - pa[z].z;
                const double q = fma(dx, dx, fma(dy, dy, dz * dz));
                const double rq = inv_sqrt64(q), r = q * rq;
                // the lists hold neither the member itself nor two test bodies, and outside
                // r_crit,ab the weight is zero
                const Changeover c0 = changeover_parts(r, i9);
                double u = c0.u, dd = c0.d;
                if constexpr (LV) {
                    const int fj = sgi[l];
                    for (int lv = 1; lv < b.nlev; ++lv) {
                        const Changeover cl = changeover_parts(r, fmin(b.i9l[(size_t)(lv - 1) * b.cap_M + fa],
                                                                       b.i9l[(size_t)(lv - 1) * b.cap_M + fj]));
                        u *= cl.u;
                        dd *= cl.d;
                    }
                }
                const double s = mj * (u * u) * inv64(dd) * ((rq * rq) * rq);
                f[z].x = fma(s, dx, f[z].x);
                f[z].y = fma(s, dy, f[z].y);
                f[z].z = fma(s, dz, f[z].z);
            }
        };
        // lane `part` sums every P-th entry from `part` on, in order; the positions of the next
        // two are loaded ahead (past the end: entry 0, unused)
        const auto entry = [&](int e) { return (int)L[e < tot ? e : 0]; };
        for (int e = part; e < tot; e += P) {
            const int l = l0;
            l0 = l1;
            l1 = entry(e + 2 * P);
            term(l);
        }
    }
    // the parts of a member, in a fixed order
    for (int off = P / 2; off > 0; off >>= 1)
#pragma unroll
        for (int z = 0; z < NZ; ++z) {
            f[z].x += __shfl_xor(f[z].x, off, 64);
            f[z].y += __shfl_xor(f[z].y, off, 64);
            f[z].z += __shfl_xor(f[z].z, off, 64);
        }
    if (FIRST && act && part == 0) b.amut[fa] = sqrt(sep2_rn(f[0].x, f[0].y, f[0].z));
#pragma unroll
    for (int z = 0; z < NZ; ++z) {
        const double ri = inv_sqrt64(sep2_rn(pa[z].x, pa[z].y, pa[z].z));
        const double s = -b.mstar[g] * (ri * ri) * ri;
        f[z].x = s * pa[z].x + f[z].x;
        f[z].y = s * pa[z].y + f[z].y;
        f[z].z = s * pa[z].z + f[z].z;
    }
    if constexpr (FIRST) {
        if (!act) return;
        // lane `part`: z_1, u_1 and z_2 of column `part`
        const double hc = H / (2 * (part + 1));
        double *p1 = reinterpret_cast<double *>(b.P + (1 + 4 * part) * cm + fa);
        double *p2 = reinterpret_cast<double *>(b.P + (2 + 4 * part) * cm + fa);
        double *v = b.V + (size_t)(2 * part) * 3 * cm + fa;
        const double y0[3] = {pa[0].x, pa[0].y, pa[0].z}, a0[3] = {f[0].x, f[0].y, f[0].z};
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const double u0 = b.Y[(3 + q) * M + fa], u1 = u0 + hc * a0[q];
            p1[q] = y0[q] + hc * u0;
            p2[q] = y0[q] + 2.0 * hc * u1;
            v[q * cm] = u1;
        }
        p1[3] = pa[0].w;
        p2[3] = i09a;
        return;
    }
    // this lane's component
    const double zi = c == 0 ? pa[0].x : c == 1 ? pa[0].y : pa[0].z;
    const double zn = c == 0 ? pa[NZ - 1].x : c == 1 ? pa[NZ - 1].y : pa[NZ - 1].z;
    const double ai = c == 0 ? f[0].x : c == 1 ? f[0].y : f[0].z;
    const double an = c == 0 ? f[NZ - 1].x : c == 1 ? f[NZ - 1].y : f[NZ - 1].z;
    const double un = up + 2.0 * h * ai; // u_i+1
    if (j < k) {
        if (!act) return;
        const double u2 = ui + 2.0 * h * an; // u_i+2
        if (part < 3) {
            reinterpret_cast<double *>(N0 + fa)[c] = zi + 2.0 * h * un;
            reinterpret_cast<double *>(N1 + fa)[c] = zn + 2.0 * h * u2;
        } else if (part < 6) {
            *U0 = u2;
            *U1 = un;
        } else if (part == 6 && j < 2) { // (later rounds find them there)
            N0[fa].w = pa[0].w;
            N1[fa].w = pa[NZ - 1].w;
        }
        return;
    }
    const double tk = part < 3 ? 0.5 * (zi + zn + h * un) : 0.5 * (ui + un + h * an);
    const bool use = act && part < 6;
    double *T0 = b.tcol + part * M + fa; // T(j, 0) of this component: T0[6 j M]
    if (use) T0[(size_t)k * 6 * M] = tk;
    if (k == 0) return;
    // the column's error estimate (Lagrange form of T(k, k) - T(k, k-1), relative to T(0, 0)):
    // per position / velocity element over the group's scales; a non-finite one is kept as the
    // all-ones pattern.  One atomic per workgroup, and only where it would raise the maximum.
    unsigned long long e = 0;
    if (use) {
        const double tz = T0[0];
        double tv[BS_KMAX], sum = 0.0;
#pragma unroll
        for (int q = 1; q < BS_KMAX; ++q) tv[q] = T0[(size_t)(q < k ? q : 0) * 6 * M];
#pragma unroll
        for (int q = 1; q < BS_KMAX; ++q)
            if (q <= k) sum = fma(LAGRANGE.d[k][q], (q == k ? tk : tv[q]) - tz, sum);
        const double err = fabs(sum) / bitsd(part < 3 ? b.sr[g] : b.sv[g]);
        e = err == err ? dbits(err) : ~0ull;
    }
    for (int off = 32; off > 0; off >>= 1) {
        const unsigned long long w = __shfl_xor(e, off, 64);
        e = w > e ? w : e;
    }
    if ((threadIdx.x & 63) == 0) ered[threadIdx.x >> 6] = e;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < P; ++w) e = ered[w] > e ? ered[w] : e;
    unsigned long long *slot = b.err + g * BS_KMAX + k;
    if (e > __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(slot, e);
}

__global__ __launch_bounds__(64) void big_decide_kernel(BigBs b, int k, double tol)
{
    const int g = blockIdx.x * 64 + threadIdx.x;
    if (g >= b.dims[0] || b.done[g] || b.acc[g] >= 0) return;
    if (b.skin && b.stale[g]) return; // a sub-step left the list's bound: no column counts
    const unsigned long long e = b.err[g * BS_KMAX + k];
    if (e != ~0ull && bitsd(e) <= tol) b.acc[g] = k;
}

// Accepted groups: Y = T(k*, k*) (the last column's verdict taken here).
__global__ __launch_bounds__(GB_THREADS) void big_accept_kernel(BigBs b, double tol)
{
    const int f = blockIdx.x * GB_THREADS + threadIdx.x;
    if (f >= b.dims[1]) return;
    const int g = b.grp[f];
    const int ks = decided(b, g, BS_KMAX - 1, tol);
    if (f == b.off[g] && ks != b.acc[g]) b.acc[g] = ks;
    if (b.done[g] || ks < 0) return;
    const size_t M = (size_t)b.dims[1];
    for (int q = 0; q < 6; ++q) {
        // every row's load in flight at once (rows above ks: T(0, 0) again, unused)
        const double t0 = b.tcol[q * M + f];
        double t[BS_KMAX], s = 0.0;
#pragma unroll
        for (int j = 1; j < BS_KMAX; ++j) t[j] = b.tcol[((size_t)(j <= ks ? j : 0) * 6 + q) * M + f];
#pragma unroll
        for (int j = 1; j < BS_KMAX; ++j)
            if (j <= ks) s = fma(LAGRANGE.w[ks][j], t[j] - t0, s);
        b.Y[q * M + f] = t0 + s;
    }
}

// Step control per group, and to the host the number of groups still short of dt, whether lists
// overflowed, and how many attempts the slowest group still needs at least (each step at most
// twice the one before it: the host enqueues that many without looking).
__global__ __launch_bounds__(GB_THREADS) void big_control_kernel(BigBs b, double tol,
                                                                 int32_t *flags)
{
    __shared__ int cnt[GB_THREADS / 64], need[GB_THREADS / 64];
    const double dt = b.dtp[0];
    int active = 0, least = 0;
    for (int g = threadIdx.x; g < b.dims[0]; g += GB_THREADS) {
        if (b.done[g]) continue;
        if (b.skin && b.stale[g]) { // a void attempt: the same step again (with wider lists)
            b.keep[g] = 0;
            ++active;
            least = max(least, 1);
            continue;
        }
        const int ks = decided(b, g, BS_KMAX - 1, tol);
        // a rejected attempt leaves Y and the skins as they were and only shortens the step: the
        // next attempt keeps its lists (the prediction and its bound hold over any shorter step)
        if (b.skin) b.keep[g] = ks < 0;
        if (ks >= 0) {
            const double t = b.last[g] ? dt : b.t[g] + b.H[g];
            b.t[g] = t;
            if (ks <= 4) b.H[g] = 2.0 * b.H[g];
            else if (ks == BS_KMAX - 1) b.H[g] = 0.5 * b.H[g];
            if (!(t < dt)) b.done[g] = 1;
        } else {
            const unsigned long long e = b.err[g * BS_KMAX + BS_KMAX - 1];
            if (e == ~0ull) { // non-finite estimate: give up on this group
                atomicOr(flags, FLAG_NOCONVERGE);
                b.done[g] = 1;
            } else {
                b.H[g] = b.H[g] * shrink_factor(bitsd(e), tol);
            }
        }
        if (!b.done[g]) {
            ++active;
            // H + 2 H + .. + 2^(n-1) H reaches dt - t
            int n = 1;
            const double rest = (dt - b.t[g]) * (1.0 - 0x1p-30);
            for (double h = b.H[g], sum = h; sum < rest && n < BIG_AHEAD; ++n) {
                h *= 2.0;
                sum += h;
            }
            least = max(least, n);
        }
    }
    for (int s = 32; s > 0; s >>= 1) {
        active += __shfl_xor(active, s, 64);
        least = max(least, __shfl_xor(least, s, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        cnt[threadIdx.x >> 6] = active;
        need[threadIdx.x >> 6] = least;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int total = 0;
        for (int w = 0; w < GB_THREADS / 64; ++w) {
            total += cnt[w];
            least = max(least, need[w]);
        }
        b.status[0] = total;
        b.status[1] = *b.ovf;
        b.status[2] = least;
    }
}

__global__ __launch_bounds__(GB_THREADS) void big_finish_kernel(BigBs b, double *x, double *y, double *z,
                                                                double *vx, double *vy, double *vz)
{
    const int f = blockIdx.x * GB_THREADS + threadIdx.x;
    if (f >= b.dims[1]) return;
    const size_t M = (size_t)b.dims[1];
    const int body = b.body[f];
    x[body] = b.Y[f];
    y[body] = b.Y[M + f];
    z[body] = b.Y[2 * M + f];
    vx[body] = b.Y[3 * M + f];
    vy[body] = b.Y[4 * M + f];
    vz[body] = b.Y[5 * M + f];
}

} // namespace

hipError_t launch_big_setup(const Layout &L, const BigBs &b, const int32_t *members, const double *x,
                            const double *y, const double *z, const double *vx, const double *vy,
                            const double *vz, const double *m, const double *rc, const double *rc_lv,
                            double dt, hipStream_t stream)
{
    if (b.G == 0) return hipSuccess;
    big_setup_groups_kernel<<<(b.G + 63) / 64, 64, 0, stream>>>(b, L.sys_of, L.mstar, members, dt);
    big_setup_kernel<<<b.n_tiles, 64, 0, stream>>>(b, L.sys_of, L.sys_off, L.n_massive, x, y, z, vx, vy, vz, m, rc,
                                                   rc_lv, L.n_total);
    return hipGetLastError();
}

hipError_t launch_big_attempt(const BigBs &b, double tol, int32_t *flags, int tile_grid, int waves,
                              hipStream_t stream)
{
    // grids for the largest layout: launches past the current one (sizes in b.dims) return at
    // once, so one captured sequence serves every step
    const int gg = (b.cap_G + 63) / 64, gm = (b.cap_M + GB_THREADS - 1) / GB_THREADS;
    const int nt = std::max(1, std::min(tile_grid, b.cap_T));
    const size_t M6 = 6 * (size_t)b.cap_M;
    double *buf[3] = {b.Y, b.Y + M6, b.Y + 2 * M6};           // Y, B1, B2
    double *box[3] = {b.bb, b.bb + 8 * (size_t)b.cap_T, b.bb + 16 * (size_t)b.cap_T};
    // waves per target tile: 16 while the tiles fit the chip in one round of workgroups, fewer
    // (more workgroups per CU, more sources per wave) for larger layouts
    if (waves != 8 && waves != 16) return hipErrorInvalidValue;
    const bool lv = b.nlev > 1;
    auto substep = waves == 16 ? (lv ? big_substep_kernel<true, 16> : big_substep_kernel<false, 16>)
                               : (lv ? big_substep_kernel<true, 8> : big_substep_kernel<false, 8>);
    big_begin_kernel<<<gg, 64, 0, stream>>>(b, flags);
    big_scale_kernel<<<gm, GB_THREADS, 0, stream>>>(b);
    big_box_kernel<<<nt, 64, 0, stream>>>(b);
    for (int k = 0; k < BS_KMAX; ++k) {
        const int nsub = 2 * (k + 1);
        // sub-step i reads zc_i and zm_i and writes zc_(i+1): zc_1 = B1 (zm_1 = Y), then the
        // new point goes into zm's buffer, B2 first
        substep<<<nt, GB_TILE * waves, 0, stream>>>(b, k, 0, buf[0], buf[0], buf[1], box[0], box[1]);
        int zc = 1, zm = 0;
        for (int i = 1; i < nsub; ++i) {
            const int out = zm == 0 ? 2 : zm;
            substep<<<nt, GB_TILE * waves, 0, stream>>>(b, k, 1, buf[zc], buf[zm], buf[out], box[zc],
                                                                       box[out]);
            zm = zc;
            zc = out;
        }
        substep<<<nt, GB_TILE * waves, 0, stream>>>(b, k, 2, buf[zc], buf[zm], nullptr, box[zc], nullptr);
        if (k > 0) big_decide_kernel<<<gg, 64, 0, stream>>>(b, k, tol); // the estimates came with T(k, 0)
    }
    big_accept_kernel<<<gm, GB_THREADS, 0, stream>>>(b, tol);
    big_control_kernel<<<1, GB_THREADS, 0, stream>>>(b, tol, flags);
    return hipGetLastError();
}

hipError_t launch_big_attempt_list(const BigBs &b, double tol, int32_t *flags, int tile_grid, hipStream_t stream)
{
    const int gg = (b.cap_G + 63) / 64, gm = (b.cap_M + GB_THREADS - 1) / GB_THREADS;
    const int nt = std::max(1, std::min(tile_grid, b.cap_T));
    const size_t M6 = 6 * (size_t)b.cap_M;
    const bool lv = b.nlev > 1;
    auto first = lv ? big_round_kernel<true, true> : big_round_kernel<false, true>;
    auto round = lv ? big_round_kernel<true, false> : big_round_kernel<false, false>;
    big_begin_kernel<<<gg, 64, 0, stream>>>(b, flags);
    big_prepare_kernel<<<(nt + 3) / 4, GB_THREADS, 0, stream>>>(b);
    if (nt <= BIG_SIDE_TILES)
        (lv ? big_list_kernel<true, 16> : big_list_kernel<false, 16>)<<<nt, 1024, 0, stream>>>(b);
    else
        (lv ? big_list_kernel<true, 8> : big_list_kernel<false, 8>)<<<nt, 512, 0, stream>>>(b);
    const int threads = 64 * BIG_LIST_LANES;
    first<<<dim3(nt, 1), threads, 0, stream>>>(b, -1, 0, -1, tol);
    // Columns in batches: side by side the columns above the accepted one have run for nothing.
    // While the tiles leave CUs idle that costs nothing; beyond, the first six run together (the
    // accepted column is mostly the fifth or sixth), and the last two only if they are needed.
    const int split = nt <= BIG_SIDE_TILES ? BS_KMAX : 6;
    int kv = -1; // the column whose verdict the launch takes: complete, but not yet decided
    for (int k0 = 0; k0 < BS_KMAX; k0 = k0 == 0 ? split : BS_KMAX) {
        const int k1 = k0 == 0 ? split : BS_KMAX;
        for (int j = 0; j < k1; ++j) { // column j ends with round j
            const int kf = std::max(k0, j);
            round<<<dim3(nt, k1 - kf), threads, 0, stream>>>(b, j, kf, kv, tol);
            kv = j >= std::max(k0, 1) ? j : -1;
        }
    }
    big_accept_kernel<<<gm, GB_THREADS, 0, stream>>>(b, tol);
    big_control_kernel<<<1, GB_THREADS, 0, stream>>>(b, tol, flags);
    return hipGetLastError();
}

hipError_t launch_big_finish(const BigBs &b, double *x, double *y, double *z, double *vx, double *vy,
                             double *vz, hipStream_t stream)
{
    if (b.G == 0) return hipSuccess;
    big_finish_kernel<<<(b.M + GB_THREADS - 1) / GB_THREADS, GB_THREADS, 0, stream>>>(b, x, y, z, vx, vy, vz);
    return hipGetLastError();
}

} // namespace genga
