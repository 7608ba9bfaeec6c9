// Long-range kick of the hybrid symplectic step (Brasser et al. 2023, Sect. 1): direct
// O(N^2) summation of Newtonian pair accelerations weighted by the changeover function,
// in FP32 pair arithmetic (coordinate differences formed in FP64) or in FP64, with the
// close-encounter pairs recorded by the same launch.  gfx950, wave64.
//
// Design (vector-ALU bound; no MFMA: a pair force is not a dense contraction, and on this chip
// the FP32 and FP64 matrix instructions take the vector ALU's own cycles):
//  * one task = up to 64 target bodies i (one per lane, FP64 position in VGPRs) and a run of
//    the system's sources j, split over the W waves of a workgroup.  The runs' lengths come
//    from the whole layout's work (kick_run_len), so that one disc, an ensemble and a handful
//    of massive bodies among test bodies all give every CU several workgroups.  The waves' and
//    the tasks' partial sums are added in a fixed order, so results are deterministic.
//  * the j index is wave-uniform: the sources' positions and masses come through the scalar
//    data path, four of an array in one load, so the inner loop has no LDS traffic or barrier.
//  * four sources per step; the changeover test is a single compare per four pairs against the
//    system's largest r_crit^2.  A lane that has a candidate only marks it (a bit per source
//    of the block of 64) and takes it out of the sums; after the block every lane works
//    through its own marks, deciding "inside r_crit,ij" in FP64 exactly as the definition
//    states, adding the pair in FP64 (weighted by K inside r_crit,ij) and recording the pairs
//    inside.  Marking keeps one copy of that code, outside the inner loop, and lanes with
//    different candidates work on them at the same time.
//  * FP32 path: FP32 partial sums over at most 32 sources, folded into FP64 accumulators
//    or into Kahan-compensated FP32 sums.  FP64 path: r^-3 from v_rsq_f64 (about 2^-24) and a
//    second-order series correction of its cube.  Where all sources of a task have one mass,
//    it is left out of the pair terms and multiplied into the sums at the end, in FP64.
//  * the same FP64 loop without the force terms lists the encounter pairs of a state on its
//    own (no kick has run on it).
#include "genga_internal.h"
#include "pair_math.h"

namespace genga {

namespace {

using CD = const __attribute__((address_space(4))) double;
using CF = const __attribute__((address_space(4))) float;

// Encounter pairs found by a wave collect in its own LDS buffer and reach the global list in
// blocks, one counter update per block, so that a dense list does not serialise on the
// counter.  The calls come from divergent code: only the wave's active lanes take part, and
// the fill count lives in LDS so that it stays one value for the whole wave.
constexpr int PAIR_BUF = 128;

struct PairBuf {
    int2 *buf;  // the wave's PAIR_BUF slots
    int *n;     // the wave's fill count
};

// orders the LDS accesses of the lanes of one wave
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ void store_pair(const KickArgs &a, int idx, int2 p)
{
    if (idx < a.pair_cap) {
        a.pairs[2 * idx] = p.x;
        a.pairs[2 * idx + 1] = p.y;
    } else {
        atomicOr(a.flags, FLAG_CAPACITY);
    }
}

// Move the buffer's n pairs, followed by the pairs (i, j) of the active lanes with em set
// (m = their mask), to the global list; the active lanes share the copying.
__device__ __forceinline__ void spill_pairs(const KickArgs &a, PairBuf pb, int n,
                                            unsigned long long m, bool em, int i, int j)
{
    const unsigned long long act = __ballot(1);
    const int lane = threadIdx.x & 63;
    const unsigned long long below = (1ull << lane) - 1;
    const int leader = __ffsll((long long)act) - 1;
    int base = 0;
    if (lane == leader) base = atomicAdd(a.pair_count, n + __popcll(m));
    base = __shfl(base, leader, 64);
    const int rank = __popcll(act & below), n_act = __popcll(act);
    for (int k = rank; k < n; k += n_act) store_pair(a, base + k, pb.buf[k]);
    if (em) store_pair(a, base + n + __popcll(m & below), make_int2(i, j));
    wave_lds_sync();
    *pb.n = 0;
    wave_lds_sync();
}

// Record (i, j) for the active lanes with em set.
__device__ __forceinline__ void emit_pair(const KickArgs &a, PairBuf pb, bool em, int i, int j)
{
    const unsigned long long m = __ballot(em);
    if (!m) return;
    const int n = *pb.n, c = __popcll(m);
    if (n + c > PAIR_BUF) {
        spill_pairs(a, pb, n, m, em, i, j);
        return;
    }
    if (em) pb.buf[n + __popcll(m & ((1ull << (threadIdx.x & 63)) - 1))] = make_int2(i, j);
    wave_lds_sync();
    *pb.n = n + c;
    wave_lds_sync();
}

// Empty the buffers of a workgroup's W waves (every lane of it calls this).  One counter update for
// all of them: the updates of one address follow each other at about 10 ns, and on dense annuli each
// wave has some pairs.  With one per wave the list of 6600 bodies in random order (59066 pairs, 10800
// waves) took 118 us and their FP32 kick 84, so 73 and 44; sparse and sorted bodies the same.
template <int W>
__device__ __forceinline__ void flush_pairs(const KickArgs &a, const int2 (*slots)[PAIR_BUF], const int *fill, int wave,
                                            int lane)
{
    __shared__ int base;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const int n = fill[w];
        if (w < wave) before += n;
        all += n;
    }
    if (all == 0) return; // all of the workgroup
    if (threadIdx.x == 0) base = atomicAdd(a.pair_count, all);
    __syncthreads();
    for (int k = lane; k < fill[wave]; k += 64) store_pair(a, base + before + k, slots[wave][k]);
}

// A marked pair (within the candidate radius of the system): exact FP64 decision; the term is
// added in FP64, inside r_crit,ij weighted by K and the pair recorded.
template <bool LIST>
__device__ __forceinline__ void near_pair(const KickArgs &a, int j, int i, bool valid, double xi, double yi, double zi,
                                          double rci, double &sx, double &sy, double &sz, PairBuf pb)
{
    if (j == i) return;
    const double dx = a.x[j] - xi, dy = a.y[j] - yi, dz = a.z[j] - zi;
    const double r2 = sep2_rn(dx, dy, dz);
    const double rcij = fmax(rci, a.rc[j]);
    const bool in = r2 < sq_rn(rcij);
    if (!LIST) {
        const double r = sqrt(r2);
        const double k = in ? changeover_k((r - 0.1 * rcij) / (0.9 * rcij)) : 1.0;
        if (k > 0.0) {
            const double s = a.m[j] * k / (r2 * r);
            sx += s * dx;
            sy += s * dy;
            sz += s * dz;
        }
    }
    if (in) emit_pair(a, pb, valid && i < j && (!a.status || (a.status[i] == 0 && a.status[j] == 0)), i, j);
}

// The marks of a block of at most 64 sources from jb on (bit k: source jb + k), lane by lane.
template <bool LIST>
__device__ __forceinline__ void near_block(const KickArgs &a, int jb, uint32_t m0, uint32_t m1, int i, bool valid,
                                           double xi, double yi, double zi, double rci, double &sx, double &sy,
                                           double &sz, PairBuf pb)
{
    while (m0 | m1) {
        int k;
        if (m0) {
            k = __builtin_ctz(m0);
            m0 &= m0 - 1;
        } else {
            k = 32 + __builtin_ctz(m1);
            m1 &= m1 - 1;
        }
        near_pair<LIST>(a, jb + k, i, valid, xi, yi, zi, rci, sx, sy, sz, pb);
    }
}

// What a task visits.  With a task list (KickArgs::tasks) the runs were laid out on the host; else
// every item's sources are cut into a.split runs.
__device__ __forceinline__ KickTask task_of(const KickArgs &a, int t)
{
    if (a.tasks) return a.tasks[t];
    const WorkItem w = a.items[t / a.split];
    const int part = t % a.split, b = a.sys_off[w.sys], e = b + w.nsrc;
    const int per = kick_run(w.nsrc, a.split);
    KickTask k;
    k.sys = w.sys;
    k.i0 = w.i0;
    k.ni = w.ni;
    k.j0 = min(b + part * per, e);
    k.j1 = min(k.j0 + per, e);
    k.c0 = a.chunk_first[w.sys];
    k.c1 = a.chunk_first[w.sys + 1];
    k.off = b;
    k.row = (uint32_t)a.split * (uint32_t)w.i0 + (uint32_t)part * (uint32_t)w.ni;
    return k;
}

// largest r_crit^2 of the task's system, the chunks over the lanes
__device__ __forceinline__ double system_rc2max(const KickArgs &a, const KickTask &t)
{
    double mx = 0.0;
    for (int k = t.c0 + (int)(threadIdx.x & 63); k < t.c1; k += 64)
        mx = fmax(mx, a.rc2_part[k]);
    return wave_maxv(mx);
}

// The FP64 candidate threshold, with a relative margin: q is formed with fused multiply-adds, the
// exact decision without them.
__device__ __forceinline__ double candidate_rc2(const KickArgs &a, const KickTask &t)
{
    return system_rc2max(a, t) * (1.0 + 1e-12) + 1e-300;
}

// The mass that all sources [j0, j1) of the task share, or NaN: from the chunks' common masses.
__device__ __forceinline__ double common_mass(const KickArgs &a, const KickTask &t, int j0, int j1)
{
    if (j0 >= j1) return 0.0;
    const int k0 = t.c0 + (j0 - t.off) / CHUNK, k1 = t.c0 + (j1 - 1 - t.off) / CHUNK;
    const double m = a.chunk_mass[k0];
    bool same = true;
    for (int k = k0 + (int)(threadIdx.x & 63); k <= k1; k += 64) same = same && a.chunk_mass[k] == m;
    return __all(same) ? m : __longlong_as_double(0x7ff8000000000000ll);
}

struct Acc32 {
    float fx, fy, fz;
};

// S + v with Kahan compensation: after the call S - C equals the exact sum of the values added
// so far up to the rounding of the last C
__device__ __forceinline__ void kahan_add(float &S, float &C, float v)
{
    const float y = v - C;
    const float t = S + y;
    C = (t - S) - y;
    S = t;
}

// UNI: the sources' mass is left out
template <bool UNI>
__device__ __forceinline__ void far32(float mj, float dx, float dy, float dz, float q, Acc32 &c)
{
    const float ri = __builtin_amdgcn_rsqf(q);
    const float s = UNI ? (ri * ri) * ri : mj * (ri * ri) * ri;
    c.fx = fmaf(s, dx, c.fx);
    c.fy = fmaf(s, dy, c.fy);
    c.fz = fmaf(s, dz, c.fz);
}

template <bool UNI>
__device__ __forceinline__ void far64(double mj, double dx, double dy, double dz, double q, double &fx, double &fy,
                                      double &fz)
{
    const double y0 = __builtin_amdgcn_rsq(q);
    // r^-3 = q^(-3/2) = y0^3 (1 - e)^(-3/2) with e = 1 - q y0^2 (|e| about 2^-23): the
    // series 1 + 3/2 e + 15/8 e^2 leaves a relative error of about 2 e^3, below the rounding
    const double y2 = y0 * y0;
    const double e = fma(-q, y2, 1.0);
    const double w = fma(fma(1.875, e, 1.5), e, 1.0);
    const double s = UNI ? w * (y2 * y0) : (mj * w) * (y2 * y0);
    fx = fma(s, dx, fx);
    fy = fma(s, dy, fy);
    fz = fma(s, dz, fz);
}

// Sources [j, j + V) of the FP32 path: the far terms into c, the candidates marked (bit j - jb).
template <bool UNI, int V>
__device__ __forceinline__ void step32(CD *X, CD *Y, CD *Z, CF *M, int j, int jb, double xi, double yi, double zi,
                                       float T, Acc32 &c, uint32_t &m0, uint32_t &m1)
{
    float dx[V], dy[V], dz[V], q[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        dx[v] = (float)(X[j + v] - xi);
        dy[v] = (float)(Y[j + v] - yi);
        dz[v] = (float)(Z[j + v] - zi);
        q[v] = fmaf(dx[v], dx[v], fmaf(dy[v], dy[v], dz[v] * dz[v]));
    }
    float mn = q[0];
#pragma unroll
    for (int v = 1; v < V; ++v) mn = fminf(mn, q[v]);
    if (__builtin_expect(mn < T, 0)) {
        uint32_t bits = 0;
#pragma unroll
        for (int v = 0; v < V; ++v)
            if (q[v] < T) {
                bits |= 1u << v;
                q[v] = INFINITY; // rsq gives 0: no term here
            }
        const int k = j - jb;
        if (k < 32) m0 |= bits << k;
        else m1 |= bits << (k - 32);
    }
#pragma unroll
    for (int v = 0; v < V; ++v) far32<UNI>(UNI ? 0.f : M[j + v], dx[v], dy[v], dz[v], q[v], c);
}

// The same in FP64 (FAR = false: candidates only).
template <bool UNI, bool FAR, int V>
__device__ __forceinline__ void step64(CD *X, CD *Y, CD *Z, CD *M, int j, int jb, double xi, double yi, double zi,
                                       double T, double &fx, double &fy, double &fz, uint32_t &m0, uint32_t &m1)
{
    double dx[V], dy[V], dz[V], q[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        dx[v] = X[j + v] - xi;
        dy[v] = Y[j + v] - yi;
        dz[v] = Z[j + v] - zi;
        q[v] = fma(dx[v], dx[v], fma(dy[v], dy[v], dz[v] * dz[v]));
    }
    double mn = q[0];
#pragma unroll
    for (int v = 1; v < V; ++v) mn = fmin(mn, q[v]);
    if (__builtin_expect(mn < T, 0)) {
        uint32_t bits = 0;
#pragma unroll
        for (int v = 0; v < V; ++v)
            if (q[v] < T) {
                bits |= 1u << v;
                // the far term of a separation of 2^200 in place of the pair's: with the
                // difference cleared it adds a zero
                q[v] = 0x1p400;
                dx[v] = dy[v] = dz[v] = 0.0;
            }
        const int k = j - jb;
        if (k < 32) m0 |= bits << k;
        else m1 |= bits << (k - 32);
    }
    if (FAR) {
#pragma unroll
        for (int v = 0; v < V; ++v) far64<UNI>(UNI ? 0.0 : M[j + v], dx[v], dy[v], dz[v], q[v], fx, fy, fz);
    }
}

// Sum the W waves' partial accelerations in a fixed order; then either finish the body or, when
// its sources are split over tasks, store this task's share for kick_finish_kernel.
template <int W>
__device__ __forceinline__ void finish(const KickArgs &a, double (*red)[W][64], int wave, int lane, bool valid, int i,
                                       const KickTask &k, double sx, double sy, double sz)
{
    red[0][wave][lane] = sx;
    red[1][wave][lane] = sy;
    red[2][wave][lane] = sz;
    __syncthreads();
    if (wave != 0) return;
    double t[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int w = 0; w < W; ++w)
#pragma unroll
        for (int q = 0; q < 3; ++q) t[q] += red[q][w][lane];
    if (!valid) return;
    if (a.direct) {
        store_accel(a, i, t[0], t[1], t[2]);
        return;
    }
    double *p = a.part + 3 * (size_t)k.row + lane;
    p[0] = t[0];
    p[k.ni] = t[1];
    p[2 * k.ni] = t[2];
}

// Adds the tasks' shares of every body in task order, then as finish() above.  One wave per item.
__global__ __launch_bounds__(256) void kick_finish_kernel(KickArgs a)
{
    const int it = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6)), lane = threadIdx.x & 63;
    if (it >= a.n_items) return;
    const WorkItem w = a.items[it];
    if (lane >= w.ni) return;
    double t[3];
    item_shares(a, it, w, lane, t);
    store_accel(a, w.i0 + lane, t[0], t[1], t[2]);
}

// Sources whose FP32 terms a wave adds up before it folds them into its accumulators: 32 of a
// long run, 4 of a run of up to 32 sources and one of a run of up to 16, whose sums are so short
// that their rounding would show.  rms force error of 40000 bodies 1.41e-7 / 1.16e-7 / 1.03e-7
// and 562 / 566 / 575 us with folds every 64 / 32 / 16 sources.
__device__ __forceinline__ int fold_len(int run)
{
    return run <= 16 ? 1 : run <= 32 ? 4 : 32;
}

// One wave's run of sources [jb, je): marks per block of 64, FP32 sums per fold_len sources.
template <bool KAHAN, bool UNI>
__device__ __forceinline__ void run32(const KickArgs &a, int jb, int je, int i, bool valid, double xi, double yi,
                                      double zi, double rci, float T, double mass, double &sx, double &sy, double &sz,
                                      PairBuf pb)
{
    CD *X = (CD *)a.x, *Y = (CD *)a.y, *Z = (CD *)a.z;
    CF *M = (CF *)a.m32;
    Acc32 S{0.f, 0.f, 0.f}, C{0.f, 0.f, 0.f}; // Kahan sums of the folds (KAHAN)
    double fx = 0.0, fy = 0.0, fz = 0.0;      // FP64 sums of the folds (else)
    const int F = fold_len(je - jb);
    for (int j0 = jb; j0 < je; j0 += 64) {
        const int j1 = min(j0 + 64, je);
        uint32_t m0 = 0, m1 = 0;
        int j = j0;
        while (j < j1) {
            const int jf = min(j + F, j1);
            Acc32 c{0.f, 0.f, 0.f};
            for (; j + 4 <= jf; j += 4) step32<UNI, 4>(X, Y, Z, M, j, j0, xi, yi, zi, T, c, m0, m1);
            for (; j < jf; ++j) step32<UNI, 1>(X, Y, Z, M, j, j0, xi, yi, zi, T, c, m0, m1);
            if (KAHAN) {
                kahan_add(S.fx, C.fx, c.fx);
                kahan_add(S.fy, C.fy, c.fy);
                kahan_add(S.fz, C.fz, c.fz);
            } else {
                fx += (double)c.fx;
                fy += (double)c.fy;
                fz += (double)c.fz;
            }
        }
        near_block<false>(a, j0, m0, m1, i, valid, xi, yi, zi, rci, sx, sy, sz, pb);
    }
    if (KAHAN) {
        fx = (double)S.fx - (double)C.fx;
        fy = (double)S.fy - (double)C.fy;
        fz = (double)S.fz - (double)C.fz;
    }
    const double f = UNI ? mass : 1.0;
    sx = fma(f, fx, sx);
    sy = fma(f, fy, sy);
    sz = fma(f, fz, sz);
}

template <bool UNI, bool LIST>
__device__ __forceinline__ void run64(const KickArgs &a, int jb, int je, int i, bool valid, double xi, double yi,
                                      double zi, double rci, double T, double mass, double &sx, double &sy, double &sz,
                                      PairBuf pb)
{
    CD *X = (CD *)a.x, *Y = (CD *)a.y, *Z = (CD *)a.z, *M = (CD *)a.m;
    double fx = 0.0, fy = 0.0, fz = 0.0;
    for (int j0 = jb; j0 < je; j0 += 64) {
        const int j1 = min(j0 + 64, je);
        uint32_t m0 = 0, m1 = 0;
        int j = j0;
        for (; j + 4 <= j1; j += 4) step64<UNI, !LIST, 4>(X, Y, Z, M, j, j0, xi, yi, zi, T, fx, fy, fz, m0, m1);
        for (; j < j1; ++j) step64<UNI, !LIST, 1>(X, Y, Z, M, j, j0, xi, yi, zi, T, fx, fy, fz, m0, m1);
        near_block<LIST>(a, j0, m0, m1, i, valid, xi, yi, zi, rci, sx, sy, sz, pb);
    }
    const double f = UNI ? mass : 1.0;
    sx = fma(f, fx, sx);
    sy = fma(f, fy, sy);
    sz = fma(f, fz, sz);
}

// The wave's share of a task's sources.
template <int W>
__device__ __forceinline__ void wave_run(const KickTask &t, int wave, int &jb, int &je)
{
    const int chunk = (t.j1 - t.j0 + W - 1) / W;
    jb = __builtin_amdgcn_readfirstlane(min(t.j0 + wave * chunk, t.j1));
    je = __builtin_amdgcn_readfirstlane(min(jb + chunk, t.j1));
}

template <int W, bool KAHAN>
__global__ __launch_bounds__(64 * W) void kick32_kernel(KickArgs a)
{
    __shared__ double red[3][W][64];
    __shared__ int2 pair_slots[W][PAIR_BUF];
    __shared__ int pair_fill[W];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const PairBuf pb{pair_slots[wave], &pair_fill[wave]};
    pair_fill[wave] = 0;
    wave_lds_sync();
    const KickTask t = task_of(a, blockIdx.x);
    const bool valid = lane < t.ni;
    const int i = t.i0 + (valid ? lane : 0);
    const double xi = a.x[i], yi = a.y[i], zi = a.z[i], rci = a.rc[i];
    // candidate threshold: the system's largest r_crit^2 with a margin that covers the FP32
    // rounding of r^2; never zero, so that the self pair is always marked
    const float T = (float)(system_rc2max(a, t) * 1.0001) + 1e-24f;
    int jb, je;
    wave_run<W>(t, wave, jb, je);
    double sx = 0.0, sy = 0.0, sz = 0.0;
    const double mass = common_mass(a, t, jb, je);
    if (mass == mass)
        run32<KAHAN, true>(a, jb, je, i, valid, xi, yi, zi, rci, T, mass, sx, sy, sz, pb);
    else
        run32<KAHAN, false>(a, jb, je, i, valid, xi, yi, zi, rci, T, mass, sx, sy, sz, pb);
    flush_pairs<W>(a, pair_slots, pair_fill, wave, lane);
    finish<W>(a, red, wave, lane, valid, i, t, sx, sy, sz);
}

template <int W>
__global__ __launch_bounds__(64 * W) void kick64_kernel(KickArgs a)
{
    __shared__ double red[3][W][64];
    __shared__ int2 pair_slots[W][PAIR_BUF];
    __shared__ int pair_fill[W];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const PairBuf pb{pair_slots[wave], &pair_fill[wave]};
    pair_fill[wave] = 0;
    wave_lds_sync();
    const KickTask t = task_of(a, blockIdx.x);
    const bool valid = lane < t.ni;
    const int i = t.i0 + (valid ? lane : 0);
    const double xi = a.x[i], yi = a.y[i], zi = a.z[i], rci = a.rc[i];
    const double T = candidate_rc2(a, t);
    int jb, je;
    wave_run<W>(t, wave, jb, je);
    double sx = 0.0, sy = 0.0, sz = 0.0;
    const double mass = common_mass(a, t, jb, je);
    if (mass == mass)
        run64<true, false>(a, jb, je, i, valid, xi, yi, zi, rci, T, mass, sx, sy, sz, pb);
    else
        run64<false, false>(a, jb, je, i, valid, xi, yi, zi, rci, T, mass, sx, sy, sz, pb);
    flush_pairs<W>(a, pair_slots, pair_fill, wave, lane);
    finish<W>(a, red, wave, lane, valid, i, t, sx, sy, sz);
}

// The encounter pairs alone, in the layout's own tasks.  A pair is found from its lower body, so of
// its sources an item looks at those from its first body on (all of them: list of 40000 bodies 343
// us, so 216; of 64 discs of 2000-8000 391 and 270); bound by the FP64 issue of three differences and
// r^2 per pair.  In the energy's tasks, which have just these sources, 200 and 269, but 700 bodies 24
// against 21 and dense lists of 12000 181 against 160.
constexpr int LIST_WAVES = 4;
__global__ __launch_bounds__(64 * LIST_WAVES) void pair_list_kernel(KickArgs a)
{
    __shared__ int2 pair_slots[LIST_WAVES][PAIR_BUF];
    __shared__ int pair_fill[LIST_WAVES];
    KickTask t = a.tasks[blockIdx.x];
    t.j0 = max(t.j0, t.i0);
    if (t.j0 >= t.j1) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const PairBuf pb{pair_slots[wave], &pair_fill[wave]};
    pair_fill[wave] = 0;
    wave_lds_sync();
    const bool valid = lane < t.ni;
    const int i = t.i0 + (valid ? lane : 0);
    const double xi = a.x[i], yi = a.y[i], zi = a.z[i], rci = a.rc[i];
    const double T = candidate_rc2(a, t);
    int jb, je;
    wave_run<LIST_WAVES>(t, wave, jb, je);
    double sx = 0.0, sy = 0.0, sz = 0.0;
    run64<true, true>(a, jb, je, i, valid, xi, yi, zi, rci, T, 0.0, sx, sy, sz, pb);
    flush_pairs<LIST_WAVES>(a, pair_slots, pair_fill, wave, lane);
}

// Per chunk the largest r_crit^2 and the mass its bodies share (NaN: they differ), the masses in
// FP32 (m32 may be null), and a cleared pair counter.
__global__ __launch_bounds__(CHUNK) void prep_kernel(const Chunk *chunks, const double *m, const double *rc,
                                                     float *m32, double *rc2_part, double *chunk_mass,
                                                     int32_t *pair_count)
{
    const Chunk c = chunks[blockIdx.x];
    const int i = c.b + (int)threadIdx.x;
    const bool on = i < c.e;
    const double m0 = m[c.b], mi = on ? m[i] : m0, rci = on ? rc[i] : 0.0;
    if (on && m32) m32[i] = (float)mi;
    const double mx = wave_maxv(rci * rci);
    __shared__ double red[CHUNK / 64];
    __shared__ int same[CHUNK / 64];
    const bool eq = __all(mi == m0);
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6] = mx;
        same[threadIdx.x >> 6] = eq;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double r = 0.0;
        bool all = true;
        for (int w = 0; w < CHUNK / 64; ++w) {
            r = fmax(r, red[w]);
            all = all && same[w] != 0;
        }
        rc2_part[blockIdx.x] = r;
        chunk_mass[blockIdx.x] = all ? m0 : __longlong_as_double(0x7ff8000000000000ll);
        if (blockIdx.x == 0) *pair_count = 0;
    }
}

// eq. (1): r_crit,i = max(n1 R_H,i, n2 dt v_i)
__global__ __launch_bounds__(256) void rcrit_kernel(int n_total, const int32_t *sys_of,
                                                    const double *mstar, const double *x,
                                                    const double *y, const double *z,
                                                    const double *vx, const double *vy,
                                                    const double *vz, const double *m, double n1,
                                                    double n2, double dt, double *rc)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_total) return;
    double ms = mstar[sys_of[i]];
    double r = sqrt(x[i] * x[i] + y[i] * y[i] + z[i] * z[i]);
    double v2 = vx[i] * vx[i] + vy[i] * vy[i] + vz[i] * vz[i];
    double inv_a = 2.0 / r - v2 / ms;
    double a = inv_a > 0.0 ? 1.0 / inv_a : r;
    double rh = a * cbrt(m[i] / (3.0 * ms));
    double vk = sqrt(ms / a);
    rc[i] = fmax(n1 * rh, n2 * dt * vk);
}

} // namespace

hipError_t launch_prep(const Layout &L, const double *m, const double *rc, float *m32, double *rc2_part,
                       double *chunk_mass, int32_t *pair_count, hipStream_t stream)
{
    if (L.n_chunks == 0) return hipSuccess;
    prep_kernel<<<L.n_chunks, CHUNK, 0, stream>>>(L.chunks, m, rc, m32, rc2_part, chunk_mass, pair_count);
    return hipGetLastError();
}

hipError_t launch_kick_shares(const KickArgs &a, int fp32, int kahan, int waves, hipStream_t stream)
{
    if (a.n_items == 0) return hipSuccess;
    const int grid = a.tasks ? a.n_tasks : a.n_items * a.split;
#define GENGA_KICK_CASE(Wv)                                                                   \
    case Wv:                                                                                  \
        if (fp32 && kahan)                                                                    \
            kick32_kernel<Wv, true><<<grid, 64 * Wv, 0, stream>>>(a);                        \
        else if (fp32)                                                                        \
            kick32_kernel<Wv, false><<<grid, 64 * Wv, 0, stream>>>(a);                       \
        else                                                                                  \
            kick64_kernel<Wv><<<grid, 64 * Wv, 0, stream>>>(a);                       \
        break;
    switch (waves) {
        GENGA_KICK_CASE(4)
        GENGA_KICK_CASE(8)
        GENGA_KICK_CASE(16)
    default:
        return hipErrorInvalidValue;
    }
#undef GENGA_KICK_CASE
    return hipGetLastError();
}

hipError_t launch_kick(const KickArgs &a, int fp32, int kahan, int waves, hipStream_t stream)
{
    const hipError_t e = launch_kick_shares(a, fp32, kahan, waves, stream);
    if (e != hipSuccess || a.direct || a.n_items == 0) return e;
    kick_finish_kernel<<<(a.n_items + 3) / 4, 256, 0, stream>>>(a);
    return hipGetLastError();
}

hipError_t launch_pair_list(const KickArgs &a, hipStream_t stream)
{
    if (a.n_tasks == 0) return hipSuccess;
    pair_list_kernel<<<a.n_tasks, 64 * LIST_WAVES, 0, stream>>>(a);
    return hipGetLastError();
}

hipError_t launch_rcrit(const Layout &L, const double *x, const double *y, const double *z,
                        const double *vx, const double *vy, const double *vz, const double *m,
                        double n1, double n2, double dt, double *rc, hipStream_t stream)
{
    if (L.n_total == 0) return hipSuccess;
    rcrit_kernel<<<(L.n_total + 255) / 256, 256, 0, stream>>>(L.n_total, L.sys_of, L.mstar, x, y, z,
                                                              vx, vy, vz, m, n1, n2, dt, rc);
    return hipGetLastError();
}

} // namespace genga
