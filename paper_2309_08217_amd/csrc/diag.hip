// Diagnostics (Brasser et al. 2023, Sect. 3.1: Delta E/E and Delta L/L) and the canonical
// order of the encounter list.  FP64.
//
// Energy of the democratic heliocentric Hamiltonian per system:
//   E = sum m v^2/2 + |sum m v|^2/(2 Mstar) - sum Mstar m/r - sum_{i<j} m_i m_j / r_ij,
//   L = sum m r x v.
// The pair sum takes 64 targets per workgroup and a run of the sources j > i, split over its
// waves; the runs' lengths come from the whole layout's work, as the kick's do, so that a few
// massive bodies among many test bodies do not keep four workgroups busy alone (20040 bodies in
// TP2 mode: 72 us when every block of targets had four parts).  The tasks' partial sums are
// reduced in a fixed order, so the result is deterministic.  Velocities may be given half a kick
// ahead: v_sync = v - vshift * a.
#include "genga_internal.h"
#include "pair_math.h"

namespace genga {

namespace {

constexpr int EW = 4;      // waves per workgroup in the pair sum
constexpr int NPART = 9;   // pairpot, kin, sunpot, px, py, pz, lx, ly, lz

using CJ64 = const __attribute__((address_space(4))) double;

// Each of v summed over the wave, in every lane; the exchanges of one round run side by side.
template <int N>
__device__ __forceinline__ void wave_sums(double (&v)[N])
{
    for (int o = 32; o > 0; o >>= 1) {
        double u[N];
#pragma unroll
        for (int k = 0; k < N; ++k) u[k] = __shfl_xor(v[k], o, 64);
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] += u[k];
    }
}

__global__ __launch_bounds__(64 * EW) void energy_kernel(const EnergyTask *tasks, const double *mstar, const double *x,
                                                         const double *y, const double *z, const double *vx,
                                                         const double *vy, const double *vz, const double *m,
                                                         const double *ax, const double *ay, const double *az,
                                                         double vshift, double *partial)
{
    __shared__ double red[EW][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    CJ64 *X = (CJ64 *)x;
    CJ64 *Y = (CJ64 *)y;
    CJ64 *Z = (CJ64 *)z;
    CJ64 *M = (CJ64 *)m;
    const EnergyTask w = tasks[blockIdx.x];
    const bool valid = lane < w.ni;
    const int i = w.i0 + (valid ? lane : 0);
    const double xi = x[i], yi = y[i], zi = z[i];
    const int chunk = (w.j1 - w.j0 + EW - 1) / EW;
    const int jb = __builtin_amdgcn_readfirstlane(min(w.j0 + wave * chunk, w.j1));
    const int je = __builtin_amdgcn_readfirstlane(min(jb + chunk, w.j1));
    double s = 0.0;
    const int jmask = min(je, w.i0 + 64);
    int j = jb;
    // sources inside the item's own range: only j > i counts (the self pair has q = 0, so it is
    // replaced by a harmless q = 1 with zero weight); four at a time, as in a small system these are
    // most of a wave's sources (257 and 1000 bodies one at a time 13.8 and 16.0 us, in fours 9.5 and 11.2,
    // and in runs of ENERGY_RUN_MIN 5.1 and 5.3)
    const auto masked = [&](int jj, double &q, double &mj) {
        const double dx = X[jj] - xi, dy = Y[jj] - yi, dz = Z[jj] - zi;
        const bool take = jj > i;
        q = take ? fma(dx, dx, fma(dy, dy, dz * dz)) : 1.0;
        mj = take ? M[jj] : 0.0;
    };
    for (; j + 4 <= jmask; j += 4) {
        double q[4], mj[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) masked(j + v, q[v], mj[v]);
#pragma unroll
        for (int v = 0; v < 4; ++v) s = fma(mj[v], inv_sqrt64(q[v]), s);
    }
    for (; j < jmask; ++j) {
        double q, mj;
        masked(j, q, mj);
        s = fma(mj, inv_sqrt64(q), s);
    }
    for (; j + 4 <= je; j += 4) {
        double q[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const double dx = X[j + v] - xi, dy = Y[j + v] - yi, dz = Z[j + v] - zi;
            q[v] = fma(dx, dx, fma(dy, dy, dz * dz));
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) s = fma(M[j + v], inv_sqrt64(q[v]), s);
    }
    for (; j < je; ++j) {
        const double dx = X[j] - xi, dy = Y[j] - yi, dz = Z[j] - zi;
        const double q = fma(dx, dx, fma(dy, dy, dz * dz));
        s = fma(M[j], inv_sqrt64(q), s);
    }
    red[wave][lane] = s;
    __syncthreads();
    if (wave != 0) return;
    double tot = 0.0;
#pragma unroll
    for (int k = 0; k < EW; ++k) tot += red[k][lane];
    const double mi = valid ? m[i] : 0.0;
    if (!w.first) {
        double v[1] = {mi * tot};
        wave_sums(v);
        if (lane == 0) partial[blockIdx.x] = v[0];
        return;
    }
    double v[NPART] = {};
    v[0] = mi * tot;
    if (valid) {
        const double ux = vx[i] - vshift * ax[i];
        const double uy = vy[i] - vshift * ay[i];
        const double uz = vz[i] - vshift * az[i];
        v[1] = 0.5 * mi * (ux * ux + uy * uy + uz * uz);
        v[2] = -mstar[w.sys] * mi / sqrt(xi * xi + yi * yi + zi * zi);
        v[3] = mi * ux;
        v[4] = mi * uy;
        v[5] = mi * uz;
        v[6] = mi * (yi * uz - zi * uy);
        v[7] = mi * (zi * ux - xi * uz);
        v[8] = mi * (xi * uy - yi * ux);
    }
    wave_sums(v);
    if (lane == 0)
        for (int k = 0; k < NPART; ++k) partial[(size_t)k * gridDim.x + blockIdx.x] = v[k];
}

// One workgroup per system: each thread sums a strided subset of the system's task partials
// in order (the pair sum of every task, the other parts of the tasks that have them, which are
// the system's first), then the lanes of a wave and the waves in fixed trees.  Bound by how fast
// one CU reads what others wrote: 20040 bodies (12 thousand tasks) took 17 us with nine sums of
// every task.  Systems of up to ENERGY_SMALL tasks take a wave each (SMALL, blocks of EnergyRun): with a
// workgroup each 100000 systems of ten bodies took 1.86 ms, now 0.11.
constexpr int EF_THREADS = 64 * ENERGY_WAVES, EF_AHEAD = 4;
static_assert(ENERGY_SMALL <= 64, "a task per lane");

__device__ __forceinline__ double strided_sum(const double *p, int t0, int t1)
{
    double t = 0.0;
    for (int it = t0 + threadIdx.x; it < t1; it += EF_AHEAD * EF_THREADS) {
        double v[EF_AHEAD]; // all in flight
#pragma unroll
        for (int u = 0; u < EF_AHEAD; ++u) v[u] = p[min(it + u * EF_THREADS, t1 - 1)];
#pragma unroll
        for (int u = 0; u < EF_AHEAD; ++u) t += it + u * EF_THREADS < t1 ? v[u] : 0.0;
    }
    return t;
}

// t: pairpot, kin, sunpot, p, l
__device__ __forceinline__ void store_energy(double *out, int s, double mstar, const double (&t)[NPART])
{
    const double p2 = t[3] * t[3] + t[4] * t[4] + t[5] * t[5];
    out[4 * (size_t)s + 0] = t[1] + p2 / (2.0 * mstar) + t[2] - t[0];
    out[4 * (size_t)s + 1] = t[6];
    out[4 * (size_t)s + 2] = t[7];
    out[4 * (size_t)s + 3] = t[8];
}

template <bool SMALL>
__global__ __launch_bounds__(EF_THREADS) void energy_finish_kernel(const EnergyRun *runs, const int32_t *task_first,
                                                                   const double *mstar, const double *partial,
                                                                   int n_tasks, double *out)
{
    __shared__ double red[NPART][ENERGY_WAVES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int s = blockIdx.x;
    double t[NPART];
    if constexpr (SMALL) {
        const EnergyRun r = runs[blockIdx.x];
        s = r.sys;
        if (r.n > 0) { // n small systems
            if (wave >= r.n) return;
            s += wave;
            const int t0 = task_first[2 * s], tk = task_first[2 * s + 1], t1 = task_first[2 * s + 2], it = t0 + lane;
            t[0] = it < t1 ? partial[it] : 0.0;
            for (int k = 1; k < NPART; ++k) t[k] = it < tk ? partial[(size_t)k * n_tasks + it] : 0.0;
            wave_sums(t);
            if (lane == 0) store_energy(out, s, mstar[s], t);
            return;
        }
    }
    const int t0 = task_first[2 * s], tk = task_first[2 * s + 1], t1 = task_first[2 * s + 2];
    // the usual number of first tasks in one load each, beside the pair sums
    t[0] = strided_sum(partial, t0, t1);
    for (int k = 1; k < NPART; ++k) {
        const double *p = partial + (size_t)k * n_tasks;
        const int it = t0 + (int)threadIdx.x;
        t[k] = it < tk ? p[it] : 0.0;
    }
    for (int it = t0 + (int)threadIdx.x + EF_THREADS; it < tk; it += EF_THREADS)
        for (int k = 1; k < NPART; ++k) t[k] += partial[(size_t)k * n_tasks + it];
    wave_sums(t);
    if (lane == 0)
        for (int k = 0; k < NPART; ++k) red[k][wave] = t[k];
    __syncthreads();
    if (threadIdx.x < NPART) {
        double v = 0.0;
        for (int w = 0; w < ENERGY_WAVES; ++w) v += red[threadIdx.x][w];
        red[threadIdx.x][0] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 0; k < NPART; ++k) t[k] = red[k][0];
        store_energy(out, s, mstar[s], t);
    }
}

// ------------------------------------------------------------------------------------------
// Canonical (lexicographic) order of the encounter list, in one launch.  Up to SORT_SMALL pairs (a
// list of a disc whose r_crit is a few Hill radii) the first workgroup sorts them in LDS, the others
// return.  Above, each workgroup takes a run of bodies i, reads the whole list, and needs nothing
// from the others: it counts the pairs below its run (where its output starts) and per body, keeps
// its own in LDS (or reads the list again), places them by body and ranks each among its body's by
// counting.  The more bodies the more workgroups, and each reads the list twice whatever its
// length.  Lists (with the listing) of dense annuli of 2049, 6600 and 12000 bodies (5700, 59000 and
// 197000 pairs) took 0.28, 3.7 and 15 ms, nearly all of it a bitonic sort of one workgroup (in global
// memory above 8192 pairs), now 0.027, 0.072 and 0.145.
// ------------------------------------------------------------------------------------------
constexpr int SORT_THREADS = 1024;
constexpr int SORT_SMALL = 512;   // pairs: 592, 714, 1659 take 21.7, 23.2, 41 us (with the listing) in one
                                  // workgroup, 19.7, 20.9, 27 in all; 439 and 489 the same, 142 18.6 and 20.6
constexpr int SORT_LDS = 8192;    // keys
constexpr int SORT_BLOCKS = 256;  // at most (40322 bodies with 64, 128, 256: 2055, 1382, 1101 us)
constexpr int SORT_BODIES = 4096; // bodies at a time (counts in a quarter of the keys' space)
constexpr int SORT_COUNT = 256;   // a body's pairs ranked by counting; more are sorted by the workgroup
constexpr int SORT_AHEAD = 8;     // pairs in flight per thread

// Ascending bitonic sort of keys[0, n), any n: every comparator puts the smaller key first, so
// what would lie beyond n (larger than all) never moves.
__device__ void bitonic(uint64_t *keys, int n, bool global_mem)
{
    for (int size = 2; size < 2 * n; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            const int flip = stride == size >> 1 ? size - 1 : stride;
            for (int k = threadIdx.x; k < n; k += SORT_THREADS) {
                const int partner = k ^ flip;
                if (partner > k && partner < n) {
                    const uint64_t x = keys[k], y = keys[partner];
                    if (x > y) {
                        keys[k] = y;
                        keys[partner] = x;
                    }
                }
            }
            if (global_mem) __threadfence();
            __syncthreads();
        }
    }
}

__device__ __forceinline__ uint64_t pair_key(int2 p) { return (uint64_t)(uint32_t)p.x << 32 | (uint32_t)p.y; }

__device__ __forceinline__ void put_pair(int32_t *dst, int dst_cap, int k, uint64_t key)
{
    if (k >= dst_cap) return;
    dst[2 * k] = (int32_t)(key >> 32);
    dst[2 * k + 1] = (int32_t)(key & 0xffffffffu);
}

// The pairs of bodies [lo, hi) (at most SORT_BODIES) of src[n].
__device__ void sort_run(const int2 *src, int n, int lo, int hi, int32_t *dst, int dst_cap, uint64_t *gkeys,
                         uint64_t *lds, int *word)
{
    int *end = reinterpret_cast<int *>(lds); // per body: its count, then where it starts, then where it ends
    uint64_t *seg = lds + SORT_BODIES / 2; // the run's pairs as they come, later a body's
    constexpr int SEG = SORT_LDS - SORT_BODIES / 2;
    const int tid = threadIdx.x, lane = tid & 63, nb = hi - lo;
    for (int b = tid; b < nb; b += SORT_THREADS) end[b] = 0;
    if (tid < 3) word[tid] = 0;
    __syncthreads();
    const auto sweep = [&](auto take) {
        for (int p = tid; p < n; p += SORT_AHEAD * SORT_THREADS) {
            int2 v[SORT_AHEAD];
#pragma unroll
            for (int u = 0; u < SORT_AHEAD; ++u) v[u] = src[min(p + u * SORT_THREADS, n - 1)];
#pragma unroll
            for (int u = 0; u < SORT_AHEAD; ++u)
                if (p + u * SORT_THREADS < n) take(v[u]);
        }
    };
    int below = 0;
    sweep([&](int2 v) {
        if (v.x < lo) ++below;
        else if (v.x < hi) {
            atomicAdd(&end[v.x - lo], 1);
            const int k = atomicAdd(&word[2], 1);
            if (k < SEG) seg[k] = pair_key(v);
        }
    });
    for (int o = 32; o > 0; o >>= 1) below += __shfl_xor(below, o, 64);
    if (lane == 0 && below) atomicAdd(&word[0], below);
    __syncthreads();
    const int base = word[0];
    // the counts to starts: a run of bodies per thread
    const int per = (nb + SORT_THREADS - 1) / SORT_THREADS, b0 = min(tid * per, nb), b1 = min(b0 + per, nb);
    int mine = 0, incl;
    for (int b = b0; b < b1; ++b) mine += end[b];
    incl = mine;
    for (int d = 1; d < 64; d <<= 1) {
        const int v = __shfl_up(incl, d, 64);
        if (lane >= d) incl += v;
    }
    if (lane == 63) word[3 + (tid >> 6)] = incl;
    __syncthreads();
    int at = incl - mine, total = 0;
    for (int w = 0; w < SORT_THREADS / 64; ++w) {
        at += w < (tid >> 6) ? word[3 + w] : 0;
        total += word[3 + w];
    }
    for (int b = b0; b < b1; ++b) {
        const int c = end[b];
        end[b] = at;
        at += c;
    }
    __syncthreads();
    uint64_t *keys = gkeys + base;
    if (total <= SEG) {
        for (int k = tid; k < total; k += SORT_THREADS)
            keys[atomicAdd(&end[(int)(seg[k] >> 32) - lo], 1)] = seg[k];
    } else {
        sweep([&](int2 v) {
            if (v.x >= lo && v.x < hi) keys[atomicAdd(&end[v.x - lo], 1)] = pair_key(v);
        });
    }
    __threadfence();
    __syncthreads();
    for (int q = tid; q < total; q += SORT_THREADS) {
        const uint64_t key = keys[q];
        const int b = (int)(key >> 32) - lo, s = b ? end[b - 1] : 0, e = end[b];
        if (e - s > SORT_COUNT) {
            word[1] = 1;
            continue;
        }
        int rank = 0;
        for (int k = s; k < e; ++k) rank += keys[k] < key;
        put_pair(dst, dst_cap, base + s + rank, key);
    }
    __syncthreads();
    if (word[1])
        for (int b = 0; b < nb; ++b) { // the same bodies in every thread
            const int s = b ? end[b - 1] : 0, c = end[b] - s;
            if (c <= SORT_COUNT) continue;
            const bool in_lds = c <= SEG;
            if (in_lds) {
                for (int k = tid; k < c; k += SORT_THREADS) seg[k] = keys[s + k];
                __syncthreads();
            }
            uint64_t *sorted = in_lds ? seg : keys + s;
            bitonic(sorted, c, !in_lds);
            for (int k = tid; k < c; k += SORT_THREADS) put_pair(dst, dst_cap, base + s + k, sorted[k]);
            __syncthreads();
        }
    __syncthreads(); // end and word are rewritten for the next bodies
}

__global__ __launch_bounds__(SORT_THREADS) void sort_pairs_kernel(const int32_t *src, const int32_t *src_count,
                                                                  int32_t src_cap, int n_total, int32_t *dst,
                                                                  int32_t dst_cap, int32_t *dst_count,
                                                                  uint64_t *gkeys, int32_t *flags)
{
    __shared__ uint64_t lkeys[SORT_LDS];
    __shared__ int word[3 + SORT_THREADS / 64];
    const int count = *src_count;
    const int n = min(count, src_cap);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *dst_count = count;
        if (count > src_cap) atomicOr(flags, FLAG_CAPACITY);
    }
    if (n <= 0) return;
    const int2 *pairs = reinterpret_cast<const int2 *>(src);
    if (n > SORT_SMALL) {
        const int per = (n_total + gridDim.x - 1) / gridDim.x;
        const int first = min((int)blockIdx.x * per, n_total), last = min(first + per, n_total);
        for (int lo = first; lo < last; lo += SORT_BODIES)
            sort_run(pairs, n, lo, min(lo + SORT_BODIES, last), dst, dst_cap, gkeys, lkeys, word);
        return;
    }
    if (blockIdx.x != 0) return;
    for (int k = threadIdx.x; k < n; k += SORT_THREADS) lkeys[k] = pair_key(pairs[k]);
    __syncthreads();
    bitonic(lkeys, n, false);
    for (int k = threadIdx.x; k < n; k += SORT_THREADS) put_pair(dst, dst_cap, k, lkeys[k]);
}

} // namespace

hipError_t launch_energy(const Layout &L, const EnergyPlan &e, const double *x, const double *y, const double *z,
                         const double *vx, const double *vy, const double *vz, const double *m, const double *ax,
                         const double *ay, const double *az, double vshift, double *out, hipStream_t stream)
{
    if (e.n_tasks > 0)
        energy_kernel<<<e.n_tasks, 64 * EW, 0, stream>>>(e.tasks, L.mstar, x, y, z, vx, vy, vz, m, ax, ay, az, vshift,
                                                         e.partial);
    if (e.n_runs > 0)
        energy_finish_kernel<true><<<e.n_runs, EF_THREADS, 0, stream>>>(e.runs, e.task_first, L.mstar, e.partial,
                                                                        e.n_tasks, out);
    else
        energy_finish_kernel<false><<<L.n_sys, EF_THREADS, 0, stream>>>(nullptr, e.task_first, L.mstar, e.partial,
                                                                        e.n_tasks, out);
    return hipGetLastError();
}

hipError_t launch_sort_pairs(const int32_t *src, const int32_t *src_count, int32_t src_cap, int n_total,
                             int32_t *dst, int32_t dst_cap, int32_t *dst_count, uint64_t *keys,
                             int32_t *flags, hipStream_t stream)
{
    // a workgroup per 64 bodies up to 32, then one per 128 (4000 bodies, 22185 pairs, with 32 and 62
    // workgroups 41 and 47 us, 12000, 197189 pairs, with 62, 64 and 93 160, 160 and 145); none but the
    // first where the list cannot be long
    const int most = std::max(std::min(n_total / 64, 32), std::min(n_total / 128, SORT_BLOCKS));
    const int blocks = src_cap > SORT_SMALL ? std::max(1, most) : 1;
    sort_pairs_kernel<<<blocks, SORT_THREADS, 0, stream>>>(src, src_count, src_cap, n_total, dst, dst_cap, dst_count,
                                                           keys, flags);
    return hipGetLastError();
}

} // namespace genga
