// Encounter groups of a level's pair list laid out on the device (hierarchical levels,
// Brasser et al. 2023, Sect. 1: the pairs closer than a level's critical radius form the groups
// that the next level integrates).  The groups are the connected components of the pairs, found
// by a grid-wide union-find in one launch; their members are taken in the order of the parent
// level's layout, grouped by a stable radix sort by root, and cut into tiles of 64 for the next
// level's kick.  Everything stays on the device; the host reads one small header per grouping
// (the sizes it needs to size the next launches).  A chain of small launches, bound by their
// number: rounds of hooking and compressing, a sort by root and position and two library scans were
// 32 launches, 167 us a grouping in the levels of 40322 bodies; now 13 launches, 109 us.
#include <cstring>

#include <rocprim/device/device_radix_sort.hpp>

#include "genga_internal.h"
#include "union_find.h"

namespace genga {

namespace {

constexpr int GL_THREADS = 256;
constexpr int GS_THREADS = 1024; // the kernels that count and place: their block sums are few

// Sort key of parent position p: the root of its body (n_total for a body in no pair) above p,
// which is already in order.  The labels are left at their roots; the header is cleared for the
// launches after this one.
__global__ __launch_bounds__(GL_THREADS) void group_keys_kernel(const int32_t *pbody, int Mp, int n_total,
                                                                const int32_t *pair_count, int32_t *lab,
                                                                uint64_t *keys, GroupHeader *hdr)
{
    const int p = blockIdx.x * GL_THREADS + threadIdx.x;
    if (p == 0) {
        GroupHeader h{};
        h.pair_count = *pair_count;
        *hdr = h;
    }
    if (p >= Mp) return;
    const int b = pbody[p], l = uf_load(lab, b);
    int r = n_total;
    if (l >= 0) {
        r = uf_root(lab, l);
        if (r != l) __hip_atomic_store(&lab[b], r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    keys[p] = (uint64_t)(uint32_t)r << 32 | (uint32_t)p;
}

// Whether a group starts at sorted position q, and whether q holds a member at all.
__device__ __forceinline__ bool group_start_at(const uint64_t *sorted, int q, int Mp, int n_total, bool &member)
{
    const int r = q < Mp ? (int)(sorted[q] >> 32) : n_total;
    member = r < n_total;
    return member && (q == 0 || (int)(sorted[q - 1] >> 32) != r);
}

// The sum of v over the block's threads before this one; all: over the block (every thread).
template <typename T>
__device__ __forceinline__ T block_before(T v, T *wsum, T &all)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    T incl = v;
    for (int d = 1; d < 64; d <<= 1) {
        const T u = __shfl_up(incl, d, 64);
        if (lane >= d) incl += u;
    }
    __syncthreads(); // wsum of an earlier call is no longer read
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    T before = incl - v;
    all = 0;
    for (int w = 0; w < GS_THREADS / 64; ++w) {
        before += w < wave ? wsum[w] : 0;
        all += wsum[w];
    }
    return before;
}

// Members in sorted order, and per block the number of groups that start in it; with slots the
// members' slots, and their labels back to -1.
__global__ __launch_bounds__(GS_THREADS) void group_mark_kernel(const uint64_t *sorted, int Mp, int n_total,
                                                                const int32_t *pbody, int32_t *body_out, int32_t *cnt,
                                                                int32_t *slots, int32_t *lab)
{
    __shared__ int wsum[GS_THREADS / 64];
    const int q = blockIdx.x * GS_THREADS + threadIdx.x;
    bool member;
    const bool start = group_start_at(sorted, q, Mp, n_total, member);
    if (member) {
        const int b = pbody[(int)(uint32_t)sorted[q]];
        body_out[q] = b;
        if (slots) {
            slots[b] = q;
            lab[b] = -1;
        }
    }
    int all;
    block_before((int)start, wsum, all);
    if (threadIdx.x == 0) cnt[blockIdx.x] = all;
}

// Group offsets; the last member writes the totals.
__global__ __launch_bounds__(GS_THREADS) void group_offsets_kernel(const uint64_t *sorted, int Mp, int n_total,
                                                                   const int32_t *cnt, int32_t *off, int32_t *off2,
                                                                   GroupHeader *hdr)
{
    __shared__ int wsum[GS_THREADS / 64];
    const int q = blockIdx.x * GS_THREADS + threadIdx.x;
    bool member, next;
    const bool start = group_start_at(sorted, q, Mp, n_total, member);
    group_start_at(sorted, q + 1, Mp, n_total, next);
    int part = 0, base, all;
    for (int k = threadIdx.x; k < (int)blockIdx.x; k += GS_THREADS) part += cnt[k];
    block_before(part, wsum, base);
    const int g = base + block_before((int)start, wsum, all);
    if (q == 0 && !member) off[0] = 0; // no member at all
    if (start) {
        off[g] = q;
        if (off2) off2[g] = q;
    }
    if (member && !next) {
        const int G = g + start;
        off[G] = q + 1;
        if (off2) off2[G] = q + 1;
        hdr->G = G;
        hdr->M = q + 1;
    }
}

// A group's tiles of 64 members, as (tiles of a group of several tiles) << 32 | (1 for a group of
// one tile), which the sums below count side by side.
__device__ __forceinline__ uint64_t tiles_of(int nb)
{
    const int nt = (nb + 63) / 64;
    return nt > 1 ? (uint64_t)nt << 32 : (uint64_t)nt;
}

// A group among those of at least `least` members, as 1 << 32 | its members.
__device__ __forceinline__ uint64_t large_of(int nb, int least) { return nb >= least ? 1ull << 32 | (uint32_t)nb : 0; }

// The largest group into the header, and per block the groups' tiles, or the large groups and their
// members (bsum[2 block]) and tiles.
__global__ __launch_bounds__(GS_THREADS) void group_sizes_kernel(const int32_t *off, GroupHeader *hdr, uint64_t *tsum,
                                                                 uint64_t *bsum, int least)
{
    __shared__ uint64_t wsum[GS_THREADS / 64];
    const int g = blockIdx.x * GS_THREADS + threadIdx.x, G = hdr->G;
    if ((int)blockIdx.x * GS_THREADS >= G) return; // the whole block
    const int nb = g < G ? off[g + 1] - off[g] : 0;
    int mx = nb;
    for (int o = 32; o > 0; o >>= 1) mx = max(mx, __shfl_xor(mx, o, 64));
    if ((threadIdx.x & 63) == 0) atomicMax(&hdr->max_nb, mx);
    uint64_t all;
    if (tsum) {
        block_before(tiles_of(nb), wsum, all);
        if (threadIdx.x == 0) tsum[blockIdx.x] = all;
    }
    if (bsum) {
        block_before(large_of(nb, least), wsum, all);
        if (threadIdx.x == 0) bsum[2 * blockIdx.x] = all;
        block_before((uint64_t)(nb >= least ? (nb + 63) / 64 : 0), wsum, all);
        if (threadIdx.x == 0) bsum[2 * blockIdx.x + 1] = all;
    }
}

// The tiles t0 .. of a group of nb members from member o on, by the wave, for every lane whose
// group has any (want): tile k of a lane's group goes to put(tile index, tile, list place).
template <typename Put>
__device__ __forceinline__ void wave_tiles(bool want, int g, int o, int nb, int t0, int l0, Put put)
{
    const int lane = threadIdx.x & 63;
    for (unsigned long long w = __ballot(want); w; w &= w - 1) {
        const int src = __builtin_ctzll(w);
        const int g1 = __shfl(g, src, 64), o1 = __shfl(o, src, 64), nb1 = __shfl(nb, src, 64);
        const int t1 = __shfl(t0, src, 64), l1 = __shfl(l0, src, 64);
        for (int k = lane; 64 * k < nb1; k += 64) put(t1 + k, make_int4(g1, o1 + 64 * k, min(64, nb1 - 64 * k), 0), l1 + k);
    }
}

// The layout of the groups of at least `least` members for the grid-wide drift: their first members
// in the layout of all (k0), their offsets in their own, tiles and sizes.
__global__ __launch_bounds__(GS_THREADS) void group_large_kernel(const int32_t *off, GroupHeader *hdr,
                                                                 const uint64_t *bsum, LargeOut out)
{
    __shared__ uint64_t wsum[GS_THREADS / 64];
    const int g = blockIdx.x * GS_THREADS + threadIdx.x, G = hdr->G;
    const int nblk = (G + GS_THREADS - 1) / GS_THREADS;
    if ((int)blockIdx.x >= nblk) return; // the whole block
    const int o = g < G ? off[g] : 0, nb = g < G ? off[g + 1] - o : 0;
    const bool large = nb >= out.least;
    uint64_t p = 0, tp = 0, base, tbase, all, tall;
    for (int k = threadIdx.x; k < (int)blockIdx.x; k += GS_THREADS) {
        p += bsum[2 * k];
        tp += bsum[2 * k + 1];
    }
    block_before(p, wsum, base);
    block_before(tp, wsum, tbase);
    const uint64_t e = base + block_before(large_of(nb, out.least), wsum, all);
    const int t0 = (int)(tbase + block_before((uint64_t)(large ? (nb + 63) / 64 : 0), wsum, tall));
    const int gi = (int)(e >> 32), f0 = (int)(uint32_t)e;
    if (large) {
        out.k0[gi] = o;
        out.off[gi] = f0;
        out.tfirst[gi] = t0;
    }
    wave_tiles(large, gi, f0, nb, t0, 0, [&](int t, int4 tile, int) { out.tiles[t] = tile; });
    if (g == G - 1) {
        const uint64_t tot = base + all;
        const int nG = (int)(tot >> 32), nM = (int)(uint32_t)tot, nT = (int)(tbase + tall);
        out.off[nG] = nM;
        out.tfirst[nG] = nT;
        out.dims[0] = hdr->large_G = nG;
        out.dims[1] = hdr->large_M = nM;
        out.dims[2] = hdr->large_T = nT;
    }
}

// Tiles of 64 members, group by group: each group's first tile (tfirst), its tiles, their places
// in the launch list tl (the tiles of groups of several tiles first, a workgroup each, then the
// tile of every group of one tile, a wave each), and the header's tile counts.
__global__ __launch_bounds__(GS_THREADS) void group_tiles_kernel(const int32_t *off, GroupHeader *hdr,
                                                                 const uint64_t *tsum, int32_t *tfirst, int4 *tiles,
                                                                 int32_t *tl)
{
    __shared__ uint64_t wsum[GS_THREADS / 64];
    const int g = blockIdx.x * GS_THREADS + threadIdx.x, G = hdr->G;
    const int nblk = (G + GS_THREADS - 1) / GS_THREADS;
    if ((int)blockIdx.x >= nblk) return; // the whole block
    uint64_t part = 0, rest = 0, base, after, all;
    for (int k = threadIdx.x; k < nblk; k += GS_THREADS) (k < (int)blockIdx.x ? part : rest) += tsum[k];
    block_before(part, wsum, base);
    block_before(rest, wsum, after);
    const int o = g < G ? off[g] : 0, nb = g < G ? off[g + 1] - o : 0, nt = (nb + 63) / 64;
    const uint64_t e = base + block_before(tiles_of(nb), wsum, all), tot = base + after;
    const int mo = (int)(e >> 32), so = (int)(uint32_t)e;
    const int n_multi = (int)(tot >> 32), n_tiles = n_multi + (int)(uint32_t)tot;
    if (g < G) tfirst[g] = mo + so;
    if (g == G - 1) {
        tfirst[G] = n_tiles;
        hdr->n_tiles = n_tiles;
        hdr->n_multi = n_multi;
    }
    if (nt == 1) {
        tiles[mo + so] = make_int4(g, o, nb, 0);
        tl[n_multi + so] = mo + so;
    }
    wave_tiles(nt > 1, g, o, nb, mo + so, mo, [&](int t, int4 tile, int l) {
        tiles[t] = tile;
        tl[l] = t;
    });
}

int bits_for(uint64_t v)
{
    int b = 0;
    while (b < 64 && (v >> b) != 0) ++b;
    return b;
}


// a monotone stand-in for atan2(y, x) on [0, 4)
__device__ __forceinline__ double pseudo_angle(double x, double y)
{
    const double s = fabs(x) + fabs(y);
    if (!(s > 0.0)) return 0.0;
    const double t = y / s; // in [-1, 1]
    return x >= 0.0 ? (y >= 0.0 ? t : 4.0 + t) : 2.0 - t;
}

// The group of layout position p: the last gi with off[gi] <= p (empty groups share their
// offset with the next one and are passed over).
__device__ __forceinline__ int group_of(const int32_t *off, int n_groups, int p)
{
    int lo = 0, hi = n_groups - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= p) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ int ring_body(const int32_t *members, const int32_t *k0, const int32_t *off, int gi,
                                         int p)
{
    const int m = k0[gi] + (p - off[gi]);
    return members ? members[m] : m;
}

__global__ __launch_bounds__(256) void ring_bounds_clear_kernel(int n_groups, uint64_t *bounds)
{
    for (int g = blockIdx.x * 256 + threadIdx.x; g < n_groups; g += gridDim.x * 256) {
        bounds[2 * g] = 0x7ff0000000000000ull; // +inf: the smallest distance so far
        bounds[2 * g + 1] = 0ull;              // +0
    }
}

// Each group's smallest and largest distance to the star over the layout positions: a wave
// whose lanes share one group reduces first; the atomics order the bit patterns, which for
// non-negative doubles is the numeric order, so the result does not depend on the order.
__global__ __launch_bounds__(256) void ring_bounds_kernel(const int32_t *members, const int32_t *k0,
                                                          const int32_t *off, int n_groups, int M, const double *x,
                                                          const double *y, uint64_t *bounds)
{
#pragma clang fp contract(off)
    const int stride = gridDim.x * 256;
    for (int base = blockIdx.x * 256; base < M; base += stride) {
        const int p = base + (int)threadIdx.x;
        const bool on = p < M;
        const int gi = on ? group_of(off, n_groups, p) : 0;
        double r0 = INFINITY, r1 = 0.0;
        if (on) {
            const int bi = ring_body(members, k0, off, gi, p);
            r0 = r1 = sqrt(x[bi] * x[bi] + y[bi] * y[bi]);
        }
        const int g0 = __builtin_amdgcn_readfirstlane(gi);
        const unsigned long long act = __ballot(true);
        if (__ballot(on && gi == g0) == act) {
            for (int d = 32; d > 0; d >>= 1) {
                r0 = fmin(r0, __shfl_xor(r0, d, 64));
                r1 = fmax(r1, __shfl_xor(r1, d, 64));
            }
            if ((threadIdx.x & 63) == 0) {
                atomicMin((unsigned long long *)&bounds[2 * g0], (unsigned long long)__double_as_longlong(r0));
                atomicMax((unsigned long long *)&bounds[2 * g0 + 1], (unsigned long long)__double_as_longlong(r1));
            }
        } else if (on) {
            atomicMin((unsigned long long *)&bounds[2 * gi], (unsigned long long)__double_as_longlong(r0));
            atomicMax((unsigned long long *)&bounds[2 * gi + 1], (unsigned long long)__double_as_longlong(r1));
        }
    }
}

// Per layout position: the member's key (gi, ring, azimuth) and body.  The rings are
// equal-width bands of distance to the star, as many as make a tile of 64 members about as
// wide as long (the band's circumference taken at the middle of the group's range); the
// quantised (ring + azimuth / 4) / rings orders the members.
__global__ __launch_bounds__(256) void ring_keys_kernel(const int32_t *members, const int32_t *k0, const int32_t *off,
                                                        int n_groups, int M, const double *x, const double *y,
                                                        const uint64_t *bounds, uint64_t *key, int32_t *val)
{
#pragma clang fp contract(off)
    for (int p = blockIdx.x * 256 + threadIdx.x; p < M; p += gridDim.x * 256) {
        const int gi = group_of(off, n_groups, p);
        const int bi = ring_body(members, k0, off, gi, p);
        const int nb = off[gi + 1] - off[gi];
        const double r0 = __longlong_as_double((long long)bounds[2 * gi]);
        const double r1 = __longlong_as_double((long long)bounds[2 * gi + 1]);
        const double width = fmax(r1 - r0, 1e-300), rmid = fmax(0.5 * (r0 + r1), 1e-300);
        const double nr = fmin(sqrt(nb * width / (64.0 * 2.0 * M_PI * rmid)), 1048576.0);
        const int rings = max(1, (int)lround(nr));
        const double r = sqrt(x[bi] * x[bi] + y[bi] * y[bi]);
        const int ring = min(rings - 1, (int)((r - r0) / width * rings));
        const double u = (ring + 0.25 * pseudo_angle(x[bi], y[bi])) / rings; // [0, 1]
        const uint64_t q = (uint64_t)fmin(4294967295.0, fmax(0.0, u * 4294967295.0));
        key[p] = (uint64_t)gi << 32 | q;
        val[p] = bi;
    }
}

} // namespace

hipError_t group_work_alloc(GroupWork &w, int cap)
{
    group_work_free(w);
    w.cap = cap > 1 ? cap : 2;
    const size_t n = (size_t)w.cap;
    hipError_t e;
    if ((e = hipMalloc((void **)&w.keys, n * sizeof(uint64_t))) != hipSuccess) return e;
    if ((e = hipMalloc((void **)&w.keys_sorted, n * sizeof(uint64_t))) != hipSuccess) return e;
    const size_t nb = (n + GS_THREADS - 1) / GS_THREADS;
    if ((e = hipMalloc((void **)&w.cnt, nb * sizeof(int32_t))) != hipSuccess) return e;
    if ((e = hipMalloc((void **)&w.tsum, nb * sizeof(uint64_t))) != hipSuccess) return e;
    if ((e = hipMalloc((void **)&w.bsum, 2 * nb * sizeof(uint64_t))) != hipSuccess) return e;
    if ((e = hipMalloc((void **)&w.hdr, sizeof(GroupHeader))) != hipSuccess) return e;
    // temporary storage of the sort, for the largest size
    if ((e = rocprim::radix_sort_keys(nullptr, w.temp_bytes, w.keys, w.keys_sorted, (unsigned int)n, 0, 64)) !=
        hipSuccess)
        return e;
    if ((e = hipMalloc(&w.temp, w.temp_bytes ? w.temp_bytes : 1)) != hipSuccess) return e;
    return hipSuccess;
}

void group_work_free(GroupWork &w)
{
    for (void *p : {(void *)w.keys, (void *)w.keys_sorted, (void *)w.cnt, (void *)w.tsum, (void *)w.bsum,
                    (void *)w.hdr, w.temp})
        if (p) (void)hipFree(p);
    w = GroupWork{};
}

hipError_t launch_group_layout(const Layout &L, GroupWork &w, const int32_t *pairs, const int32_t *pair_count,
                               int32_t pair_cap, int32_t *lab, const int32_t *pbody, int Mp, const GroupOut &out,
                               hipStream_t stream)
{
    if (Mp > w.cap) return hipErrorInvalidValue;
    if (Mp <= 0) return hipMemsetAsync(w.hdr, 0, sizeof(GroupHeader), stream);
    hipError_t e;
    if ((e = launch_uf_union(pairs, pair_count, pair_cap, lab, stream)) != hipSuccess) return e;
    const int nb = (Mp + GL_THREADS - 1) / GL_THREADS, ns = (Mp + GS_THREADS - 1) / GS_THREADS;
    group_keys_kernel<<<nb, GL_THREADS, 0, stream>>>(pbody, Mp, L.n_total, pair_count, lab, w.keys, w.hdr);
    // the positions below the roots are in order: only the roots' bits are sorted
    size_t bytes = w.temp_bytes;
    if ((e = rocprim::radix_sort_keys(w.temp, bytes, w.keys, w.keys_sorted, (unsigned int)Mp, 32,
                                      32 + bits_for((uint64_t)L.n_total), stream)) != hipSuccess)
        return e;
    group_mark_kernel<<<ns, GS_THREADS, 0, stream>>>(w.keys_sorted, Mp, L.n_total, pbody, out.body, w.cnt,
                                                   out.member_slot, lab);
    group_offsets_kernel<<<ns, GS_THREADS, 0, stream>>>(w.keys_sorted, Mp, L.n_total, w.cnt, out.off, out.off2, w.hdr);
    // groups have at least two members
    const int ng = (Mp / 2 + GS_THREADS) / GS_THREADS;
    group_sizes_kernel<<<ng, GS_THREADS, 0, stream>>>(out.off, w.hdr, out.tiles ? w.tsum : nullptr,
                                                    out.large.k0 ? w.bsum : nullptr, out.large.least);
    if (out.tiles)
        group_tiles_kernel<<<ng, GS_THREADS, 0, stream>>>(out.off, w.hdr, w.tsum, out.tfirst, out.tiles, out.tl);
    if (out.large.k0) group_large_kernel<<<ng, GS_THREADS, 0, stream>>>(out.off, w.hdr, w.bsum, out.large);
    return hipGetLastError();
}

hipError_t order_work_alloc(OrderWork &w, int cap)
{
    order_work_free(w);
    w.cap = cap > 1 ? cap : 2;
    const size_t n = (size_t)w.cap;
    hipError_t e;
    if ((e = hipMalloc((void **)&w.keys, n * sizeof(uint64_t))) != hipSuccess) return e;
    if ((e = hipMalloc((void **)&w.keys_sorted, n * sizeof(uint64_t))) != hipSuccess) return e;
    if ((e = hipMalloc((void **)&w.vals, n * sizeof(int32_t))) != hipSuccess) return e;
    if ((e = hipMalloc((void **)&w.bounds, 2 * n * sizeof(uint64_t))) != hipSuccess) return e;
    int32_t *out = nullptr;
    if ((e = rocprim::radix_sort_pairs(nullptr, w.temp_bytes, w.keys, w.keys_sorted, w.vals, out, (unsigned int)n, 0,
                                       64)) != hipSuccess)
        return e;
    return hipMalloc(&w.temp, w.temp_bytes ? w.temp_bytes : 1);
}

void order_work_free(OrderWork &w)
{
    for (void *p : {(void *)w.keys, (void *)w.keys_sorted, (void *)w.vals, (void *)w.bounds, w.temp})
        if (p) (void)hipFree(p);
    w = OrderWork{};
}

hipError_t launch_ring_order(const int32_t *members, const int32_t *k0, const int32_t *off, int n_groups, int M,
                             const double *x, const double *y, OrderWork &w, int32_t *body_out, hipStream_t stream)
{
    if (n_groups <= 0 || M <= 0) return hipSuccess;
    if (M > w.cap || n_groups > w.cap) return hipErrorInvalidValue;
    const int grid = std::min((M + 255) / 256, 2048);
    ring_bounds_clear_kernel<<<std::min((n_groups + 255) / 256, 256), 256, 0, stream>>>(n_groups, w.bounds);
    ring_bounds_kernel<<<grid, 256, 0, stream>>>(members, k0, off, n_groups, M, x, y, w.bounds);
    ring_keys_kernel<<<grid, 256, 0, stream>>>(members, k0, off, n_groups, M, x, y, w.bounds, w.keys, w.vals);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    size_t bytes = w.temp_bytes;
    return rocprim::radix_sort_pairs(w.temp, bytes, w.keys, w.keys_sorted, w.vals, body_out, (unsigned int)M, 0,
                                     32 + bits_for((uint64_t)n_groups), stream);
}

} // namespace genga
