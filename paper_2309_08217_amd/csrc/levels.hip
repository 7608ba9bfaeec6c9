// Kicks of the intermediate levels of the hierarchical step (Brasser et al. 2023, Sect. 1:
// symplectic levels with reduced steps between the level-0 step and the Bulirsch-Stoer step).
// Level l integrates each group of level l-1 in Strang sub-steps; its kick carries the share
// W_l K_l of the Newtonian pair force, W_l = prod_{k<l} (1 - K_k), K_k the changeover of
// level k's critical radius, and the same pass lists the pairs of the group closer than the
// level's critical radius (the next level's groups).  FP64 throughout: these are
// close-encounter forces.
//
// Layout as in the grid-wide Bulirsch-Stoer: the members of the parent groups are ordered by
// ring and azimuth (on the device, once per step, and passed on from level to level) and cut into
// tiles of 64.  In a
// group of several tiles a workgroup of 16 waves (4 when such tiles outnumber the CUs, so that
// several workgroups share a CU) takes one target tile, lists the source tiles
// of the group whose box lies within the group's largest level-(l-1) radius of the target
// tile's box (no pair beyond that radius carries weight at level l), then the sources in reach of
// the box in them, and deals these out to its waves, four at a time; a group of one tile is one
// wave, its members the sources in order.
#include "genga_internal.h"
#include "pair_math.h"

namespace genga {

namespace {

constexpr int LT_TILE = 64;

// Per member f: mass, TP2 flag, the radii of levels 0..level; per group: the largest
// level-(level-1) radius squared, as the maximum over its tiles (bit patterns of non-negative
// doubles order as the values, so an integer atomic max gives the exact maximum).  One wave
// per tile; cut2 cleared first.
__global__ __launch_bounds__(256) void level_cut_clear_kernel(double *cut2, int G)
{
    const int g = blockIdx.x * 256 + threadIdx.x;
    if (g < G) cut2[g] = 0.0;
}

__global__ __launch_bounds__(64) void level_tiles_setup_kernel(LevelTiles t, const int32_t *sys_of,
                                                               const int32_t *sys_off, const int32_t *n_massive,
                                                               const double *m, const double *rc0,
                                                               const double *rcl, int n_total, int level)
{
    const int4 tile = t.tiles[blockIdx.x];
    double mx = 0.0;
    if ((int)threadIdx.x < tile.z) {
        const int f = tile.y + threadIdx.x, body = t.body[f], s = sys_of[body];
        t.mass[f] = m[body];
        t.test[f] = body - sys_off[s] >= n_massive[s];
        for (int k = 0; k <= level; ++k) {
            const double r = k == 0 ? rc0[body] : rcl[(size_t)(k - 1) * n_total + body];
            t.rc[(size_t)k * t.cap_M + f] = r;
            t.i9[(size_t)k * t.cap_M + f] = 1.0 / (0.9 * r);
        }
        mx = fmax(0.0, sq_rn(t.rc[(size_t)(level - 1) * t.cap_M + f]));
    }
    mx = wave_maxv(mx);
    if (threadIdx.x == 0)
        atomicMax((unsigned long long *)&t.cut2[tile.x], (unsigned long long)__double_as_longlong(mx));
}

// Positions of the members of each tile, and the tile's box.  One wave per tile.
__global__ __launch_bounds__(64) void level_tiles_pos_kernel(LevelTiles t, const double *x, const double *y,
                                                             const double *z, int32_t *clear)
{
    const int me = blockIdx.x;
    if (clear && me == 0 && threadIdx.x == 0) *clear = 0; // the kick after this launch appends pairs
    const int4 tile = t.tiles[me];
    const bool v = (int)threadIdx.x < tile.z;
    const int f = tile.y + (v ? (int)threadIdx.x : 0);
    const int body = t.body[f];
    const double px = x[body], py = y[body], pz = z[body];
    if (v) {
        t.X[f] = px;
        t.Y[f] = py;
        t.Z[f] = pz;
    }
    tile_box(v, px, py, pz, t.bb, me);
}

// The level's pairs found by a wave collect in its own LDS buffer and reach the list in
// blocks, one counter update per block: the pairs of a level kick over a whole disc number
// ~10^5, and one update per wave and source had queued on the counter.  Every lane of the
// wave takes part in each call (the fill count is the same in every lane).
constexpr int LV_BUF = 128;

__device__ __forceinline__ void lv_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ void lv_store(const LevelKickArgs &a, int idx, int2 p)
{
    if (idx < a.pair_cap) {
        a.pairs[2 * idx] = p.x;
        a.pairs[2 * idx + 1] = p.y;
    } else {
        atomicOr(a.flags, FLAG_CAPACITY);
    }
}

__device__ __forceinline__ void lv_flush(const LevelKickArgs &a, int2 *buf, int &fill)
{
    if (fill == 0) return;
    lv_wave_sync();
    const int lane = threadIdx.x & 63;
    int base = 0;
    if (lane == 0) base = atomicAdd(a.pair_count, fill);
    base = __shfl(base, 0, 64);
    for (int k = lane; k < fill; k += 64) lv_store(a, base + k, buf[k]);
    lv_wave_sync();
    fill = 0;
}

__device__ __forceinline__ void lv_emit(const LevelKickArgs &a, int2 *buf, int &fill, bool em, int i, int j)
{
    const unsigned long long m = __ballot(em);
    if (!m) return;
    const int c = __popcll(m);
    if (fill + c > LV_BUF) lv_flush(a, buf, fill);
    if (em) buf[fill + __popcll(m & ((1ull << (threadIdx.x & 63)) - 1))] = make_int2(i, j);
    fill += c;
}

// One target member (a lane) of a level kick.
struct LvTarget {
    bool valid, test;
    int f, body;
    double x, y, z;
    double i9[LEVELS_MAX]; // 1 / (0.9 radius) of levels 0..level (0 above)
    double rc_up, rc_lv;   // the radii of level - 1 and level
};

__device__ __forceinline__ LvTarget lv_target(const LevelTiles &t, int4 tile, int lv)
{
    LvTarget me;
    const int lane = threadIdx.x & 63;
    me.valid = lane < tile.z;
    me.f = tile.y + (me.valid ? lane : 0);
    me.body = t.body[me.f];
    me.x = t.X[me.f];
    me.y = t.Y[me.f];
    me.z = t.Z[me.f];
    me.test = t.test[me.f] != 0;
#pragma unroll
    for (int k = 0; k < LEVELS_MAX; ++k) me.i9[k] = k <= lv ? t.i9[(size_t)k * t.cap_M + me.f] : 0.0;
    me.rc_up = t.rc[(size_t)(lv - 1) * t.cap_M + me.f];
    me.rc_lv = t.rc[(size_t)lv * t.cap_M + me.f];
    return me;
}

// A source member's words.
struct LvSource {
    double x, y, z, m;
    double i9[LEVELS_MAX];
    double rc_up, rc_lv;
    int f, body, test;
};

// Whether the source is inside level (l-1)'s radius of the target.
__device__ __forceinline__ bool lv_inside(const LvTarget &me, const LvSource &j)
{
    const double q = sep2_rn(j.x - me.x, j.y - me.y, j.z - me.z);
    return me.valid && j.f != me.f && !(me.test && j.test != 0) && q < sq_rn(fmax(me.rc_up, j.rc_up));
}

// The term of a source inside (has) for the target, and the level's pair.  Every lane of the wave
// calls it, with a source of its own.
__device__ __forceinline__ void lv_source(const LevelKickArgs &a, const LvTarget &me, int lv, bool has,
                                          const LvSource &j, double &ax, double &ay, double &az, int2 *buf, int &fill)
{
    bool em = false;
    if (has) {
        const double dx = j.x - me.x, dy = j.y - me.y, dz = j.z - me.z;
        const double q = sep2_rn(dx, dy, dz);
        // W_l K_l = prod_{k<l} u_k^2 / d_k times y_l^2 / d_l (loops over the fixed bound, so the
        // radii stay in registers)
        const double rq = inv_sqrt64(q), r = q * rq;
        double n = 1.0, d = 1.0;
#pragma unroll
        for (int k = 0; k < LEVELS_MAX; ++k) {
            if (k > lv) break;
            const Changeover c = changeover_parts(r, fmin(me.i9[k], j.i9[k]));
            n *= k < lv ? c.u : c.y;
            d *= c.d;
        }
        // (a weight of zero is no term, also at zero separation, where r^-3 is not finite)
        const double s = n > 0.0 ? j.m * (n * n) * inv64(d) * ((rq * rq) * rq) : 0.0;
        ax = fma(s, dx, ax);
        ay = fma(s, dy, ay);
        az = fma(s, dz, az);
        em = a.emit && me.body < j.body && q < sq_rn(fmax(me.rc_lv, j.rc_lv));
    }
    lv_emit(a, buf, fill, em, me.body, j.body);
}

// The words of member f.
__device__ __forceinline__ LvSource lv_load(const LevelTiles &t, int lv, int f)
{
    LvSource s;
    s.x = t.X[f];
    s.y = t.Y[f];
    s.z = t.Z[f];
    s.m = t.mass[f];
#pragma unroll
    for (int k = 0; k < LEVELS_MAX; ++k) s.i9[k] = k <= lv ? t.i9[(size_t)k * t.cap_M + f] : 0.0;
    s.rc_up = t.rc[(size_t)(lv - 1) * t.cap_M + f];
    s.rc_lv = t.rc[(size_t)lv * t.cap_M + f];
    s.f = f;
    s.body = t.body[f];
    s.test = t.test[f];
    return s;
}

// Sources in LDS.
template <int N>
struct LvStage {
    double2 xy[N], zm[N], rr[N], i9[N][LEVELS_MAX / 2];
    int2 fb[N]; // member, body (a test body's bits flipped)
    __device__ __forceinline__ void put(int e, const LvSource &s)
    {
        xy[e] = make_double2(s.x, s.y);
        zm[e] = make_double2(s.z, s.m);
        rr[e] = make_double2(s.rc_up, s.rc_lv);
#pragma unroll
        for (int k = 0; k < LEVELS_MAX; k += 2) i9[e][k / 2] = make_double2(s.i9[k], s.i9[k + 1]);
        fb[e] = make_int2(s.f, s.test ? ~s.body : s.body);
    }
    __device__ __forceinline__ LvSource get(int e) const
    {
        LvSource s;
        s.x = xy[e].x;
        s.y = xy[e].y;
        s.z = zm[e].x;
        s.m = zm[e].y;
        s.rc_up = rr[e].x;
        s.rc_lv = rr[e].y;
#pragma unroll
        for (int k = 0; k < LEVELS_MAX; k += 2) {
            s.i9[k] = i9[e][k / 2].x;
            s.i9[k + 1] = i9[e][k / 2].y;
        }
        s.f = fb[e].x;
        s.test = fb[e].y < 0;
        s.body = s.test ? ~fb[e].y : fb[e].y;
        return s;
    }
};
static_assert(LEVELS_MAX % 2 == 0, "levels in pairs");

// The terms of the staged sources e0, e0 + step, .. below n: the wave marks up to 64 of them per
// target, then every lane works through its own marks.  (With the term behind the test a wave does
// it for almost every source, for a quarter of its lanes.)
template <int N>
__device__ __forceinline__ void lv_sources(const LevelKickArgs &a, const LvTarget &me, int lv, const LvStage<N> &stage,
                                           int e0, int step, int n, double &ax, double &ay, double &az, int2 *buf,
                                           int &fill)
{
    for (int b = e0; b < n; b += 64 * step) {
        unsigned long long m = 0;
        for (int k = 0; k < 64 && b + k * step < n; ++k)
            if (lv_inside(me, stage.get(b + k * step))) m |= 1ull << k;
        while (__ballot(m != 0)) {
            const bool has = m != 0;
            const int k = has ? __builtin_ctzll(m) : 0;
            m &= m - 1; // (zero stays zero)
            lv_source(a, me, lv, has, stage.get(b + k * step), ax, ay, az, buf, fill);
        }
    }
}

// Groups of more than one tile: one workgroup of W waves per target tile (tiles listed first
// in t.tl).  Bound by the FP64 arithmetic of the pairs.  A tile's own radius around its box holds
// about half of the sources of the tiles it touches, so they are sorted out first, a lane each, and
// staged in LDS for the marks and the terms (lv_sources).  Kicks of 40322 bodies: 62 us with every
// source of the tiles through scalar loads and the term behind the test; 55 with the sources sorted
// out; 42 with marks; 33 with one update of the pair counter a workgroup in place of one a wave (they
// follow each other at about 10 ns).
constexpr int LV_CAND = 32; // source tiles at a time
template <int W>
__global__ __launch_bounds__(LT_TILE *W) void level_tiles_kick_kernel(LevelTiles t, LevelKickArgs a)
{
    __shared__ uint16_t near_tile[BIG_TILES_PER_GROUP];
    __shared__ uint16_t live[LV_CAND * LT_TILE]; // (source tile, source), in order
    __shared__ union {
        LvStage<W * LT_TILE> stage;
        double red[3][W][LT_TILE]; // once the sources are done
    } S;
    __shared__ int wave_cnt[W], pair_base;
    __shared__ int2 pair_buf[W][LV_BUF];
    const int me = t.tl[blockIdx.x];
    const int4 tile = t.tiles[me]; // (group, first member, count, -)
    const int g = tile.x;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int o = t.off[g], nb = t.off[g + 1] - o;
    const int tf = t.tfirst[g], nt = t.tfirst[g + 1] - tf;
    const int lv = a.level;
    const LvTarget tg = lv_target(t, tile, lv);
    const double cut = t.cut2[g] * (1.0 + 0x1p-30);
    const double *bt = t.bb + (size_t)me * 8;
    const double tlx = bt[0], tly = bt[1], tlz = bt[2], thx = bt[3], thy = bt[4], thz = bt[5];
    const auto outside = [&](double lx, double ly, double lz, double hx, double hy, double hz) {
        const double gx = fmax(0.0, fmax(lx - thx, tlx - hx));
        const double gy = fmax(0.0, fmax(ly - thy, tly - hy));
        const double gz = fmax(0.0, fmax(lz - thz, tlz - hz));
        return (gx * gx + gy * gy) + gz * gz;
    };
    // the place of a thread's item in the order of the threads after n_all earlier ones
    const auto place = [&](bool is, int &n_all) {
        const unsigned long long bal = __ballot(is);
        if (lane == 0) wave_cnt[wave] = __popcll(bal);
        __syncthreads();
        int pos = n_all + __popcll(bal & ((1ull << lane) - 1));
        for (int w = 0; w < W; ++w) {
            if (w < wave) pos += wave_cnt[w];
            n_all += wave_cnt[w];
        }
        __syncthreads();
        return pos;
    };
    // source tiles of the group in reach: one test per thread (in passes of W * 64 tiles)
    int n_near = 0;
    for (int t0 = 0; t0 < nt; t0 += W * LT_TILE) {
        const int tt = t0 + (int)threadIdx.x;
        bool near = false;
        if (tt < nt) {
            const double *bs = t.bb + (size_t)(tf + tt) * 8;
            near = outside(bs[0], bs[1], bs[2], bs[3], bs[4], bs[5]) <= cut;
        }
        const int pos = place(near, n_near);
        if (near) near_tile[pos] = (uint16_t)tt;
    }
    __syncthreads();
    int2 *buf = pair_buf[wave];
    int fill = 0;
    double ax = 0.0, ay = 0.0, az = 0.0;
    const double *up = t.rc + (size_t)(lv - 1) * t.cap_M;
    const double up2 = wave_maxv(tg.valid ? sq_rn(tg.rc_up) : 0.0);
    for (int c0 = 0; c0 < n_near; c0 += LV_CAND) {
        int n_live = 0;
        for (int c = 0; c < min(LV_CAND, n_near - c0); c += W) { // a source tile per wave, a source per lane
            bool is = false;
            if (c0 + c + wave < n_near && c + wave < LV_CAND) {
                const int s = LT_TILE * near_tile[c0 + c + wave] + lane;
                if (s < nb) {
                    const int f = o + s;
                    const double x = t.X[f], y = t.Y[f], z = t.Z[f];
                    is = outside(x, y, z, x, y, z) <= fmax(up2, sq_rn(up[f])) * (1.0 + 0x1p-30);
                }
            }
            const int pos = place(is, n_live);
            if (is) live[pos] = (uint16_t)((c + wave) * LT_TILE + lane);
        }
        __syncthreads();
        for (int l0 = 0; l0 < n_live; l0 += W * LT_TILE) {
            const int n = min(W * LT_TILE, n_live - l0);
            if ((int)threadIdx.x < n) {
                const int e = live[l0 + threadIdx.x];
                S.stage.put(threadIdx.x, lv_load(t, lv, o + LT_TILE * near_tile[c0 + e / LT_TILE] + e % LT_TILE));
            }
            __syncthreads();
            lv_sources(a, tg, lv, S.stage, wave, W, n, ax, ay, az, buf, fill);
            __syncthreads(); // stage (and at last live) is rewritten
        }
        if (n_live == 0) __syncthreads(); // near_tile has been read by every wave
    }
    // the sums, and the waves' pairs with one counter update for all of them
    if (lane == 0) wave_cnt[wave] = fill;
    S.red[0][wave][lane] = ax;
    S.red[1][wave][lane] = ay;
    S.red[2][wave][lane] = az;
    __syncthreads();
    int before = 0, all = 0;
    for (int w = 0; w < W; ++w) {
        if (w < wave) before += wave_cnt[w];
        all += wave_cnt[w];
    }
    if (threadIdx.x == 0 && all > 0) pair_base = atomicAdd(a.pair_count, all);
    if (wave == 0 && tg.valid) {
        double sx = 0.0, sy = 0.0, sz = 0.0;
        for (int w = 0; w < W; ++w) {
            sx += S.red[0][w][lane];
            sy += S.red[1][w][lane];
            sz += S.red[2][w][lane];
        }
        a.vx[tg.body] += a.tau * sx;
        a.vy[tg.body] += a.tau * sy;
        a.vz[tg.body] += a.tau * sz;
    }
    __syncthreads();
    for (int k = lane; k < fill; k += 64) lv_store(a, pair_base + before + k, buf[k]);
}

// Groups of one tile (up to 64 members): one wave per group, its members the sources in order.
__global__ __launch_bounds__(LT_TILE) void level_tile_one_kernel(LevelTiles t, LevelKickArgs a)
{
    __shared__ int2 buf[LV_BUF];
    __shared__ LvStage<LT_TILE> stage;
    const int4 tile = t.tiles[t.tl[t.n_multi + blockIdx.x]];
    const LvTarget tg = lv_target(t, tile, a.level);
    if (tg.valid) stage.put(threadIdx.x, lv_load(t, a.level, tg.f));
    __syncthreads();
    int fill = 0;
    double ax = 0.0, ay = 0.0, az = 0.0;
    lv_sources(a, tg, a.level, stage, 0, 1, tile.z, ax, ay, az, buf, fill);
    lv_flush(a, buf, fill);
    if (!tg.valid) return;
    a.vx[tg.body] += a.tau * ax;
    a.vy[tg.body] += a.tau * ay;
    a.vz[tg.body] += a.tau * az;
}

} // namespace

hipError_t launch_level_tiles_setup(const Layout &L, const LevelTiles &t, const double *m, const double *rc0,
                                    const double *rcl, int level, hipStream_t stream)
{
    if (t.G == 0 || t.n_tiles == 0) return hipSuccess;
    level_cut_clear_kernel<<<(t.G + 255) / 256, 256, 0, stream>>>(t.cut2, t.G);
    level_tiles_setup_kernel<<<t.n_tiles, 64, 0, stream>>>(t, L.sys_of, L.sys_off, L.n_massive, m, rc0, rcl,
                                                           L.n_total, level);
    return hipGetLastError();
}

hipError_t launch_level_kick(const LevelTiles &t, const LevelKickArgs &a, const double *x, const double *y,
                             const double *z, int waves, hipStream_t stream)
{
    if (t.n_tiles == 0) return a.emit ? hipMemsetAsync(a.pair_count, 0, sizeof(int32_t), stream) : hipSuccess;
    level_tiles_pos_kernel<<<t.n_tiles, 64, 0, stream>>>(t, x, y, z, a.emit ? a.pair_count : nullptr);
    if (t.n_multi > 0) {
        if (waves == 16)
            level_tiles_kick_kernel<16><<<t.n_multi, LT_TILE * 16, 0, stream>>>(t, a);
        else if (waves == 4)
            level_tiles_kick_kernel<4><<<t.n_multi, LT_TILE * 4, 0, stream>>>(t, a);
        else
            return hipErrorInvalidValue;
    }
    if (t.n_tiles > t.n_multi) level_tile_one_kernel<<<t.n_tiles - t.n_multi, LT_TILE, 0, stream>>>(t, a);
    return hipGetLastError();
}

} // namespace genga
