// Internal declarations shared by the HIP sources of the kick library (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "genga.h"

namespace genga {

// One unit of kick / energy work: up to 64 consecutive bodies (one per lane) of one system,
// all massive or all test bodies.
struct WorkItem {
    int32_t sys;
    int32_t i0;   // first body (global index)
    int32_t ni;   // number of bodies, 1..64
    int32_t nsrc; // sources: the first nsrc bodies of the system (all, or the massive ones
                  // for test-body targets)
};

enum DeviceFlag : int32_t {
    FLAG_CAPACITY = 1,
    FLAG_NONFINITE = 2,
    FLAG_NOCONVERGE = 4,   // Bulirsch-Stoer step
    FLAG_KEPLER = 8,       // Kepler solve
    FLAG_BADPAIR = 16,     // a caller's pair list held an invalid pair
};

// Maximum sizes of the close-encounter step (one workgroup builds the groups in LDS).
constexpr int CE_MAX_MEMBERS = 8192;
constexpr int CE_MAX_GROUPS = CE_MAX_MEMBERS / 2; // groups of at least two
constexpr int COLLIDE_CAP = 4096;          // colliding pairs per drift
constexpr int CE_MAX_GROUP = 64;
constexpr int BS_KMAX = 8;

// A run of at most CHUNK consecutive bodies of one system: the unit of the O(N) kernels
// (r_crit maxima, momentum sums, Sun drift; one body per thread), so block reductions never mix
// systems.
constexpr int CHUNK = 256;
struct Chunk {
    int32_t sys, b, e, pad;
};

struct Layout {
    int32_t n_sys = 0;
    int32_t n_total = 0;
    int32_t n_chunks = 0;
    int32_t *sys_off = nullptr;     // device [n_sys + 1]
    int32_t *sys_of = nullptr;      // device [n_total], system of each body
    double *mstar = nullptr;        // device [n_sys]
    Chunk *chunks = nullptr;        // device [n_chunks], systems in order
    int32_t *chunk_first = nullptr; // device [n_sys + 1]
    int32_t *n_massive = nullptr;   // device [n_sys]: bodies [off, off + n_massive) are massive
};

// A task of the kick's own plan: the item's targets and a run of its sources, with what the kick
// would otherwise look up one load after another.
struct KickTask {
    int32_t sys, i0, ni, j0, j1;
    int32_t c0, c1; // the system's chunks
    int32_t off;    // the system's first body
    uint32_t row;   // where its share starts: the bodies of the tasks before it
};

struct KickArgs {
    const WorkItem *items;
    int32_t n_items;
    const int32_t *sys_off;
    const double *x, *y, *z;
    double *vx, *vy, *vz;         // updated when update_v != 0
    const double *m, *rc;
    const float *m32;             // masses in FP32 (FP32 kick)
    const double *rc2_part;       // [n_chunks] max r_crit^2 per chunk
    const double *chunk_mass;     // [n_chunks] the mass a chunk's bodies share, NaN if they differ
    const int32_t *chunk_first;   // [n_sys + 1]
    double *ax, *ay, *az;         // a_i out (FP64), always written
    double tau;
    int32_t update_v;
    int32_t *pairs;               // [pair_cap][2]
    int32_t *pair_count;
    int32_t pair_cap;
    int32_t *flags;
    const KickTask *tasks;        // [n_tasks], items in order; null: every item's sources in `split`
                                  //   runs, task = item * split + run
    const int32_t *task_first;    // [n_items + 1] an item's tasks (with tasks)
    const uint32_t *item_row;     // [n_items] its first task's row (with tasks)
    int32_t n_tasks;
    int32_t split;
    int32_t direct;               // one task per item: it writes the bodies itself
    double *part;                 // shares of the targets (else): [3][ni] of a task at 3 row
    const int32_t *status;        // with collisions: bodies with status != 0 are in no pair
};

// A workgroup of launch_kick_close and of the launches around a drift alone, of CLOSE_WAVES waves: a
// run of items of one system, or several systems of up to CLOSE_SMALL items, each with the same number
// of waves, one an item.  (With a workgroup for every system 100000 systems of ten bodies took 2435 us a
// kick's close, now 120.)
constexpr int CLOSE_WAVES = 16;
constexpr int CLOSE_SMALL = 8;
// Each item of a run takes four waves, two or one, the most with which the blocks fit one per CU: 40000
// bodies (625 items of 20 tasks) take 13 us with four and 18 with one, 64 systems of 4096 (4096 items of
// one task) 21 with one and 39 with four.
inline int close_parts(int n_items, int n_cu)
{
    int p = 4;
    while (p > 1 && (int64_t)n_items * p > (int64_t)CLOSE_WAVES * n_cu) p /= 2;
    return p;
}
// (Summed by every workgroup of the system that takes it, the momentum of 4 million bodies made their
// genga_drift 676 us; summed once 217.  1.1 million, the first it is done for: 118 and 82.)
constexpr int LARGE_ROWS = 1024;
struct CloseBlock {
    int32_t sys, waves; // a system's waves: CLOSE_WAVES (a run of items), else systems [sys, sys + n)
    int32_t item, n;    // a run: items [item, item + n)
    int32_t f0, f1;     // a run: the system's items
    int32_t row;        // where its sums go in StepMomentum::kick: a run has one, else each system
    double mstar;       // a run: the system's
};

// Momentum sums that the launches of a step hand on to each other instead of passes of their own.
struct StepMomentum {
    const CloseBlock *blocks = nullptr;  // [n_blocks], systems in order
    const int32_t *row_first = nullptr;  // [n_sys + 1] a system's rows of kick
    const int32_t *item_first = nullptr; // [n_sys + 1] a system's items
    const double *mstar = nullptr;       // [n_sys]
    int32_t n_blocks = 0;
    bool small = false;                  // there are blocks of several systems
    const int32_t *large = nullptr;      // [n_large] systems of more than LARGE_ROWS rows of kick: whoever
    int32_t n_large = 0;                 //   takes their momentum reads one sum, formed by a launch of its own
    double *sys_kick = nullptr, *sys_kepler = nullptr; // [n_sys][3] these sums (of kick, kepler)
    int32_t parts = 1;                   // a run's waves per item
    double *kick = nullptr;    // [rows][3] sum m v after the kick
    double *kepler = nullptr;  // [n_items][3] sum m v after the drift, bodies outside groups
    double *group = nullptr;   // [CE_MAX_GROUPS][3] the same of the groups, which are in system order
    int32_t *group_sys = nullptr;
    int32_t *group_n = nullptr; // the groups the drift had (n_groups is the next kick's while it closes)
    double tau = 0.0;          // half a Sun drift: positions + tau P / Mstar
    int32_t *clear = nullptr;  // pair count, cleared by the drift once the groups are built
};

constexpr int KICK_MAX_SPLIT = 4;

// Error message for genga_last_error(); returns code.
int fail(int code, const char *fmt, ...);

// Source split reported for a layout (genga_get_kick_shape) before any tuning: the number of
// workgroups per item that wastes the least of the last round at one workgroup per CU.
inline int default_kick_split(int n_items, int n_cu)
{
    int best = 1;
    double best_eff = 0.0;
    for (int sp = 1; sp <= KICK_MAX_SPLIT; ++sp) {
        const double tasks = (double)n_items * sp;
        const double rounds = __builtin_ceil(tasks / n_cu);
        const double eff = tasks / (rounds * n_cu);
        if (eff > best_eff + 0.02) {
            best_eff = eff;
            best = sp;
        }
    }
    return best;
}

// The layout's own task plan.  Run length of a task's sources: the shortest of KICK_RUN_MIN,
// 2 KICK_RUN_MIN, .. that keeps the layout within KICK_TASKS_PER_CU tasks per CU (source visits
// = sum over the items of their sources).  Long runs spare prologues, short ones even out the
// CUs' shares: FP32 kick of 40000 bodies 620 / 576 / 562 us, of 64 discs of 2000-8000 bodies
// 611 / 614 / 567 us with 16 / 32 / 64 tasks per CU; a shortest run of 512 costs 2048 bodies
// 19.4 against 15.1 us, one of 128 gives 40 massive among 20000 test bodies 52 against 35 us.
constexpr int KICK_RUN_MIN = 256;
constexpr int KICK_TASKS_PER_CU = 64;
inline int run_len(int64_t source_visits, int n_cu, int len)
{
    n_cu = n_cu < 256 ? n_cu : 256;
    while (len < (1 << 30) && source_visits / len > (int64_t)KICK_TASKS_PER_CU * n_cu) len *= 2; // n <= 2^30
    return len;
}
// The kick's: runs of KICK_RUN_MIN only up to KICK_SHORT_PER_CU tasks per CU, where they fill it.
// Above, their prologues cost more than the even shares bring (FP32 / FP64 kick of 8000 bodies
// 42.5 / 56.4 us with 256, 38.2 / 53.5 with 512, of 16000 127 / 175 and 119 / 169, of 10 discs of
// 2000-8000 109 / 149 and 99 / 141; of 6600, 10 tasks per CU, 34.2 / 45.3 and 34.0 / 46.8).  Not
// where the items have few such runs each, whose lengths then differ too much (64 discs of
// 500-1500 bodies 46.7 / 63.1 and 49.2 / 66.5 us).
constexpr int KICK_SHORT_PER_CU = 14;
inline int kick_run_len(int64_t source_visits, int64_t n_items, int n_cu)
{
    const int64_t cus = n_cu < 256 ? n_cu : 256;
    const bool many = source_visits / KICK_RUN_MIN > KICK_SHORT_PER_CU * cus &&
                      source_visits >= 6 * KICK_RUN_MIN * n_items;
    return run_len(source_visits, n_cu, many ? 2 * KICK_RUN_MIN : KICK_RUN_MIN);
}
// The energy's, whose prologues are shorter (no r_crit, no candidates) and whose sources next to the
// targets are masked: genga_energy with 64 / 128 / 256 takes 12.2 / 13.1 / 16.9 us for 2048 bodies, 14.1 /
// 14.5 / 17.6 for 4000, 12.1 / 13.9 / 16.8 for 16 systems of 300, 30.5 / 29.8 / 31.2 for 9000.
constexpr int ENERGY_RUN_MIN = 64;
// Tasks of an item of nsrc sources at that run length, and the length of each task's run when
// nsrc sources are cut into `parts` (a multiple of four, so that whole quads stay whole).
inline int kick_runs(int nsrc, int len) { return nsrc < len + len / 2 ? 1 : (nsrc + len / 2) / len; }
__host__ __device__ inline int kick_run(int nsrc, int parts) { return ((nsrc + parts - 1) / parts + 3) / 4 * 4; }

// Waves per workgroup of the kick before any tuning: 4, of which 7 workgroups share a CU; 16 when
// the plan has one task per item and leaves CUs idle, where only shorter runs per wave help
// (257 bodies, FP64: 13.3 us with 8 waves, 16.0 with 4).
inline int default_kick_waves(int n_items, int n_tasks, int n_cu)
{
    return n_tasks == n_items && n_items <= n_cu ? 16 : 4;
}

// Address of the allocation-free entry point's scratch array on `device` (looked up once).
int noalloc_prepare(int device, unsigned char **ptr_out, int *n_cu_out);

// A task of the energy's pair sum: an item's targets and sources [j0, j1) of those after its first
// body; the item's first task also sums its kinetic parts.  The tasks of system s are
// [task_first[2 s], task_first[2 s + 2]), first tasks up to task_first[2 s + 1].
struct EnergyTask {
    int32_t sys, i0, ni, j0, j1, first;
};
// A workgroup of the energy's finishing launch: the systems [sys, sys + n) of up to ENERGY_SMALL tasks,
// a wave each, or (n = 0) the system sys.
constexpr int ENERGY_WAVES = 16, ENERGY_SMALL = 64;
struct EnergyRun {
    int32_t sys, n;
};
struct EnergyPlan {
    const EnergyTask *tasks = nullptr;   // [n_tasks], systems in order
    const int32_t *task_first = nullptr; // [2 n_sys + 1]
    int32_t n_tasks = 0;
    const EnergyRun *runs = nullptr;     // [n_runs]
    int32_t n_runs = 0;                  // 0: no small system, a workgroup for each
    double *partial = nullptr;           // [9][n_tasks]
};

// Kernel launchers (each enqueues on `stream`; return hipError_t of the launch).
// What the kick takes per chunk (r_crit^2 maxima, common masses), the masses in FP32 (m32 may be
// null) and a cleared pair count.
hipError_t launch_prep(const Layout &L, const double *m, const double *rc, float *m32, double *rc2_part,
                       double *chunk_mass, int32_t *pair_count, hipStream_t stream);
// kahan: the FP32 kick's blocks are summed with Kahan compensation in FP32 (else in FP64)
hipError_t launch_kick(const KickArgs &a, int fp32, int kahan, int waves, hipStream_t stream);
// Arrays of the one-workgroup group builder.
struct GroupBuild {
    const int32_t *pairs, *pair_count;
    int32_t pair_cap;
    int32_t *lab, *mark, *members, *group_start, *n_groups, *member_slot, *wg_list, *flags;
};
// The kick without its finishing launch, for launch_kick_close.
hipError_t launch_kick_shares(const KickArgs &a, int fp32, int kahan, int waves, hipStream_t stream);
// Finishes a kick inside a step: the tasks' shares summed, v += tau a; with pm.tau != 0 first the
// second half of the preceding drift's Sun drift (from pm.kepler and pm.group); then the sums of
// m v into pm.kick; and, from a workgroup of its own, with groups != null the encounter groups
// of the kick's pairs.
hipError_t launch_kick_close(const KickArgs &a, double *x, double *y, double *z, const StepMomentum &pm,
                             const GroupBuild *groups, hipStream_t stream);
// The encounter pairs of the state only (no forces, nothing written but a.pairs / a.pair_count).
hipError_t launch_pair_list(const KickArgs &a, hipStream_t stream);
hipError_t launch_rcrit(const Layout &L, const double *x, const double *y, const double *z,
                        const double *vx, const double *vy, const double *vz, const double *m,
                        double n1, double n2, double dt, double *rc, hipStream_t stream);
hipError_t launch_sun_drift(const Layout &L, double *x, double *y, double *z, const double *vx,
                            const double *vy, const double *vz, const double *m, double tau,
                            double *mom_part, hipStream_t stream);

// A caller's pair list src[min(*src_count, cap)][2] checked (0 <= i < j < n_total, one system)
// and copied to dst; *dst_count = *src_count, or 0 with FLAG_BADPAIR when a pair is invalid
// (bad: a device word, zero on entry and left zero).
struct PairImport {
    const int32_t *sys_of = nullptr;
    int32_t n_total = 0;
    const int32_t *src = nullptr, *src_count = nullptr;
    int32_t *dst = nullptr, *dst_count = nullptr;
    int32_t cap = 0;
    int32_t *bad = nullptr, *flags = nullptr;
};
hipError_t launch_import_pairs(const PairImport &p, hipStream_t stream);
// import (may be null): the end of an import that launch_drift_open began.
hipError_t launch_ce_groups(const GroupBuild &g, hipStream_t stream, const PairImport *import = nullptr);
// A drift outside a step: what comes before launch_ce_groups and launch_drift (the momentum sums
// for its first shift, the pairs of an import), and the second half of the Sun drift after it.
hipError_t launch_drift_open(const WorkItem *items, const double *vx, const double *vy, const double *vz,
                             const double *m, const StepMomentum &pm, const PairImport *import, hipStream_t stream);
// launch_sun_shift: positions + tau P / Mstar, P from the sums a step's kick left.  launch_drifted:
// the sums a step's drift leaves, when the drift ran in parts; pm.clear zeroed.
hipError_t launch_sun_shift(const WorkItem *items, int n_items, const double *mstar, double *x, double *y, double *z,
                            const StepMomentum &pm, hipStream_t stream);
hipError_t launch_drifted(const WorkItem *items, int n_items, const double *vx, const double *vy, const double *vz,
                          const double *m, const StepMomentum &pm, hipStream_t stream);
hipError_t launch_drift_close(const WorkItem *items, double *x, double *y, double *z, const StepMomentum &pm,
                              hipStream_t stream);
// Kepler drift of the bodies outside encounter groups and Bulirsch-Stoer of each group of up
// to CE_MAX_GROUP members (groups of 9 and more in a launch of their own, listed in wg_list:
// [0] their number, then the groups; room for bs_blocks + 1); clears member_slot for the next
// step.  Larger groups
// are flagged (GENGA_ERR_CAPACITY) and Kepler-drifted, or, with big_groups != 0, left alone
// for the grid-wide path below.
// A second stream for the launch of the groups of 9..64 members, forked from and joined back
// into the drift's stream by the two events (default priority; used only while the drift's
// stream is not being captured into a graph, where the two launches stay in sequence).
struct DriftSide {
    hipStream_t stream = nullptr;
    hipEvent_t fork = nullptr, join = nullptr;
};
// pm (may be null): the launch itself applies the first half of the Sun drift (pm->kick, pm->tau)
// and leaves the sums of m v after the drift; wg_listed: wg_list is already there.
hipError_t launch_drift(const Layout &L, const WorkItem *items, int n_items, double *x, double *y, double *z,
                        double *vx, double *vy, double *vz, const double *m, const double *rc, double dt,
                        const int32_t *members, const int32_t *group_start, const int32_t *n_groups,
                        int32_t *member_slot, int32_t *flags, int big_groups, int bs_blocks, int32_t *wg_list,
                        hipStream_t stream, const double *rc_lv = nullptr, int nlev = 1, bool kepler = true,
                        const DriftSide *side = nullptr, const StepMomentum *pm = nullptr, bool wg_listed = false);
// Grid-wide union-find of the encounter pairs (large-group mode, levels; lab all -1 on entry).
hipError_t launch_uf_union(const int32_t *pairs, const int32_t *pair_count, int32_t pair_cap, int32_t *lab,
                           hipStream_t stream);

// Grid-wide Bulirsch-Stoer for the groups of more than CE_MAX_GROUP members.  Members of the G
// large groups are numbered f = 0..M-1, group g holding [off[g], off[g+1]) (in an order the
// host chooses: body[f]); state arrays are SoA with stride M.  Capacities (cap_*) follow the
// layout: every body in one group at most; a group spans at most BIG_TILES_PER_GROUP tiles.
struct BigBs {
    int32_t G = 0, M = 0, n_tiles = 0; // host copies of dims[0..2]
    int32_t cap_M = 0, cap_G = 0, cap_T = 0; // allocated members, groups, tiles
    int32_t *dims = nullptr;       // device [4]: G, M, n_tiles (read by the attempt kernels)
    double *dtp = nullptr;         // device [1]: dt of the step
    int32_t *k0 = nullptr;         // [G] first entry of the group in members[]
    int32_t *off = nullptr;        // [G + 1]
    int4 *tiles = nullptr;         // [n_tiles] (group, first member, count, 0): 64 targets
    int32_t *tfirst = nullptr;     // [G + 1] first tile of each group
    double *bb = nullptr;          // [3][cap_T][8] tile boxes of Y, B1, B2
    int32_t *body = nullptr, *grp = nullptr, *test = nullptr; // [M]
    double *rc = nullptr, *mass = nullptr, *i09 = nullptr;    // [M]; i09 = 1 / (0.9 r_crit)
    double *Y = nullptr;           // [3][6][cap_M]: the state, then two sub-step buffers (stride M)
    double *tcol = nullptr;        // [BS_KMAX][6][M]: T(k, 0)
    double *mstar = nullptr, *t = nullptr, *H = nullptr, *rcmax2 = nullptr; // [G]
    int32_t *last = nullptr, *attempts = nullptr, *acc = nullptr, *done = nullptr; // [G]
    unsigned long long *sr = nullptr, *sv = nullptr; // [G] bit patterns of max |r|, max |v|
    unsigned long long *err = nullptr;               // [G][BS_KMAX] bit patterns of the estimates
    // hierarchical levels: with nlev > 1 the pair weight is prod_{k<nlev} (1 - K_k), level 0
    // from rc, level k >= 1 from rcl[(k - 1) * cap_M + f]; the candidate radius is the deepest
    // level's.  Fixed when the attempt graph is captured.
    int32_t nlev = 1;
    double *rcl = nullptr;         // [LEVELS_MAX - 1][cap_M]
    double *i9l = nullptr;         // [LEVELS_MAX - 1][cap_M] 1 / (0.9 rcl)
    // neighbour lists (the list path), built at the start of every attempt (bigbs.hip)
    int32_t *ltot = nullptr;       // [cap_M] the list's length
    uint16_t *ll = nullptr;        // [cap_M][BIG_LIST_CAP] the list, as slot positions
                                   //   (slot * 64 + position in the slot's source tile)
    int2 *slot = nullptr;          // [cap_T][BIG_LIST_SLOTS] per target tile: the source tiles holding
                                   //   an entry of its members' lists, in tile order, as (first
                                   //   member, members)
    int32_t *nslot = nullptr;      // [cap_T] their number
    double4 *pred = nullptr;       // [cap_M] the star's pull A at the attempt's start and the bound S
    double *skin = nullptr;        // [cap_M] skin factor of each body's bound (indexed by body): 2 at the
                                   //   step's start, times 4 after each crossing
    int32_t *crossed = nullptr;    // [cap_M] the member crossed its bound in the last attempt
    double *amut = nullptr;        // [cap_M] |pair acceleration| at the last attempt's start (column 0's
                                   //   first sub-step, on either path)
    int32_t *stale = nullptr;      // [G] a sub-step crossed a bound: the group's attempt is void
    int32_t *keep = nullptr;       // [G] the group's last attempt was rejected (not void): same start, a
                                   //   shorter step, so its lists and bounds still hold
    double *sbb = nullptr;         // [cap_T][BIG_BOX] per tile: the lowest position, velocity and A by
                                   //   component, the highest, the largest S
    // the list path's state buffers, so that the extrapolation columns advance side by side:
    // buffer 0 holds Y's positions, buffers 1 + 4k .. 4 + 4k column k's, two of one round and two of
    // the next
    double4 *P = nullptr;          // [1 + 4 BS_KMAX][cap_M] (x, y, z, mass), in a pair's second buffer (.., 1 / (0.9 r_crit))
    double *V = nullptr;           // [2 BS_KMAX][3][cap_M] the columns' velocities
    int32_t *status = nullptr;     // pinned host words that big_control_kernel writes: groups not yet at dt,
                                   //   lists overflowed, attempts the slowest group needs at least
    int32_t *ovf = nullptr;        // device word: a list exceeded BIG_LIST_CAP (the host falls back to tiles)
};
constexpr int BIG_TILES_PER_GROUP = 1024; // a workgroup of 1024 threads tests one source tile each
constexpr int BIG_BOX = 20;
constexpr int BIG_LIST_CAP = 1024;        // sources per member on the list path
constexpr int BIG_LIST_LANES = 8;         // lanes that share one member's list in a sub-step
constexpr int BIG_AHEAD = 16;             // attempts enqueued without looking at most
constexpr int BIG_LIST_SLOTS = 16;        // source tiles a target tile's sub-step stages in LDS
constexpr int LEVELS_MAX = 4;             // symplectic levels of the hierarchical step

// rc_lv: with b.nlev > 1, the critical radii of levels 1..nlev-1 ([nlev - 1][n_total]).
hipError_t launch_big_setup(const Layout &L, const BigBs &b, const int32_t *members, const double *x,
                            const double *y, const double *z, const double *vx, const double *vy,
                            const double *vz, const double *m, const double *rc, const double *rc_lv,
                            double dt, hipStream_t stream);
// One attempt of every active group: a fixed sequence of launches that takes its sizes and dt
// from device memory, so it can be captured once and replayed.
// tile_grid: workgroups of the per-tile launches (they visit the tiles grid-stride); waves: 8
// or 16 per workgroup (the sources of a target tile split over them).
hipError_t launch_big_attempt(const BigBs &b, double tol, int32_t *flags, int tile_grid, int waves,
                              hipStream_t stream);
// The same attempt on the list path: lists built at its start, then one launch per pass, in which
// the columns that still have that sub-step sum every member's list (BIG_LIST_LANES lanes per
// member) side by side.
hipError_t launch_big_attempt_list(const BigBs &b, double tol, int32_t *flags, int tile_grid, hipStream_t stream);
hipError_t launch_big_finish(const BigBs &b, double *x, double *y, double *z, double *vx, double *vy,
                             double *vz, hipStream_t stream);
// Members of the parent groups of a hierarchical level, laid out as the grid-wide
// Bulirsch-Stoer lays out its groups: group g holds members [off[g], off[g+1]) (body[f], in an
// order the host chooses), cut into tiles of 64 (group, first member, count, 0).
struct LevelTiles {
    int32_t G = 0, M = 0, n_tiles = 0, cap_M = 0; // sizes (host and kernel arguments)
    int32_t *off = nullptr, *tfirst = nullptr;   // [G + 1]
    int4 *tiles = nullptr;                       // [n_tiles]
    int32_t *body = nullptr, *test = nullptr;    // [M]
    double *X = nullptr, *Y = nullptr, *Z = nullptr, *mass = nullptr; // [M]
    double *rc = nullptr;                        // [LEVELS_MAX][cap_M]: radii of levels 0..
    double *i9 = nullptr;                        // [LEVELS_MAX][cap_M]: 1 / (0.9 rc)
    double *bb = nullptr;                        // [n_tiles][8] tile boxes of X, Y, Z
    double *cut2 = nullptr;                      // [G] largest level-(l-1) radius^2 of the group
    int32_t *tl = nullptr;                       // [n_tiles] tile indices: the n_multi tiles of groups of
    int32_t n_multi = 0;                         //   more than one tile, then one tile per smaller group
};

// Kick of level `level` (1 <= level < nlev) over the members of the parent groups:
// v += tau * sum over the member's group of m_j W_l K_l (r_j - r_i) / r^3 (FP64), and with
// emit the pairs of a group closer than the level's radius (body i < body j) into pairs.
struct LevelKickArgs {
    double *vx = nullptr, *vy = nullptr, *vz = nullptr;
    int32_t level = 1, emit = 0;
    double tau = 0.0;
    int32_t *pairs = nullptr, *pair_count = nullptr, *flags = nullptr;
    int32_t pair_cap = 0;
};
// Constants of the members (mass, TP2 flag, radii of levels 0..level) and each group's cut-off.
hipError_t launch_level_tiles_setup(const Layout &L, const LevelTiles &t, const double *m, const double *rc0,
                                    const double *rcl, int level, hipStream_t stream);
// Gather the members' positions and tile boxes, then kick (waves: 4 or 16 per workgroup of a
// multi-tile group's target tile).  An emitting kick starts its pair count from zero.
hipError_t launch_level_kick(const LevelTiles &t, const LevelKickArgs &a, const double *x, const double *y,
                             const double *z, int waves, hipStream_t stream);
// Kepler drift over dt of the bodies list[0..n-1] (with skip: those with skip[body] < 0; every
// listed skip[body] is then reset to -1).
hipError_t launch_kepler_list(const Layout &L, const int32_t *list, int32_t n, double *x, double *y,
                              double *z, double *vx, double *vy, double *vz, double dt, int32_t *flags,
                              hipStream_t stream, int32_t *skip = nullptr);

// Encounter groups of a level's pair list laid out on the device (groups.hip).  The host reads
// only the header, once per grouping.
struct GroupHeader {
    int32_t G, M;            // groups, members
    int32_t n_tiles, n_multi; // tiles of 64; of them in groups of several tiles
    int32_t max_nb;          // largest group
    int32_t pair_count;      // length of the pair list (may exceed its capacity)
    int32_t large_G, large_M, large_T; // groups of the large layout, their members and tiles
};
// Where the layout goes: body[M] the members group by group, each group in the parent order;
// off[G + 1]; with tiles != null also tfirst[G + 1], tiles[n_tiles] (group, first member, count,
// 0) in group order, and tl[n_tiles]: the tiles of groups of several tiles first, then the one
// tile of each smaller group.
// off2: a second copy of off; member_slot: the members' places in body, their labels then back to
// -1; large: with k0 != null the groups of at least `least` members laid out as the grid-wide
// Bulirsch-Stoer takes them, except for their members' order (k0[g] the group's first in body).
struct LargeOut {
    int32_t *k0 = nullptr, *off = nullptr, *tfirst = nullptr, *dims = nullptr;
    int4 *tiles = nullptr;
    int32_t least = 0;
};
struct GroupOut {
    int32_t *body = nullptr, *off = nullptr, *off2 = nullptr, *tfirst = nullptr, *tl = nullptr, *member_slot = nullptr;
    int4 *tiles = nullptr;
    LargeOut large;
};
struct GroupWork {
    uint64_t *keys = nullptr, *keys_sorted = nullptr; // [cap]
    int32_t *cnt = nullptr;                           // groups by block of 1024 members
    uint64_t *tsum = nullptr, *bsum = nullptr;        // tiles, large groups by block of 1024 groups
    GroupHeader *hdr = nullptr;                       // device
    void *temp = nullptr;                             // sort temporary storage
    size_t temp_bytes = 0;
    int cap = 0;                                      // largest parent layout
};
hipError_t group_work_alloc(GroupWork &w, int cap);
// The members of every group of a layout in ring / azimuth order about the star (the order the
// force tiles want: 64 consecutive members close together): per group, equal-width rings of
// distance to the star, as many as make a tile of 64 members about as wide as long, then the
// azimuth; a stable radix sort of the keys (group, quantised ring + azimuth / 4) with the body
// as value.  members[k0[gi] ..] are group gi's bodies, off[gi] its first slot in body_out.
struct OrderWork {
    uint64_t *keys = nullptr, *keys_sorted = nullptr; // [cap]
    int32_t *vals = nullptr;                          // [cap]
    uint64_t *bounds = nullptr;                       // [2 cap]: per group, smallest and largest distance
    void *temp = nullptr;
    size_t temp_bytes = 0;
    int cap = 0;
};
hipError_t order_work_alloc(OrderWork &w, int cap);
void order_work_free(OrderWork &w);
// Per group gi: its members members[k0[gi] ..] (members NULL: the bodies k0[gi], k0[gi] + 1, ..)
// in ring / azimuth order into body_out[off[gi] ..], groups one after the other.  M (the
// layout's size) and n_groups at most the work's capacity.
hipError_t launch_ring_order(const int32_t *members, const int32_t *k0, const int32_t *off, int n_groups, int M,
                             const double *x, const double *y, OrderWork &w, int32_t *body_out, hipStream_t stream);
void group_work_free(GroupWork &w);
// Union-find of pairs (lab all -1 on entry; afterwards every body of a pair holds its component's
// smallest body, the caller clears it); then the components' members in the order of the parent
// layout pbody[Mp] into `out`, and the header.
hipError_t launch_group_layout(const Layout &L, GroupWork &w, const int32_t *pairs, const int32_t *pair_count,
                               int32_t pair_cap, int32_t *lab, const int32_t *pbody, int Mp, const GroupOut &out,
                               hipStream_t stream);

// Collisions (perfect mergers) and removal by distance: caller-owned mass (the bodies' m),
// radius and status arrays; a list of the colliding pairs of the current drift.
struct CollideArgs {
    double *mass = nullptr, *radius = nullptr;
    int32_t *status = nullptr;   // 0 live, 1 merged into another body, 2 removed by distance
    int32_t *list = nullptr, *count = nullptr, *flags = nullptr;
    int32_t cap = 0;
    double r_min = 0.0, r_max = 0.0;
};
// Colliding encounter pairs at the start of a drift over dt (appended to c.list).
hipError_t launch_collide_check(const CollideArgs &c, const int32_t *pairs, const int32_t *pair_count,
                                int32_t pair_cap, const double *x, const double *y, const double *z,
                                const double *vx, const double *vy, const double *vz, double dt,
                                hipStream_t stream);
// After the drift: merge the listed pairs in order (the count is cleared), then removal.
hipError_t launch_collide_resolve(const CollideArgs &c, int n_total, double *x, double *y, double *z, double *vx,
                                  double *vy, double *vz, hipStream_t stream);

// dst[k] = src[idx[k]], k < n.
hipError_t launch_gather(const int32_t *idx, int n, const double *src, double *dst, hipStream_t stream);
hipError_t launch_gather(const int32_t *idx, int n, const int32_t *src, int32_t *dst, hipStream_t stream);

hipError_t launch_energy(const Layout &L, const EnergyPlan &e, const double *x, const double *y, const double *z,
                         const double *vx, const double *vy, const double *vz, const double *m, const double *ax,
                         const double *ay, const double *az, double vshift, double *out, hipStream_t stream);
// The list src in lexicographic order in dst (keys: room for src_cap).
hipError_t launch_sort_pairs(const int32_t *src, const int32_t *src_count, int32_t src_cap, int n_total,
                             int32_t *dst, int32_t dst_cap, int32_t *dst_count, uint64_t *keys,
                             int32_t *flags, hipStream_t stream);

} // namespace genga
