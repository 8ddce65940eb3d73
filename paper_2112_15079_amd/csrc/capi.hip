// C ABI of the library (declared in include/nbody.h): argument validation,
// workspace layout, the step loop of Eqs. (3)-(4) with HIP-graph replay, the
// reverse sweep of the discrete adjoint, the batched ensemble and the tile
// autotuner.  Every floating-point step runs in the kernels; this file only
// sequences launches.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <functional>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <tuple>
#include <vector>

#include "common.hpp"
#include "nbody.h"

using namespace nb;

namespace {

// ---------------------------------------------------------------------------
// errors

thread_local std::string g_err;

int fail(int code, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

#define NB_HIP(expr)                                                                   \
    do {                                                                               \
        hipError_t e_ = (expr);                                                        \
        if (e_ != hipSuccess)                                                          \
            return fail(NBODY_EHIP, "%s failed: %s", #expr, hipGetErrorString(e_));    \
    } while (0)

#define NB_TRY(expr)                       \
    do {                                   \
        int s_ = (expr);                   \
        if (s_ != NBODY_OK) return s_;     \
    } while (0)

constexpr int64_t kMaxBodies = (int64_t)1 << 30;

// ---------------------------------------------------------------------------
// tile table

std::mutex g_mu;
struct TunedTile {
    Tile tile;
    bool forced;   // nbody_set_tile (runs then take this tile at any size); the
                   // autotuner's tiles leave runs that stay on the chip there
};
std::map<std::tuple<int, int, int>, TunedTile> g_tiles;   // (kind, precision, size class)

constexpr int kBatchChunkMax = 16;
// Partial slots of an ensemble's workspace: the one-way passes use at most
// kBatchChunkMax per body, the each-pair-once pass one per 256-body range of
// the body's system, so it takes ensembles of systems up to 10,240 bodies.
constexpr int kBatchSlots = 40;

int size_class(int64_t n)
{
    // quarter-octave classes
    return (int)std::floor(4.0 * std::log2((double)std::max<int64_t>(n, 1)));
}

// Chunks allowed by the workspace: part buffers hold at most this many.
int chunk_cap(int64_t n)
{
    const int64_t c = ((int64_t)1 << 22) / std::max<int64_t>(n, 1);
    return (int)std::max<int64_t>(1, std::min<int64_t>(kMaxChunks, c));
}

// Systems up to this size default to the single-workgroup variant; up to
// kFusedDefault, to the fused force-and-step kernel with 8 waves per 64
// targets (variant 4).
constexpr int64_t kSmallDefault = 160;
constexpr int64_t kFusedDefault = 512;
// The autotuner tries the fused force-and-step kernel up to this size.
constexpr int64_t kFusedMax = 16384;
// From these sizes single systems default to the each-pair-once pass
// (variant 5, four waves sharing four target blocks per lane), up to
// kMutualMaxN bodies; below them the pass has too few workgroups to fill the
// chip.  The FP64 one-way pass takes two waves per 64 targets from 4,096
// bodies, where the pair-once step is already the faster (21.1 against
// 24.6 us per step at 4,300; 20.9 against 20.0 at 4,000 with one wave); the
// split form's one-way pass is cheaper than the FP64 one, so its crossover
// comes later (35.1 against 37.4 us per step at 8,000, 31.1 against 30.3
// at 7,000).
constexpr int64_t kMutualDefault = 4096;
constexpr int64_t kMutualSplitDefault = 8000;
// The adjoint's transpose-Jacobian pass with each pair once, from this size
// (shape (kVjpMutualTpl, 4); measured: 29.9 against 36.5 us for the one-way
// pass at 5,000 bodies, 29.7 against 28.4 at 4,300).
constexpr int64_t kVjpMutualDefault = 4500;
constexpr int kVjpMutualTpl = 4;

// The each-pair-once pass serves single systems (FP64 or split) of up to
// kMutualMaxN bodies: one partial per range of 256 bodies (plus a few for a
// split last round), 512 slots (1.6 GB of partials) at the largest.

bool mutual_fits(int kind, int prec, int64_t n)
{
    (void)prec;   // (the adjoint, kind 1, is FP64)
    return ((kind == 0 || kind == 1) && n <= kMutualMaxN) || kind == 2;   // (ensembles: per plan)
}

// Partial slots of a single system's workspace: the one-way passes' chunks,
// or one per range (plus the extra slots of a split last round) where the
// each-pair-once pass may run.
int part_slots(int64_t n)
{
    if (n > kMutualMaxN) return chunk_cap(n);
    return std::max({chunk_cap(n), mutual_slots(n, 4, 4), mutual_force_slots(NBODY_FP64, n, 4, 4)});
}

// Defaults from tile sweeps on MI355X (the autotuner refines them): one
// workgroup running whole steps for small systems (as many source slices as
// 1024 lanes allow, at most 16); then one kernel per step with 8 waves
// sharing each 64 targets; otherwise about 8192 wavefronts in flight;
// scalar-operand sources for FP64 below ~3e4 bodies (each pair once from
// 4,096, split from 8,000, to 131,072), LDS tiles with 4 targets per lane
// above; the split form's one-way passes prefer the LDS tiles at every size.
// The force pass alone (variants 0-2): partials for a separate epilogue.
Tile force_only_tile(int prec, int64_t n)
{
    Tile t{1, 1, 1, 0};
    if (prec == NBODY_FP64) {
        if (n < 32768) t = Tile{1, n < 4096 ? 1 : 2, 1, 1};
        else           t = Tile{4, 1, 1, 0};
    } else if (n >= 32768) {
        t = Tile{2, 8, 1, 0};
    }
    const int64_t tpb = targets_per_block(t);
    const int64_t tb = (n + tpb - 1) / tpb;
    int64_t c = std::max<int64_t>(1, 8192 / (tb * t.waves));
    c = std::min<int64_t>(c, std::max<int64_t>(1, n / (64 * t.waves)));
    t.chunks = (int)std::min<int64_t>(c, chunk_cap(n));
    return t;
}

Tile heuristic_tile(int kind, int prec, int64_t n)
{
    // the compensated split form runs in the each-pair-once pass only
    if (prec == NBODY_SPLIT_COMPENSATED) return Tile{4, 4, 1, 5};
    if (kind == 2) return Tile{2, 1, kBatchChunkMax, 0};   // ensemble: per-system chunks
    if (kind == 1 && n >= kVjpMutualDefault && mutual_fits(kind, prec, n))
        return Tile{kVjpMutualTpl, 4, 1, 5};   // transpose Jacobian, each pair once
    if (kind == 0 && n <= kSmallDefault)
        return Tile{1, 16, (int)std::max<int64_t>(1, std::min<int64_t>(16, 1024 / n)), 3};
    if (kind == 0 && n <= kFusedDefault) return Tile{1, 8, 1, 4};
    if (kind != 1 && n >= (prec == NBODY_FP64 ? kMutualDefault : kMutualSplitDefault) &&
        mutual_fits(kind, prec, n))
        return Tile{4, 4, 1, 5};
    if (kind == 0) return force_only_tile(prec, n);
    if (kind == 1) {
        // transpose-Jacobian pass: scalar-operand sources, two waves per 128
        // targets, sources split in up to 64 chunks of >= 16
        const int64_t c = std::min<int64_t>({64, std::max<int64_t>(1, n / 16),
                                             (int64_t)chunk_cap(n)});
        return Tile{1, 2, (int)c, 1};
    }
    return Tile{1, 1, 1, 0};
}

Tile pick_tile(int kind, int prec, int64_t n)
{
    {
        std::lock_guard<std::mutex> lk(g_mu);
        auto it = g_tiles.find(std::make_tuple(kind, prec, size_class(n)));
        if (it != g_tiles.end() && !(it->second.tile.variant == 3 && n > kSmallMax) &&
            !(it->second.tile.variant == 5 && !mutual_fits(kind, prec, n)) &&
            !(prec == NBODY_SPLIT_COMPENSATED && it->second.tile.variant != 5)) {
            Tile t = it->second.tile;
            t.chunks = std::min(t.chunks, chunk_cap(n));
            return t;
        }
    }
    return heuristic_tile(kind, prec, n);
}

// ---------------------------------------------------------------------------
// the workgroups that stay on the chip (kernels_group.hip)

// Runs of single systems of these sizes take the group kernel unless
// nbody_set_tile chose a tile for the size (us per step, FP64, 300-step runs:
// 1.55 against 1.43 with one workgroup alone at 64 bodies, 1.76 against 2.44 at
// 100; 16.0 against 20.8 each pair once at 4,095: above, 256 workgroups of 16
// targets would not hold the system, nor LDS its sources).  The autotuner's tiles
// do not change that: none is faster (us per step, 400-step runs, against the best
// of its tiles, FP64 and split: 1.72 and 1.63 against 1.83 and 2.12 at 80 bodies,
// 1.9 and 1.9 against 4.0 and 4.1 at 131, 3.5 and 3.7 against 10.1 and 10.7 at
// 1,000, 13.7 and 12.0 against 15.1 and 15.4 at 3,500, 15.8 and 13.7 against 17.9
// and 16.3 at 4,095).
constexpr int64_t kGroupMin = 80;
constexpr int64_t kGroupMax = 4095;

// The group kernel's shape for n bodies: few enough targets per workgroup that
// the chip's 256 CUs are used, one workgroup each (us per step at 1,000
// bodies: 3.4 with 250 workgroups of 4 targets, 4.0 with 125 of 8), with two
// waves per SIMD where a round's latency hides behind them (1,000 bodies: 3.4
// with 1,024 threads, 3.7 with 512; 500 bodies: 2.6 and 2.5).  Between 1,024 and
// 2,560 bodies the targets per workgroup grow in steps of one to two, by three or
// five lanes side by side (us per step, FP64 and split, against the next power
// of two or twelve: 3.9 and 4.0 against 4.4 and 4.1 at 1,100; 7.4 and 6.6 against
// 8.2 and 7.5 at 2,079; 8.8 and 7.9 against 9.3 and 8.3 at 2,500).  Above, their
// idle lanes cost more than the finer steps give (14 targets against 12: 12.1
// against 10.5 at 3,000; against 16: 13.8 and 13.8 at 3,500).
GroupShape group_shape(int64_t n)
{
    if (n <= 256) return {1, 8, 512};
    if (n <= 768) return {1, 4, 512};
    if (n <= 1024) return {1, 4, 1024};
    if (n <= 1280) return {1, 5, 1024};
    if (n <= 1536) return {2, 3, 512};
    if (n <= 2048) return {2, 4, 512};
    if (n <= 2304) return {3, 3, 512};
    if (n <= 2560) return {2, 5, 1024};
    if (n <= 3072) return {3, 4, 1024};
    return {4, 4, 512};
}

// Up to 256 bodies the at most 32 workgroups are placed on one XCD (one in eight
// of those launched: workgroups go to the XCDs in turn), whose L2 then carries
// the exchange: 1.8 against 2.1 us per step at 131 bodies.
int group_spread(int64_t n) { return n <= 256 ? 8 : 1; }

// Whether a run (or force evaluation) of a single system takes it.
bool group_route(int prec, int64_t n)
{
    if (prec == NBODY_SPLIT_COMPENSATED || n < kGroupMin || n > kGroupMax) return false;
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_tiles.find(std::make_tuple(0, prec, size_class(n)));
    return it == g_tiles.end() || !it->second.forced;
}

// Launch indices of one launch.
constexpr int64_t kGroupSegment = 1024;

// Launch indices 0 .. last of a run by the group kernel: A with everything but
// the indices, in `blocks` workgroups; n_max: the largest of nsys systems.
int group_launches(int prec, const GroupShape& g, GroupArgs A, int blocks, int64_t n_max, int nsys,
                   int64_t last, hipStream_t s)
{
    double* const traj = A.traj;
    for (int64_t a = 0; a <= last;) {
        // (never one index alone that drifts: it would write where others read)
        int64_t b = std::min(a + kGroupSegment - 1, last);
        if (last - b == 1) b = last;
        A.traj = traj ? traj + a * 3 * A.n : nullptr;
        A.i0 = a;
        A.i1 = b;
        NB_HIP(launch_group(prec == NBODY_SPLIT ? 1 : 0, g, A, blocks, n_max, 12 * A.n, nsys, s));
        // a launch that stores nothing but the trajectory hands its last
        // position on through the trajectory buffer
        A.pos_in = A.pos_out ? A.pos_out : A.traj ? A.traj + (b - a) * 3 * A.n : nullptr;
        a = b + 1;
    }
    return NBODY_OK;
}

// ... of a single system of n bodies, a run of `steps` steps with the state in
// pos, vel (with traj the positions after each drift are stored and pos is only
// read); or, with acc, the accelerations at pos (body p's at acc_perm[p] if
// given).  xbuf: 12 n doubles, 16-byte
// aligned; reg: its registration words (both unused when last = 0).
int group_run(int prec, const double* pos_in, double* pos_out, double* vel, const double* mass,
              int64_t n, const int64_t* nmaj, double G, double dt, int64_t last, int64_t steps,
              double* acc, double* traj, double* xbuf, uint32_t* reg, uint32_t* flags,
              hipStream_t s, const int32_t* acc_perm = nullptr)
{
    GroupArgs A{};
    A.pos_in = pos_in;
    A.pos_out = pos_out;
    A.vel = vel;
    A.mass = mass;
    A.xbuf = xbuf;
    A.reg = reg;
    A.nmaj = nmaj;
    A.acc = acc;
    A.acc_perm = acc_perm;
    A.traj = traj;
    A.flags = flags;
    A.n = n;
    A.stride = n;
    A.G = G;
    A.dt = dt;
    A.steps = steps;
    A.spread = group_spread(n);
    const GroupShape g = group_shape(n);
    const int64_t tw = (int64_t)g.tpl * g.lanes;
    return group_launches(prec, g, A, (int)((n + tw - 1) / tw), n, 1, last, s);
}

// The registration words of a workspace, behind the flags word: those of the
// caller's stream (0), the adjoint's second (1) and its reverse sweep (2).
uint32_t* group_reg(uint32_t* flags, int which = 0)
{
    return flags + 16 + kGroupRegWords * which;
}

// The shape of the reverse sweep for n bodies, and whether a CU has registers and
// LDS for a workgroup of it beside one of the run kernel, so that the sweep of a
// segment and the recompute of the next one run side by side (us per step of the
// reverse half over 20 segments, side by side, in turn, and by a product and its
// reduction per position with a recompute by launches: 2.5, 4.1 and 9.6 at 131
// bodies, 6.5, 7.9 and 12.9 at 1,000, 12.7, 15.6 and 16.2 at 2,048, 15.2, 18.8
// and 16.2 at 2,079).  That takes 512 threads, the registers of the shape table,
// and the LDS up to 2,251 bodies; up to 1,670 there is room for the positions
// too (1,600 bodies: 9.8 with them in LDS, 10.2 read ahead from the caches).
// Above, the two take turns, in shapes that have a CU to themselves (forward,
// recompute and sweep, in turn against all three by launches: over two segments
// 29.0 and 41.6 at 2,252, 39.1 and 51.5 at 3,072, 59.1 and 69.4 at 4,095; over 20
// segments, where launches overlap better, 30.6 and 37.2, 40.4 and 45.2, 60.6 and
// 64.7, at 3,073 48.6 and 47.3).
GroupVjpShape group_vjp_shape(int64_t n, bool* beside)
{
    constexpr size_t kLds = 160 * 1024 - 2048;   // (static LDS and granules)
    const size_t run = group_lds_bytes(n, group_shape(n));
    auto fits = [&](const GroupVjpShape& g) { return run + group_vjp_lds_bytes(n, g) <= kLds; };
    *beside = true;
    if (n <= 256) return {1, 8, 512, true};
    if (n <= 1024) return {1, 4, 512, true};
    if (n <= 1280) return {1, 5, 512, true};
    if (n <= 1536) return {2, 3, 512, true};
    if (n <= 2048) return {2, 4, 512, fits({2, 4, 512, true})};
    if (fits({2, 5, 512, false})) return {2, 5, 512, false};
    *beside = false;
    if (n <= 2560) return {5, 2, 512, false};
    if (n <= 3072) return {3, 4, 512, false};
    return {4, 4, 512, false};
}

// Whether the reverse sweep of segments of K steps takes the group kernel, where
// the runs do (`group`) and unless nbody_set_tile chose a tile for the product.
// (One position alone would be written where others still read.)
bool group_vjp_route(bool group, int64_t n, int64_t K)
{
    if (K < 2 || !group) return false;
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_tiles.find(std::make_tuple(1, (int)NBODY_FP64, size_class(n)));
    return it == g_tiles.end() || !it->second.forced;
}

// Positions of one segment's reverse sweep, in launches of two to about
// kGroupSegment of them.
int group_sweep(GroupVjpArgs A, hipStream_t s)
{
    bool beside;
    const GroupVjpShape g = group_vjp_shape(A.n, &beside);
    A.spread = group_spread(A.n);
    int64_t left = A.count;
    for (int64_t pieces = (left + kGroupSegment - 1) / kGroupSegment; pieces > 0; --pieces) {
        A.count = (left + pieces - 1) / pieces;
        NB_HIP(launch_group_vjp(g, A, s));
        A.k1 -= A.count - (A.last ? 1 : 0);
        A.last = nullptr;
        left -= A.count;
    }
    return NBODY_OK;
}

// ---------------------------------------------------------------------------
// workspace layout

struct Layout {
    size_t flags = 0, part = 0, alt = 0, gm = 0, perm = 0, nmaj = 0, offs = 0, pos_c = 0, vel_c = 0,
           mass_c = 0, alt_c = 0, units = 0, bchunks = 0, ck = 0, seg = 0, lam_r = 0,
           lam_v = 0, g_m = 0, u = 0, vtmp = 0, rk_vs = 0, rk_sr = 0, rk_sv = 0, seg2 = 0,
           part2 = 0, vtmp2 = 0, total = 0;
};

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct Alloc {
    size_t off = 0;
    size_t take(size_t bytes)
    {
        const size_t o = off;
        off = align256(off + std::max<size_t>(bytes, 1));
        return o;
    }
};

Layout layout(int op, int64_t n, int32_t ns, int64_t steps, int64_t K, int prec)
{
    Layout L;
    Alloc a;
    const size_t d = sizeof(double);
    L.flags = a.take(256);
    const int cap = op == NBODY_OP_BATCHED     ? kBatchSlots
                  : op == NBODY_OP_ENERGY      ? chunk_cap(n)
                  : op == NBODY_OP_ACCEL_SHARD ? kMaxChunks
                                               : part_slots(n);
    const bool adj = op == NBODY_OP_ADJOINT || op == NBODY_OP_ADJOINT_SWEEP;
    const int planes = adj ? 4 : 3;
    L.part = a.take((size_t)cap * planes * n * d);
    L.alt = a.take(3 * n * d);
    L.gm = a.take(n * d);
    if (prec != NBODY_FP64 && !adj && op != NBODY_OP_ENERGY) {
        L.perm = a.take(n * sizeof(int32_t));
        L.nmaj = a.take((size_t)ns * sizeof(int64_t));
        L.offs = a.take((size_t)(ns + 1) * sizeof(int64_t));
        L.pos_c = a.take(3 * n * d);
        L.vel_c = a.take(3 * n * d);
        L.mass_c = a.take(n * d);
        L.alt_c = a.take(3 * n * d);
    }
    if (op == NBODY_OP_RK4) {   // stage velocity and slope sums (alt is the stage position)
        L.rk_vs = a.take(3 * n * d);
        L.rk_sr = a.take(3 * n * d);
        L.rk_sv = a.take(3 * n * d);
    }
    if (op == NBODY_OP_ACCEL_SHARD)   // target blocks of >= 64 bodies times <= kMaxChunks chunks
        L.units = a.take((size_t)(n / 64 + 2) * kMaxChunks * sizeof(BatchUnit));
    if (op == NBODY_OP_BATCHED) {
        if (!L.offs) L.offs = a.take((size_t)(ns + 1) * sizeof(int64_t));
        // units: per system ceil(n_k/64) target blocks (the smallest tile) times
        // at most kBatchChunkMax chunks.
        const int64_t max_units = (n / 64 + ns) * kBatchChunkMax;   // >= any tile's unit count
        L.units = a.take((size_t)max_units * sizeof(BatchUnit));
        L.bchunks = a.take(n);
    }
    if (adj) {
        const int64_t nck = (steps + K - 1) / K;
        // the checkpoints: in the workspace for NBODY_OP_ADJOINT, in the
        // caller's buffer for the split forward and reverse calls
        if (op == NBODY_OP_ADJOINT) L.ck = a.take((size_t)(nck + 1) * 6 * n * d);
        L.seg = a.take((size_t)std::min(K, std::max<int64_t>(steps, 1)) * 3 * n * d);
        // the next segment's positions, recomputed on a second stream while the
        // reverse sweep works on this one, with that stream's partials and velocity
        L.seg2 = a.take((size_t)std::min(K, std::max<int64_t>(steps, 1)) * 3 * n * d);
        L.part2 = a.take((size_t)cap * 3 * n * d);
        L.vtmp2 = a.take(3 * n * d);
        L.lam_r = a.take(3 * n * d);
        L.lam_v = a.take(3 * n * d);
        L.g_m = a.take(n * d);
        L.u = a.take(3 * n * d);
        L.vtmp = a.take(3 * n * d);
    }
    L.total = a.off;
    return L;
}

template <typename T>
T* at(void* ws, size_t off)
{
    return reinterpret_cast<T*>(static_cast<char*>(ws) + off);
}

// ---------------------------------------------------------------------------
// validation

int check_common(const void* pos, const void* mass, int64_t n, double G)
{
    if (!pos || !mass) return fail(NBODY_EINVAL, "null position or mass pointer");
    if (n < 1) return fail(NBODY_EINVAL, "n must be >= 1 (got %lld)", (long long)n);
    if (n > kMaxBodies) return fail(NBODY_EUNSUPPORTED, "n = %lld exceeds 2^30", (long long)n);
    if (!std::isfinite(G)) return fail(NBODY_EINVAL, "G is not finite");
    return NBODY_OK;
}

int check_prec(int32_t prec, double small_mass)
{
    if (prec != NBODY_FP64 && prec != NBODY_SPLIT && prec != NBODY_SPLIT_COMPENSATED)
        return fail(NBODY_EINVAL, "unknown precision %d", prec);
    if (prec != NBODY_FP64 && !(small_mass >= 0.0 && std::isfinite(small_mass)))
        return fail(NBODY_EINVAL, "split threshold must be finite and >= 0");
    return NBODY_OK;
}

// The compensated split form runs in the each-pair-once pass, which takes
// single systems of up to kMutualMaxN bodies.
int check_comp_size(int32_t prec, int64_t n)
{
    if (prec == NBODY_SPLIT_COMPENSATED && n > kMutualMaxN)
        return fail(NBODY_EUNSUPPORTED,
                    "the compensated split form takes at most %lld bodies (got %lld)",
                    (long long)kMutualMaxN, (long long)n);
    return NBODY_OK;
}

int check_ws(const void* ws, size_t have, size_t need)
{
    if (!ws) return fail(NBODY_EWORKSPACE, "workspace is NULL (need %zu bytes)", need);
    if (have < need) return fail(NBODY_EWORKSPACE, "workspace has %zu bytes, need %zu", have, need);
    if (reinterpret_cast<uintptr_t>(ws) % 256 != 0)
        return fail(NBODY_EINVAL, "workspace must be 256-byte aligned");
    return NBODY_OK;
}

// ---------------------------------------------------------------------------
// graph capture: a private capture stream per device (default priority).

std::map<int, hipStream_t> g_capture_streams;

int capture_stream(hipStream_t* out)
{
    int dev = 0;
    NB_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_capture_streams.find(dev);
    if (it == g_capture_streams.end()) {
        hipStream_t s = nullptr;
        NB_HIP(hipStreamCreateWithFlags(&s, hipStreamNonBlocking));
        it = g_capture_streams.emplace(dev, s).first;
    }
    *out = it->second;
    return NBODY_OK;
}

// A second stream per device (default priority, non-blocking) and the events
// that order it against the caller's stream in the adjoint's pipelined reverse
// sweep; g_adjoint_mu serialises the enqueue of adjoint calls, so the cached
// events are recorded and waited on by one call at a time.
struct SideStream {
    hipStream_t stream = nullptr;
    hipEvent_t fwd = nullptr, ready[2] = {nullptr, nullptr}, freed[2] = {nullptr, nullptr};
    std::mutex adjoint_mu;
};
std::map<int, std::unique_ptr<SideStream>> g_side;

int side_stream(SideStream** out)
{
    int dev = 0;
    NB_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_side.find(dev);
    if (it == g_side.end()) {
        auto ss = std::make_unique<SideStream>();
        NB_HIP(hipStreamCreateWithFlags(&ss->stream, hipStreamNonBlocking));
        for (hipEvent_t* e : {&ss->fwd, &ss->ready[0], &ss->ready[1], &ss->freed[0], &ss->freed[1]})
            NB_HIP(hipEventCreateWithFlags(e, hipEventDisableTiming));
        it = g_side.emplace(dev, std::move(ss)).first;
    }
    *out = it->second.get();
    return NBODY_OK;
}

struct GraphKey {
    std::vector<uint64_t> v;
    bool operator<(const GraphKey& o) const { return v < o.v; }
};

struct GraphEntry {
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    int device = 0;
    uint64_t used = 0;   // last use (for eviction)
};

// Captured graphs, keyed by everything they bake in (device, sizes, scalars,
// buffer addresses).  At most kMaxGraphs are kept; the least recently used
// one is dropped first.  g_graph_mu serialises capture, lookup and launch.
constexpr size_t kMaxGraphs = 64;
std::mutex g_graph_mu;
std::map<GraphKey, GraphEntry> g_graphs;
uint64_t g_graph_tick = 0;

// A graph may still be running when it is dropped: wait for its device first.
void destroy_graph(const GraphEntry& e)
{
    int cur = 0;
    if (hipGetDevice(&cur) == hipSuccess && hipSetDevice(e.device) == hipSuccess) {
        (void)hipDeviceSynchronize();
        (void)hipSetDevice(cur);
    }
    if (e.exec) (void)hipGraphExecDestroy(e.exec);
    if (e.graph) (void)hipGraphDestroy(e.graph);
}

void drop_graphs()
{
    std::lock_guard<std::mutex> lk(g_graph_mu);
    for (auto& kv : g_graphs) destroy_graph(kv.second);
    g_graphs.clear();
}

void drop_batch_plans();

uint64_t bits(double x)
{
    uint64_t u;
    std::memcpy(&u, &x, sizeof u);
    return u;
}

uint64_t ptrbits(const void* p) { return (uint64_t)reinterpret_cast<uintptr_t>(p); }

// The cached graph for key_in on the current device, captured from
// `body(stream)` first if there is none.  body must only enqueue kernels.
// Call with g_graph_mu held.
template <typename F>
int find_or_capture(const GraphKey& key_in, F&& body, GraphEntry** out)
{
    int dev = 0;
    NB_HIP(hipGetDevice(&dev));
    GraphKey key = key_in;
    key.v.push_back((uint64_t)dev);
    auto it = g_graphs.find(key);
    if (it == g_graphs.end()) {
        hipStream_t cs = nullptr;
        NB_TRY(capture_stream(&cs));
        NB_HIP(hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal));
        const int st = body(cs);
        hipGraph_t g = nullptr;
        const hipError_t ee = hipStreamEndCapture(cs, &g);
        if (st != NBODY_OK) {
            if (g) (void)hipGraphDestroy(g);
            return st;
        }
        if (ee != hipSuccess) return fail(NBODY_EHIP, "hipStreamEndCapture: %s", hipGetErrorString(ee));
        hipGraphExec_t ge = nullptr;
        const hipError_t ie = hipGraphInstantiate(&ge, g, nullptr, nullptr, 0);
        if (ie != hipSuccess) {
            (void)hipGraphDestroy(g);
            return fail(NBODY_EHIP, "hipGraphInstantiate: %s", hipGetErrorString(ie));
        }
        while (g_graphs.size() >= kMaxGraphs) {
            auto victim = g_graphs.begin();
            for (auto jt = g_graphs.begin(); jt != g_graphs.end(); ++jt)
                if (jt->second.used < victim->second.used) victim = jt;
            destroy_graph(victim->second);
            g_graphs.erase(victim);
        }
        GraphEntry e;
        e.graph = g;
        e.exec = ge;
        e.device = dev;
        it = g_graphs.emplace(key, e).first;
    }
    it->second.used = ++g_graph_tick;
    *out = &it->second;
    return NBODY_OK;
}

// Captures `body` once per key (plus the current device) and launches the
// instantiated graph on `stream`.
template <typename F>
int run_graph(const GraphKey& key, hipStream_t stream, F&& body)
{
    std::lock_guard<std::mutex> lk(g_graph_mu);
    GraphEntry* e = nullptr;
    NB_TRY(find_or_capture(key, body, &e));
    NB_HIP(hipGraphLaunch(e->exec, stream));
    return NBODY_OK;
}

// ---------------------------------------------------------------------------
// the step loop

// One system (or the concatenated batch) of the kick-drift-kick step loop.
struct StepPlan {
    int prec = 0;
    Tile tile{};
    int chunks = 1;                 // chunks for the epilogue (single system)
    int64_t n = 0;
    double G = 0, dt = 0;
    const double* mass = nullptr;   // in the working order
    const double* gm = nullptr;     // G * mass, same order
    double* vel = nullptr;          // working velocity
    double* buf[2] = {nullptr, nullptr};   // position ping-pong
    double* part = nullptr;
    uint32_t* flags = nullptr;
    const int64_t* nmaj = nullptr;
    // batched
    const BatchUnit* units = nullptr;
    int64_t num_units = 0;
    int grid = 0;
    const int8_t* bchunks = nullptr;
};

int force(const StepPlan& P, const double* pos, hipStream_t s)
{
    if (P.units && P.tile.variant == 5)
        NB_HIP(launch_force_mutual_batched(P.prec, P.tile.tpl, P.tile.waves, pos, P.gm, P.n,
                                           P.units, P.num_units, P.nmaj, P.part, s));
    else if (P.units)
        NB_HIP(launch_force_batched(P.prec, P.tile, pos, P.mass, P.gm, P.n, P.G, P.units,
                                    P.num_units, P.nmaj, P.grid, P.part, s));
    else
        NB_HIP(launch_force(P.prec, P.tile, pos, P.mass, P.gm, P.n, P.nmaj, P.G, P.part, s));
    return NBODY_OK;
}

// The force pass at pin followed by the epilogue in `mode` (one fused kernel
// for a variant-4 tile).
int force_and_step(const StepPlan& P, const double* pin, double* pout, int mode, hipStream_t s)
{
    if (P.tile.variant == 4 && !P.units) {
        NB_HIP(launch_step_fused(P.prec, P.tile, pin, pout, P.vel, P.gm, P.n, P.nmaj, P.dt, mode,
                                 nullptr, P.flags, s));
        return NBODY_OK;
    }
    NB_TRY(force(P, pin, s));
    NB_HIP(launch_step(P.part, P.chunks, P.bchunks, P.n, P.vel, pin, pout, nullptr, P.dt, mode,
                       P.flags, s));
    return NBODY_OK;
}

// Launch i of a run of `steps` steps (i = 0 .. steps): the force pass at r_i
// (in buf[i & 1]) followed by the epilogue.
int step_launch(const StepPlan& P, int64_t i, int64_t steps, hipStream_t s)
{
    int mode = 0;
    if (i > 0) mode |= kClose;
    if (i < steps) mode |= kOpen;
    return force_and_step(P, P.buf[i & 1], P.buf[(i + 1) & 1], mode, s);
}

constexpr int64_t kGraphSteps = 64;   // middle launches per captured graph

GraphKey steps_key(const StepPlan& P)
{
    GraphKey key;
    key.v = {1, (uint64_t)P.prec, (uint64_t)P.tile.tpl, (uint64_t)P.tile.waves,
             (uint64_t)P.tile.chunks, (uint64_t)P.tile.variant, (uint64_t)P.chunks, (uint64_t)P.n,
             bits(P.G), bits(P.dt), ptrbits(P.mass), ptrbits(P.gm), ptrbits(P.vel),
             ptrbits(P.buf[0]), ptrbits(P.buf[1]), ptrbits(P.part), ptrbits(P.flags),
             ptrbits(P.nmaj), ptrbits(P.units), (uint64_t)P.num_units, (uint64_t)P.grid,
             ptrbits(P.bchunks)};
    return key;
}

// Launches 0..steps; r_0 must be in buf[0].  The final r_steps lands in
// buf[steps & 1].  With use_graph the middle launches (both half kicks and
// the drift) run as replays of one captured graph of kGraphSteps launches,
// each replay starting on an odd launch index (r_i in buf[1]); the first
// launch, the last and the middle ones left over are enqueued directly.
// (Once the GPU's clock has settled, direct launches cost no more GPU time
// than graph replays for a short run; graphs save host time on long ones.)
int run_steps(const StepPlan& P, int64_t steps, hipStream_t stream, bool use_graph)
{
    if (steps <= 0) return NBODY_OK;
    NB_TRY(step_launch(P, 0, steps, stream));
    int64_t i = 1;
    if (use_graph && steps > kGraphSteps) {
        const GraphKey key = steps_key(P);
        for (; i + kGraphSteps <= steps; i += kGraphSteps)   // launches i .. i + 63 < steps
            NB_TRY(run_graph(key, stream, [&](hipStream_t cs) {
                for (int64_t k = 0; k < kGraphSteps; ++k) {
                    const int b = (int)((1 + k) & 1);
                    NB_TRY(force_and_step(P, P.buf[b], P.buf[b ^ 1], kClose | kOpen, cs));
                }
                return (int)NBODY_OK;
            }));
    }
    for (; i <= steps; ++i) NB_TRY(step_launch(P, i, steps, stream));
    return NBODY_OK;
}

// The split form's working copies of one system, in class order.
struct ClassOrdered {
    const int32_t* perm;
    const int64_t* nmaj;
    double *pos, *vel, *mass, *gm;
};

int split_prepare(void* ws, const Layout& L, const double* pos, const double* vel,
                  const double* mass, int64_t n, double G, double small_mass, hipStream_t s,
                  ClassOrdered* c)
{
    int32_t* perm = at<int32_t>(ws, L.perm);
    int64_t* nmaj = at<int64_t>(ws, L.nmaj);
    *c = {perm, nmaj, at<double>(ws, L.pos_c), at<double>(ws, L.vel_c), at<double>(ws, L.mass_c),
          at<double>(ws, L.gm)};
    NB_HIP(launch_class_order(pos, vel, mass, nullptr, 1, n, n, small_mass, G, perm, nmaj, c->pos,
                              c->vel, c->mass, c->gm, s));
    return NBODY_OK;
}

// Whether two arrays of doubles share memory.
bool overlap(const double* a, int64_t na, const double* b, int64_t nb)
{
    return std::less<const double*>()(a, b + nb) && std::less<const double*>()(b, a + na);
}

// Fourth-order Runge-Kutta: `steps` steps of four force passes and stage
// updates; the position buffer r is updated in place.  Groups of kRk4Graph
// steps are replayed from a captured graph.
constexpr int64_t kRk4Graph = 16;

int rk4_steps(const StepPlan& P, double* r, double* v, double* rs, double* vs, double* sr,
              double* sv, int64_t steps, hipStream_t stream)
{
    auto one = [&](hipStream_t cs) -> int {
        for (int stage = 1; stage <= 4; ++stage) {
            NB_TRY(force(P, stage == 1 ? r : rs, cs));
            NB_HIP(launch_rk4_stage(P.part, P.chunks, P.n, stage, P.dt, r, v, rs, vs, sr, sv,
                                    P.flags, cs));
        }
        return NBODY_OK;
    };
    int64_t i = 0;
    if (steps >= 2 * kRk4Graph) {
        GraphKey key;
        key.v = {5, (uint64_t)P.prec, (uint64_t)P.tile.tpl, (uint64_t)P.tile.waves,
                 (uint64_t)P.tile.chunks, (uint64_t)P.tile.variant, (uint64_t)P.chunks,
                 (uint64_t)P.n, bits(P.G), bits(P.dt), ptrbits(P.mass), ptrbits(P.gm),
                 ptrbits(P.part), ptrbits(P.flags), ptrbits(P.nmaj), ptrbits(r), ptrbits(v),
                 ptrbits(rs), ptrbits(vs), ptrbits(sr), ptrbits(sv)};
        for (; i + kRk4Graph <= steps; i += kRk4Graph)
            NB_TRY(run_graph(key, stream, [&](hipStream_t cs) -> int {
                for (int64_t k = 0; k < kRk4Graph; ++k) NB_TRY(one(cs));
                return NBODY_OK;
            }));
    }
    for (; i < steps; ++i) NB_TRY(one(stream));
    return NBODY_OK;
}

}  // namespace

// ===========================================================================
// C ABI

extern "C" {

const char* nbody_last_error(void) { return g_err.c_str(); }

const char* nbody_version(void) { return "nbody-gfx950 1.0"; }

size_t nbody_workspace_bytes(int32_t op, int64_t n_total, int32_t num_systems, int64_t steps,
                             int64_t checkpoint_every, int32_t precision)
{
    if (n_total < 1 || n_total > kMaxBodies || num_systems < 1) return 0;
    if (op < NBODY_OP_ACCEL || op > NBODY_OP_ACCEL_SHARD) return 0;
    if (op == NBODY_OP_ACCEL_SHARD && (precision != NBODY_FP64 || num_systems != 1)) return 0;
    if (precision != NBODY_FP64 && precision != NBODY_SPLIT &&
        precision != NBODY_SPLIT_COMPENSATED)
        return 0;
    if ((op == NBODY_OP_ADJOINT || op == NBODY_OP_ADJOINT_SWEEP) &&
        (checkpoint_every < 1 || steps < 0))
        return 0;
    return layout(op, n_total, num_systems, steps, checkpoint_every, precision).total;
}

int32_t nbody_accel(const double* pos, const double* vel, const double* mass, int64_t n,
                    double G, double dt, int64_t steps, double* acc_out, int32_t precision,
                    double small_mass, void* workspace, size_t workspace_bytes, void* stream)
{
    (void)vel;
    (void)dt;
    (void)steps;
    g_err.clear();
    NB_TRY(check_common(pos, mass, n, G));
    NB_TRY(check_prec(precision, small_mass));
    NB_TRY(check_comp_size(precision, n));
    if (!acc_out) return fail(NBODY_EINVAL, "acc_out is NULL");
    const Layout L = layout(NBODY_OP_ACCEL, n, 1, 0, 1, precision);
    NB_TRY(check_ws(workspace, workspace_bytes, L.total));
    hipStream_t s = static_cast<hipStream_t>(stream);
    const Tile tile = pick_tile(0, precision, n);
    const int chunks = force_slots(precision, n, tile);
    double* part = at<double>(workspace, L.part);
    uint32_t* flags = at<uint32_t>(workspace, L.flags);
    double* gm = at<double>(workspace, L.gm);
    const bool group = group_route(precision, n);
    const bool small = tile.variant == 3;
    const bool fused = tile.variant == 4;
    if (precision == NBODY_FP64 && (group || small || fused)) {
        // One kernel reads the bodies and stores the accelerations: where those
        // go over its inputs, by way of the workspace (a workgroup that starts
        // late still reads what another has long stored).
        const bool over = overlap(acc_out, 3 * n, pos, 3 * n) || overlap(acc_out, 3 * n, mass, n);
        double* acc = over ? at<double>(workspace, L.alt) : acc_out;
        if (group) {
            NB_TRY(group_run(0, pos, nullptr, nullptr, mass, n, nullptr, G, 0.0, 0, 0, acc,
                             nullptr, nullptr, nullptr, flags, s));
        } else if (small) {
            NB_HIP(launch_run_small(0, tile, pos, nullptr, nullptr, mass, n, nullptr, G, 0.0, 0, 0,
                                    0, acc, nullptr, flags, s));
        } else {
            NB_HIP(launch_scale(mass, G, n, gm, s));
            NB_HIP(launch_step_fused(0, tile, pos, nullptr, nullptr, gm, n, nullptr, 0.0, kStoreAcc,
                                     acc, flags, s));
        }
        if (over) NB_HIP(launch_scale(acc, 1.0, 3 * n, acc_out, s));
        return NBODY_OK;
    }
    if (precision == NBODY_FP64) {
        NB_HIP(launch_scale(mass, G, n, gm, s));
        NB_HIP(launch_force(0, tile, pos, mass, gm, n, nullptr, G, part, s));
        NB_HIP(launch_step(part, chunks, nullptr, n, nullptr, nullptr, nullptr, acc_out, 0.0,
                           kStoreAcc, flags, s));
        return NBODY_OK;
    }
    ClassOrdered c;
    NB_TRY(split_prepare(workspace, L, pos, nullptr, mass, n, G, small_mass, s, &c));
    if (group)
        return group_run(precision, c.pos, nullptr, nullptr, c.mass, n, c.nmaj, G, 0.0, 0, 0,
                         acc_out, nullptr, nullptr, nullptr, flags, s, c.perm);
    if (!small && !fused) {
        NB_HIP(launch_force(precision, tile, c.pos, c.mass, c.gm, n, c.nmaj, G, part, s));
        NB_HIP(launch_step(part, chunks, nullptr, n, nullptr, nullptr, nullptr, acc_out, 0.0,
                           kStoreAcc, flags, s, c.perm));
        return NBODY_OK;
    }
    double* acc_c = at<double>(workspace, L.alt_c);
    if (small)
        NB_HIP(launch_run_small(1, tile, c.pos, nullptr, nullptr, c.mass, n, c.nmaj, G, 0.0, 0, 0,
                                0, acc_c, nullptr, flags, s));
    else
        NB_HIP(launch_step_fused(1, tile, c.pos, nullptr, nullptr, c.gm, n, c.nmaj, 0.0, kStoreAcc,
                                 acc_c, flags, s));
    NB_HIP(launch_scatter(c.perm, n, acc_c, acc_out, nullptr, nullptr, s));
    return NBODY_OK;
}

}  // extern "C"

namespace {

// Checks the arguments of a velocity-Verlet run (the workspace excepted).
int check_run(const double* pos, const double* vel, const double* mass, int64_t n, double G,
              double dt, int64_t steps, int32_t precision, double small_mass)
{
    NB_TRY(check_common(pos, mass, n, G));
    NB_TRY(check_prec(precision, small_mass));
    NB_TRY(check_comp_size(precision, n));
    if (!vel) return fail(NBODY_EINVAL, "vel is NULL");
    if (steps < 0) return fail(NBODY_EINVAL, "steps must be >= 0");
    if (!std::isfinite(dt)) return fail(NBODY_EINVAL, "dt is not finite");
    return NBODY_OK;
}

// The step loop of nbody_verlet_run on the workspace `ws` (laid out as L),
// replayed from graphs or enqueued directly.
int verlet_run_on(double* pos, double* vel, const double* mass, int64_t n, double G, double dt,
                  int64_t steps, int32_t precision, double small_mass, void* ws, const Layout& L,
                  hipStream_t s, bool use_graph)
{
    if (steps == 0) return NBODY_OK;
    StepPlan P;
    P.prec = precision;
    P.tile = pick_tile(0, precision, n);
    P.chunks = force_slots(precision, n, P.tile);
    P.n = n;
    P.G = G;
    P.dt = dt;
    P.part = at<double>(ws, L.part);
    P.flags = at<uint32_t>(ws, L.flags);
    double* alt = at<double>(ws, L.alt);
    double* gm = at<double>(ws, L.gm);
    P.gm = gm;
    const bool group = group_route(precision, n);
    const bool small = P.tile.variant == 3;
    if (precision == NBODY_FP64) {
        if (group)
            return group_run(0, pos, pos, vel, mass, n, nullptr, G, dt, steps, steps, nullptr,
                             nullptr, P.part, group_reg(P.flags), P.flags, s);
        if (small) {
            NB_HIP(launch_run_small(0, P.tile, pos, pos, vel, mass, n, nullptr, G, dt, 0, steps,
                                    steps, nullptr, nullptr, P.flags, s));
            return NBODY_OK;
        }
        P.mass = mass;
        P.vel = vel;
        NB_HIP(launch_scale(mass, G, n, gm, s));
        // r_0 in the caller's buffer, r_1 in the workspace's: the same roles
        // for every run (the captured graphs do not depend on the step
        // count); an odd run ends in the workspace's buffer and is copied
        // back by a kernel (1.0 * x is exact)
        P.buf[0] = pos;
        P.buf[1] = alt;
        NB_TRY(run_steps(P, steps, s, use_graph));
        if (steps & 1) NB_HIP(launch_scale(alt, 1.0, 3 * n, pos, s));
        return NBODY_OK;
    }
    ClassOrdered c;
    NB_TRY(split_prepare(ws, L, pos, vel, mass, n, G, small_mass, s, &c));
    const double* r_end = c.pos;
    if (group) {
        NB_TRY(group_run(precision, c.pos, c.pos, c.vel, c.mass, n, c.nmaj, G, dt, steps, steps,
                         nullptr, nullptr, P.part, group_reg(P.flags), P.flags, s));
    } else if (small) {
        NB_HIP(launch_run_small(1, P.tile, c.pos, c.pos, c.vel, c.mass, n, c.nmaj, G, dt, 0, steps,
                                steps, nullptr, nullptr, P.flags, s));
    } else {
        P.nmaj = c.nmaj;
        P.mass = c.mass;
        P.vel = c.vel;
        P.buf[0] = c.pos;
        P.buf[1] = at<double>(ws, L.alt_c);
        NB_TRY(run_steps(P, steps, s, use_graph));
        r_end = P.buf[steps & 1];
    }
    NB_HIP(launch_scatter(c.perm, n, r_end, pos, c.vel, vel, s));
    return NBODY_OK;
}

// Scratch of nbody_verlet_run_static: one array per device, held until the
// process ends.  Host code never uses the array's name as an address: the
// device address comes from hipGetSymbolAddress, once per device.
constexpr size_t kStaticScratchBytes = (size_t)32 << 20;
__device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

int static_scratch(void** out)
{
    int dev = 0;
    NB_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices)
        return fail(NBODY_EUNSUPPORTED, "device %d is beyond the library's %d", dev, kMaxDevices);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(NBODY_EHIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return NBODY_OK;
}

}  // namespace

extern "C" {

int32_t nbody_verlet_run(double* pos, double* vel, const double* mass, int64_t n, double G,
                         double dt, int64_t steps, int32_t precision, double small_mass,
                         void* workspace, size_t workspace_bytes, void* stream)
{
    g_err.clear();
    NB_TRY(check_run(pos, vel, mass, n, G, dt, steps, precision, small_mass));
    const Layout L = layout(NBODY_OP_RUN, n, 1, steps, 1, precision);
    NB_TRY(check_ws(workspace, workspace_bytes, L.total));
    return verlet_run_on(pos, vel, mass, n, G, dt, steps, precision, small_mass, workspace, L,
                         static_cast<hipStream_t>(stream), true);
}

int32_t nbody_verlet_run_static(double* pos, double* vel, const double* mass, int64_t n, double G,
                                double dt, int64_t steps, int32_t precision, double small_mass,
                                void* stream)
{
    g_err.clear();
    NB_TRY(check_run(pos, vel, mass, n, G, dt, steps, precision, small_mass));
    const Layout L = layout(NBODY_OP_RUN, n, 1, steps, 1, precision);
    if (L.total > kStaticScratchBytes)
        return fail(NBODY_EUNSUPPORTED,
                    "n = %lld needs %zu bytes of scratch; the static scratch holds %zu "
                    "(use nbody_verlet_run with a workspace)",
                    (long long)n, L.total, kStaticScratchBytes);
    if (steps == 0) return NBODY_OK;
    void* ws = nullptr;
    NB_TRY(static_scratch(&ws));
    hipStream_t s = static_cast<hipStream_t>(stream);
    // the flags word starts each call at zero (a fill kernel, not a memset)
    NB_HIP(launch_fill(at<double>(ws, L.flags), 0.0, 1, s));
    return verlet_run_on(pos, vel, mass, n, G, dt, steps, precision, small_mass, ws, L, s, false);
}

int32_t nbody_rk4_run(double* pos, double* vel, const double* mass, int64_t n, double G,
                      double dt, int64_t steps, int32_t precision, double small_mass,
                      void* workspace, size_t workspace_bytes, void* stream)
{
    g_err.clear();
    NB_TRY(check_common(pos, mass, n, G));
    NB_TRY(check_prec(precision, small_mass));
    NB_TRY(check_comp_size(precision, n));
    if (!vel) return fail(NBODY_EINVAL, "vel is NULL");
    if (steps < 0) return fail(NBODY_EINVAL, "steps must be >= 0");
    if (!std::isfinite(dt)) return fail(NBODY_EINVAL, "dt is not finite");
    const Layout L = layout(NBODY_OP_RK4, n, 1, steps, 1, precision);
    NB_TRY(check_ws(workspace, workspace_bytes, L.total));
    if (steps == 0) return NBODY_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);

    StepPlan P;
    P.prec = precision;
    P.tile = pick_tile(0, precision, n);
    if (P.tile.variant == 3 || P.tile.variant == 4)   // whole-step variants
        P.tile = force_only_tile(precision, n);
    P.chunks = force_slots(precision, n, P.tile);
    P.n = n;
    P.G = G;
    P.dt = dt;
    P.part = at<double>(workspace, L.part);
    P.flags = at<uint32_t>(workspace, L.flags);
    double* gm = at<double>(workspace, L.gm);
    P.gm = gm;
    double* rs = at<double>(workspace, L.alt);
    double* vs = at<double>(workspace, L.rk_vs);
    double* sr = at<double>(workspace, L.rk_sr);
    double* sv = at<double>(workspace, L.rk_sv);
    if (precision == NBODY_FP64) {
        P.mass = mass;
        NB_HIP(launch_scale(mass, G, n, gm, s));
        return rk4_steps(P, pos, vel, rs, vs, sr, sv, steps, s);
    }
    ClassOrdered c;
    NB_TRY(split_prepare(workspace, L, pos, vel, mass, n, G, small_mass, s, &c));
    P.mass = c.mass;
    P.nmaj = c.nmaj;
    NB_TRY(rk4_steps(P, c.pos, c.vel, rs, vs, sr, sv, steps, s));
    NB_HIP(launch_scatter(c.perm, n, c.pos, pos, c.vel, vel, s));
    return NBODY_OK;
}

int32_t nbody_energy(const double* pos, const double* vel, const double* mass, int64_t n,
                     double G, double* out, void* workspace, size_t workspace_bytes, void* stream)
{
    g_err.clear();
    NB_TRY(check_common(pos, mass, n, G));
    if (!vel || !out) return fail(NBODY_EINVAL, "vel or out is NULL");
    const Layout L = layout(NBODY_OP_ENERGY, n, 1, 0, 1, NBODY_FP64);
    NB_TRY(check_ws(workspace, workspace_bytes, L.total));
    hipStream_t s = static_cast<hipStream_t>(stream);
    // the partial region holds chunk_cap(n) slots of 3 n doubles for this op
    NB_HIP(launch_energy(pos, vel, mass, n, G, at<double>(workspace, L.part), 3 * n * chunk_cap(n),
                         out, s));
    return NBODY_OK;
}

int32_t nbody_momenta(const double* pos, const double* vel, const double* mass, int64_t n,
                      double* out, void* stream)
{
    g_err.clear();
    NB_TRY(check_common(pos, mass, n, 1.0));
    if (!vel || !out) return fail(NBODY_EINVAL, "vel or out is NULL");
    NB_HIP(launch_momenta(pos, vel, mass, n, out, static_cast<hipStream_t>(stream)));
    return NBODY_OK;
}

int32_t nbody_get_flags(void* workspace, void* stream, int32_t clear, int32_t* flags_host)
{
    g_err.clear();
    if (!workspace || !flags_host) return fail(NBODY_EINVAL, "null workspace or flags pointer");
    hipStream_t s = static_cast<hipStream_t>(stream);
    uint32_t v = 0;
    NB_HIP(hipMemcpyAsync(&v, workspace, sizeof v, hipMemcpyDeviceToHost, s));
    NB_HIP(hipStreamSynchronize(s));
    *flags_host = (int32_t)v;
    if (clear) {
        NB_HIP(hipMemsetAsync(workspace, 0, sizeof(uint32_t), s));
        NB_HIP(hipStreamSynchronize(s));
    }
    return NBODY_OK;
}

int32_t nbody_get_tile(int32_t kind, int32_t precision, int64_t n, nbody_tile* tile_host)
{
    g_err.clear();
    if (!tile_host || kind < 0 || kind > 2 || (kind != 2 && n < 1))
        return fail(NBODY_EINVAL, "bad arguments");
    NB_TRY(check_prec(precision, 0.0));
    if (kind == 2) n = 0;
    const Tile t = pick_tile(kind, precision, n);
    tile_host->targets_per_lane = t.tpl;
    tile_host->waves = t.waves;
    tile_host->chunks = t.chunks;
    tile_host->variant = t.variant;
    return NBODY_OK;
}

// Checks a tile and enters it: as the caller's choice for runs too (forced), or
// as the autotuner's.
static int store_tile(int32_t kind, int32_t precision, int64_t n, const nbody_tile* tile_host,
                      bool forced)
{
    if (!tile_host || kind < 0 || kind > 2 || (kind != 2 && n < 1))
        return fail(NBODY_EINVAL, "bad arguments");
    NB_TRY(check_prec(precision, 0.0));
    if (kind == 2) n = 0;
    Tile t{tile_host->targets_per_lane, tile_host->waves, tile_host->chunks, tile_host->variant};
    if (!tile_supported(t) ||
        (kind == 1 && t.variant != 5 && (t.tpl > 2 || t.waves > 4 || t.variant > 1)) ||
        (precision == NBODY_SPLIT_COMPENSATED && t.variant != 5) ||
        (t.variant == 3 && (kind != 0 || n > kSmallMax)) || (t.variant == 4 && kind != 0) ||
        (t.variant == 5 && !mutual_fits(kind, precision, n)))
        return fail(NBODY_EINVAL, "unsupported tile (%d, %d, %d, variant %d) for kind %d",
                    t.tpl, t.waves, t.chunks, t.variant, kind);
    std::lock_guard<std::mutex> lk(g_mu);
    g_tiles[std::make_tuple(kind, precision, size_class(n))] = TunedTile{t, forced};
    return NBODY_OK;
}

int32_t nbody_set_tile(int32_t kind, int32_t precision, int64_t n, const nbody_tile* tile_host)
{
    g_err.clear();
    return store_tile(kind, precision, n, tile_host, true);
}

int32_t nbody_set_tuned_tile(int32_t kind, int32_t precision, int64_t n,
                             const nbody_tile* tile_host)
{
    g_err.clear();
    return store_tile(kind, precision, n, tile_host, false);
}

void nbody_reset_caches(void)
{
    drop_graphs();
    std::lock_guard<std::mutex> lk(g_mu);
    g_tiles.clear();
    drop_batch_plans();
}

// The adjoint's forward run (checkpoints (r, v) every K steps into ck, the
// final state into pos_out / vel_out) and/or its reverse sweep from those
// checkpoints, on a workspace laid out as L.  Arguments are checked.
static int adjoint_core(const double* pos0, const double* vel0, const double* mass, int64_t n,
                        double G, double dt, int64_t steps, int64_t checkpoint_every, double* ck,
                        bool forward, bool reverse, const double* grad_posT,
                        const double* grad_velT, double* grad_pos0, double* grad_vel0,
                        double* grad_mass, double* pos_out, double* vel_out, void* workspace,
                        const Layout& L, hipStream_t s)
{
    const size_t b3 = 3 * n * sizeof(double);
    const int64_t K = checkpoint_every;
    const int64_t nck = (steps + K - 1) / K;
    double* seg = at<double>(workspace, L.seg);
    double* alt = at<double>(workspace, L.alt);
    double* lam_r = at<double>(workspace, L.lam_r);
    double* lam_v = at<double>(workspace, L.lam_v);
    double* g_m = at<double>(workspace, L.g_m);
    double* u = at<double>(workspace, L.u);
    double* vtmp = at<double>(workspace, L.vtmp);
    double* part = at<double>(workspace, L.part);
    double* seg2 = at<double>(workspace, L.seg2);
    double* part2 = at<double>(workspace, L.part2);
    double* vtmp2 = at<double>(workspace, L.vtmp2);
    uint32_t* flags = at<uint32_t>(workspace, L.flags);
    SideStream* side = nullptr;
    NB_TRY(side_stream(&side));
    std::lock_guard<std::mutex> adjoint_lock(side->adjoint_mu);
    hipStream_t sb = side->stream;
    auto ck_r = [&](int64_t k) { return ck + k * 6 * n; };
    auto ck_v = [&](int64_t k) { return ck + k * 6 * n + 3 * n; };

    // Forward run, storing (r, v) every K steps.  Each segment is a complete
    // run of nbody_verlet_run, so segments chain bit for bit.  A segment runs
    // on fixed work buffers (position ping-pong w0/w1, velocity wv) from a
    // captured graph, so every full-length segment replays the same graph.
    double* w0 = alt;
    double* w1 = u;
    double* wv = vtmp;
    StepPlan P;
    P.prec = NBODY_FP64;
    P.tile = pick_tile(0, NBODY_FP64, n);
    P.chunks = force_slots(NBODY_FP64, n, P.tile);
    P.n = n;
    P.G = G;
    P.dt = dt;
    double* gm = at<double>(workspace, L.gm);
    P.mass = mass;
    P.gm = gm;
    P.part = part;
    P.flags = flags;
    P.vel = wv;
    P.buf[0] = w0;
    P.buf[1] = w1;
    // The recompute takes the forward run's kernel, whichever that is: the sweep
    // linearises about the very positions of the run, bit for bit.
    const bool group = group_route(NBODY_FP64, n);
    // The group kernel's sweep does all positions of a segment in one launch (the
    // closing half kick too), beside the group kernel's recompute or in turn with
    // it; then the second stream is the caller's.
    const bool group_rev = group_vjp_route(group, n, std::min(K, steps));
    if (group_rev) {
        bool beside;
        (void)group_vjp_shape(n, &beside);
        if (!beside) sb = s;
    }
    const bool small = P.tile.variant == 3;
    const Tile vt = pick_tile(1, NBODY_FP64, n);
    const int vchunks = vjp_chunks(n, vt);
    auto key_of = [&](uint64_t kind, int64_t kseg, uint64_t first, const double* segp) {
        GraphKey key;
        key.v = {kind, (uint64_t)kseg, first, (uint64_t)n, bits(G), bits(dt),
                 (uint64_t)P.tile.tpl, (uint64_t)P.tile.waves, (uint64_t)P.tile.chunks,
                 (uint64_t)P.tile.variant, (uint64_t)vt.tpl, (uint64_t)vt.waves,
                 (uint64_t)vt.chunks, ptrbits(mass), ptrbits(P.gm), ptrbits(part), ptrbits(flags),
                 ptrbits(w0), ptrbits(w1), ptrbits(wv), ptrbits(segp), ptrbits(lam_r),
                 ptrbits(lam_v), ptrbits(g_m), ptrbits(part2), ptrbits(vtmp2)};
        return key;
    };
    // segments longer than this run their launches directly instead of from
    // a graph (a graph is captured once per segment length and replayed)
    constexpr int64_t kMaxGraphSegment = 1024;
    auto maybe_graph_on = [&](hipStream_t st, const GraphKey& key, int64_t kseg,
                              auto&& body) -> int {
        if (kseg <= kMaxGraphSegment) return run_graph(key, st, body);
        return body(st);
    };
    auto maybe_graph = [&](const GraphKey& key, int64_t kseg, auto&& body) -> int {
        return maybe_graph_on(s, key, kseg, body);
    };
    if (!group) NB_HIP(launch_scale(mass, G, n, gm, s));
    if (forward) {
        NB_HIP(hipMemcpyAsync(ck_r(0), pos0, b3, hipMemcpyDeviceToDevice, s));
        NB_HIP(hipMemcpyAsync(ck_v(0), vel0, b3, hipMemcpyDeviceToDevice, s));
        for (int64_t c = 0; c < nck; ++c) {
            const int64_t kseg = std::min(K, steps - c * K);
            NB_HIP(hipMemcpyAsync(w0, ck_r(c), b3, hipMemcpyDeviceToDevice, s));
            NB_HIP(hipMemcpyAsync(wv, ck_v(c), b3, hipMemcpyDeviceToDevice, s));
            const double* r_end = w0;
            if (group) {
                NB_TRY(group_run(0, w0, w0, wv, mass, n, nullptr, G, dt, kseg, kseg, nullptr,
                                      nullptr, part, group_reg(flags), flags, s));
            } else if (small) {
                NB_HIP(launch_run_small(0, P.tile, w0, w0, wv, mass, n, nullptr, G, dt, 0, kseg, kseg,
                                        nullptr, nullptr, flags, s));
            } else {
                NB_TRY(maybe_graph(key_of(2, kseg, 0, seg), kseg, [&](hipStream_t cs) {
                    for (int64_t i = 0; i <= kseg; ++i) {
                        const int st = step_launch(P, i, kseg, cs);
                        if (st != NBODY_OK) return st;
                    }
                    return (int)NBODY_OK;
                }));
                r_end = P.buf[kseg & 1];
            }
            NB_HIP(hipMemcpyAsync(ck_r(c + 1), r_end, b3, hipMemcpyDeviceToDevice, s));
            NB_HIP(hipMemcpyAsync(ck_v(c + 1), wv, b3, hipMemcpyDeviceToDevice, s));
        }
        if (pos_out) NB_HIP(hipMemcpyAsync(pos_out, ck_r(nck), b3, hipMemcpyDeviceToDevice, s));
        if (vel_out) NB_HIP(hipMemcpyAsync(vel_out, ck_v(nck), b3, hipMemcpyDeviceToDevice, s));
    }
    if (!reverse) return NBODY_OK;

    // Reverse sweep: one transpose-Jacobian product of Eq. (1) per force
    // pass, its chunk reduction fused with the adjoint of the drift that
    // precedes the pass (lam_v += dt lam_r), the cotangent c lam_v scaled
    // inside the product.
    NB_HIP(hipMemcpyAsync(lam_r, grad_posT, b3, hipMemcpyDeviceToDevice, s));
    NB_HIP(hipMemcpyAsync(lam_v, grad_velT, b3, hipMemcpyDeviceToDevice, s));
    NB_HIP(launch_fill(g_m, 0.0, n, s));
    if (steps > 0 && !group_rev) {
        // closing half kick of the last step: v_T = v_{T-1/2} + dt/2 a(r_T)
        NB_HIP(launch_vjp(vt, ck_r(nck), mass, lam_v, 0.5 * dt, n, G, part, s));
        NB_HIP(launch_vjp_reduce(part, vchunks, n, lam_r, g_m, lam_v, dt, true, s));
    }
    // Segments in reverse order, pipelined over two streams: the side stream
    // recomputes the positions of segment c - 1 (from its checkpoint, into the
    // other segment buffer, with its own partials and velocity) while the
    // caller's stream runs the reverse sweep of segment c.  Events order a
    // buffer's recompute after the sweep that last read it and before the
    // sweep that reads it.
    StepPlan R = P;   // recompute plan: positions of one segment into seg slots
    R.vel = vtmp2;
    R.part = part2;
    double* segbuf[2] = {seg, seg2};
    bool freed_recorded[2] = {false, false};
    auto recompute = [&](int64_t c) -> int {
        const int b = (int)(c & 1);
        const int64_t kseg = std::min(K, steps - c * K);
        double* sg = segbuf[b];
        if (freed_recorded[b]) NB_HIP(hipStreamWaitEvent(sb, side->freed[b], 0));
        NB_HIP(hipMemcpyAsync(sg, ck_r(c), b3, hipMemcpyDeviceToDevice, sb));
        NB_HIP(hipMemcpyAsync(vtmp2, ck_v(c), b3, hipMemcpyDeviceToDevice, sb));
        if (group) {
            // (the segment's positions r_{cK+1} .. r_{cK+kseg-1}, as below)
            if (kseg >= 2)
                NB_TRY(group_run(0, sg, nullptr, vtmp2, mass, n, nullptr, G, dt, kseg - 2,
                                      kseg, nullptr, sg + 3 * n, part2, group_reg(flags, 1),
                                      flags, sb));
        } else NB_TRY(maybe_graph_on(sb, key_of(3, kseg, 0, sg), kseg, [&](hipStream_t cs) -> int {
            // positions r_{cK+1} .. r_{cK+kseg-1} of the segment into its slots
            if (small && kseg >= 2)
                NB_HIP(launch_run_small(0, R.tile, sg, nullptr, vtmp2, mass, n, nullptr, G, dt, 0,
                                        kseg - 2, kseg, nullptr, sg + 3 * n, flags, cs));
            for (int64_t k = 0; !small && k + 1 < kseg; ++k) {
                double* pin = sg + k * 3 * n;
                NB_TRY(force_and_step(R, pin, pin + 3 * n, (k > 0 ? kClose : 0) | kOpen, cs));
            }
            return (int)NBODY_OK;
        }));
        NB_HIP(hipEventRecord(side->ready[b], sb));
        return NBODY_OK;
    };
    auto sweep = [&](int64_t c) -> int {
        const int b = (int)(c & 1);
        const int64_t kseg = std::min(K, steps - c * K);
        const double* sg = segbuf[b];
        NB_HIP(hipStreamWaitEvent(s, side->ready[b], 0));
        if (group_rev) {   // (two positions at least: K of them, or one and the last)
            GroupVjpArgs A{};
            A.seg = sg;
            A.last = c == nck - 1 ? ck_r(nck) : nullptr;
            A.mass = mass;
            A.lam_r = lam_r;
            A.lam_v = lam_v;
            A.g_m = g_m;
            A.xbuf = part;
            A.reg = group_reg(flags, 2);
            A.n = n;
            A.G = G;
            A.dt = dt;
            A.k1 = kseg - 1;
            A.count = kseg + (A.last ? 1 : 0);
            A.first = c == 0 ? 1 : 0;
            NB_TRY(group_sweep(A, s));
        } else NB_TRY(maybe_graph(key_of(4, kseg, c == 0, sg), kseg, [&](hipStream_t cs) -> int {
            for (int64_t k = kseg - 1; k >= 0; --k) {
                const int64_t i = c * K + k;
                // kick v_{i+1/2} = v_{i-1/2} + dt a(r_i)   (dt/2 for i = 0); the
                // drift r_i = r_{i-1} + dt v_{i-1/2} before it (i > 0)
                NB_HIP(launch_vjp(vt, sg + k * 3 * n, mass, lam_v, i > 0 ? dt : 0.5 * dt, n, G,
                                  part, cs));
                NB_HIP(launch_vjp_reduce(part, vchunks, n, lam_r, g_m, lam_v, dt, i > 0, cs));
            }
            return (int)NBODY_OK;
        }));
        NB_HIP(hipEventRecord(side->freed[b], s));
        freed_recorded[b] = true;
        return NBODY_OK;
    };
    if (nck > 0) {
        // the checkpoints (forward run, above) and G m come before any recompute
        NB_HIP(hipEventRecord(side->fwd, s));
        NB_HIP(hipStreamWaitEvent(sb, side->fwd, 0));
        NB_TRY(recompute(nck - 1));
        for (int64_t c = nck - 1; c >= 0; --c) {
            if (c > 0) NB_TRY(recompute(c - 1));
            NB_TRY(sweep(c));
        }
    }
    NB_HIP(hipMemcpyAsync(grad_pos0, lam_r, b3, hipMemcpyDeviceToDevice, s));
    NB_HIP(hipMemcpyAsync(grad_vel0, lam_v, b3, hipMemcpyDeviceToDevice, s));
    NB_HIP(hipMemcpyAsync(grad_mass, g_m, n * sizeof(double), hipMemcpyDeviceToDevice, s));
    return NBODY_OK;
}

static int check_adjoint(const double* pos0, const double* vel0, const double* mass, int64_t n,
                         double G, double dt, int64_t steps, int64_t checkpoint_every)
{
    NB_TRY(check_common(pos0, mass, n, G));
    if (!vel0) return fail(NBODY_EINVAL, "null velocity pointer");
    if (steps < 0) return fail(NBODY_EINVAL, "steps must be >= 0");
    if (checkpoint_every < 1) return fail(NBODY_EINVAL, "checkpoint_every must be >= 1");
    if (!std::isfinite(dt)) return fail(NBODY_EINVAL, "dt is not finite");
    return NBODY_OK;
}

int32_t nbody_verlet_adjoint(const double* pos0, const double* vel0, const double* mass, int64_t n,
                             double G, double dt, int64_t steps, int64_t checkpoint_every,
                             const double* grad_posT, const double* grad_velT, double* grad_pos0,
                             double* grad_vel0, double* grad_mass, double* pos_out,
                             double* vel_out, void* workspace, size_t workspace_bytes,
                             void* stream)
{
    g_err.clear();
    NB_TRY(check_adjoint(pos0, vel0, mass, n, G, dt, steps, checkpoint_every));
    if (!grad_posT || !grad_velT || !grad_pos0 || !grad_vel0 || !grad_mass)
        return fail(NBODY_EINVAL, "null cotangent or gradient pointer");
    const Layout L = layout(NBODY_OP_ADJOINT, n, 1, steps, checkpoint_every, NBODY_FP64);
    NB_TRY(check_ws(workspace, workspace_bytes, L.total));
    return adjoint_core(pos0, vel0, mass, n, G, dt, steps, checkpoint_every,
                        at<double>(workspace, L.ck), true, true, grad_posT, grad_velT, grad_pos0,
                        grad_vel0, grad_mass, pos_out, vel_out, workspace, L,
                        static_cast<hipStream_t>(stream));
}

int32_t nbody_verlet_checkpoints(const double* pos0, const double* vel0, const double* mass,
                                 int64_t n, double G, double dt, int64_t steps,
                                 int64_t checkpoint_every, double* checkpoints, double* pos_out,
                                 double* vel_out, void* workspace, size_t workspace_bytes,
                                 void* stream)
{
    g_err.clear();
    NB_TRY(check_adjoint(pos0, vel0, mass, n, G, dt, steps, checkpoint_every));
    if (!checkpoints) return fail(NBODY_EINVAL, "null checkpoint buffer");
    const Layout L = layout(NBODY_OP_ADJOINT_SWEEP, n, 1, steps, checkpoint_every, NBODY_FP64);
    NB_TRY(check_ws(workspace, workspace_bytes, L.total));
    return adjoint_core(pos0, vel0, mass, n, G, dt, steps, checkpoint_every, checkpoints, true,
                        false, nullptr, nullptr, nullptr, nullptr, nullptr, pos_out, vel_out,
                        workspace, L, static_cast<hipStream_t>(stream));
}

int32_t nbody_verlet_adjoint_from_checkpoints(const double* checkpoints, const double* mass,
                                              int64_t n, double G, double dt, int64_t steps,
                                              int64_t checkpoint_every, const double* grad_posT,
                                              const double* grad_velT, double* grad_pos0,
                                              double* grad_vel0, double* grad_mass,
                                              void* workspace, size_t workspace_bytes,
                                              void* stream)
{
    g_err.clear();
    if (!checkpoints) return fail(NBODY_EINVAL, "null checkpoint buffer");
    NB_TRY(check_adjoint(checkpoints, checkpoints + 3 * n, mass, n, G, dt, steps,
                         checkpoint_every));
    if (!grad_posT || !grad_velT || !grad_pos0 || !grad_vel0 || !grad_mass)
        return fail(NBODY_EINVAL, "null cotangent or gradient pointer");
    const Layout L = layout(NBODY_OP_ADJOINT_SWEEP, n, 1, steps, checkpoint_every, NBODY_FP64);
    NB_TRY(check_ws(workspace, workspace_bytes, L.total));
    return adjoint_core(nullptr, nullptr, mass, n, G, dt, steps, checkpoint_every,
                        const_cast<double*>(checkpoints), false, true, grad_posT, grad_velT,
                        grad_pos0, grad_vel0, grad_mass, nullptr, nullptr, workspace, L,
                        static_cast<hipStream_t>(stream));
}

}  // extern "C"

namespace {

// Work list of the batched launch, cached per (offsets, tile).
struct BatchPlan {
    std::vector<BatchUnit> units;
    std::vector<int8_t> bchunks;
    std::vector<int64_t> offsets;
    std::vector<GroupUnit> group_units;   // the group kernel's list instead
    int64_t n_max = 0;
};

// Work lists of recent ensembles (host memory; uploaded each run).  At most
// kMaxBatchPlans are kept, the least recently used dropped first.
constexpr size_t kMaxBatchPlans = 8;
std::map<std::vector<int64_t>, std::shared_ptr<BatchPlan>> g_batch;
std::map<std::vector<int64_t>, uint64_t> g_batch_used;
uint64_t g_batch_tick = 0;

void drop_batch_plans()
{
    // uploads of a plan read its host vectors asynchronously
    (void)hipDeviceSynchronize();
    g_batch.clear();
    g_batch_used.clear();
}

constexpr int64_t kBatchChunkLen = 1024;   // sources per chunk in the ensemble

// Drops the least recently used work list when the cache is full.  Call with
// g_mu held.
void evict_batch_plan_locked()
{
    if (g_batch.size() < kMaxBatchPlans) return;
    // uploads of the dropped plan read its host vectors asynchronously
    (void)hipDeviceSynchronize();
    auto victim = g_batch.begin();
    for (auto jt = g_batch.begin(); jt != g_batch.end(); ++jt)
        if (g_batch_used[jt->first] < g_batch_used[victim->first]) victim = jt;
    g_batch_used.erase(victim->first);
    g_batch.erase(victim);
}

std::shared_ptr<BatchPlan> batch_plan(const int64_t* offs, int32_t ns, const Tile& t)
{
    std::vector<int64_t> key(offs, offs + ns + 1);
    key.push_back(t.tpl);
    key.push_back(t.waves);
    key.push_back(t.variant);
    std::lock_guard<std::mutex> lk(g_mu);
    g_batch_used[key] = ++g_batch_tick;
    auto it = g_batch.find(key);
    if (it != g_batch.end()) return it->second;
    evict_batch_plan_locked();
    auto bp = std::make_shared<BatchPlan>();
    bp->offsets.assign(offs, offs + ns + 1);
    const int64_t n_total = offs[ns];
    bp->bchunks.resize(n_total);
    if (t.variant == 5) {
        // each pair once: units (system, g, r), r >= g, over the system's
        // ranges, whose count is the system's number of partial slots
        for (int32_t k = 0; k < ns; ++k) {
            const int64_t nk = offs[k + 1] - offs[k];
            const int R = mutual_ranges(nk);
            if (R > kBatchSlots) {
                g_batch_used.erase(key);
                return nullptr;
            }
            for (int g = 0; g < R; ++g)
                for (int r = g; r < R; ++r) {
                    BatchUnit u;
                    u.body0 = offs[k];
                    u.n = (int32_t)nk;
                    u.sys = k;
                    u.tblock = g;
                    u.chunk = r;
                    u.chunks = R;
                    u.pad = 0;
                    bp->units.push_back(u);
                }
            std::fill(bp->bchunks.begin() + offs[k], bp->bchunks.begin() + offs[k + 1], (int8_t)R);
        }
        g_batch[key] = bp;
        return bp;
    }
    const int64_t tb_size = targets_per_block(t);
    for (int32_t k = 0; k < ns; ++k) {
        const int64_t nk = offs[k + 1] - offs[k];
        const int chunks = (int)std::min<int64_t>(kBatchChunkMax,
                                                  std::max<int64_t>(1, (nk + kBatchChunkLen - 1) / kBatchChunkLen));
        Tile tk = t;
        tk.chunks = chunks;
        const int eff = effective_chunks(nk, tk);
        const int64_t tblocks = (nk + tb_size - 1) / tb_size;
        for (int64_t b = 0; b < tblocks; ++b)
            for (int c = 0; c < eff; ++c) {
                BatchUnit u;
                u.body0 = offs[k];
                u.n = (int32_t)nk;
                u.sys = k;
                u.tblock = (int32_t)b;
                u.chunk = c;
                u.chunks = chunks;
                u.pad = 0;
                bp->units.push_back(u);
            }
        std::fill(bp->bchunks.begin() + offs[k], bp->bchunks.begin() + offs[k + 1], (int8_t)eff);
    }
    // Largest systems first, so the persistent grid's static round-robin over
    // the list ends with the cheap units.
    std::stable_sort(bp->units.begin(), bp->units.end(),
                     [](const BatchUnit& a, const BatchUnit& b) { return a.n > b.n; });
    g_batch[key] = bp;
    return bp;
}

int device_cus(int* cus)
{
    int dev = 0;
    NB_HIP(hipGetDevice(&dev));
    NB_HIP(hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, dev));
    return NBODY_OK;
}

int check_offsets(const int64_t* offsets_host, int32_t num_systems)
{
    if (!offsets_host || num_systems < 1) return fail(NBODY_EINVAL, "need offsets and >= 1 system");
    if (offsets_host[0] != 0) return fail(NBODY_EINVAL, "offsets[0] must be 0");
    for (int32_t k = 0; k < num_systems; ++k) {
        if (offsets_host[k + 1] <= offsets_host[k])
            return fail(NBODY_EINVAL, "system %d is empty or offsets decrease", k);
        if (offsets_host[k + 1] - offsets_host[k] > ((int64_t)1 << 24))
            return fail(NBODY_EUNSUPPORTED, "system %d has more than 2^24 bodies", k);
    }
    return NBODY_OK;
}

// The ensemble's tile: the tuned one if nbody_autotune_batched ran, else
// each pair once (4, 4) when every system's ranges fit the workspace and the
// pair-weighted mean system size (sum n^2 / sum n) reaches kBatchMutualMin
// bodies (smaller systems leave its workgroups mostly idle), else the
// one-way heuristic.
constexpr int64_t kBatchMutualMin = 2048;

Tile batch_tile(int prec, const int64_t* offs, int32_t ns)
{
    {
        std::lock_guard<std::mutex> lk(g_mu);
        auto it = g_tiles.find(std::make_tuple(2, prec, size_class(0)));
        if (it != g_tiles.end()) return it->second.tile;
    }
    double sn = 0.0, sn2 = 0.0;
    bool fits = true;
    for (int32_t k = 0; k < ns; ++k) {
        const double nk = (double)(offs[k + 1] - offs[k]);
        sn += nk;
        sn2 += nk * nk;
        fits = fits && mutual_ranges(offs[k + 1] - offs[k]) <= kBatchSlots;
    }
    if (prec == NBODY_SPLIT_COMPENSATED) return Tile{4, 4, 1, 5};   // each pair once only
    if (fits && sn2 >= (double)kBatchMutualMin * sn) return Tile{4, 4, 1, 5};
    return heuristic_tile(2, prec, 0);
}

// Uploads the ensemble's work list for tile t and fills the batched fields of
// P.  An each-pair-once tile whose ranges exceed the workspace's slots for
// some system gives way to the heuristic tile.
int batched_plan_upload(const int64_t* offsets_host, int32_t ns, const Tile& t_in, void* ws,
                        const Layout& L, hipStream_t s, StepPlan* P)
{
    Tile t = t_in;
    auto bp = batch_plan(offsets_host, ns, t);
    if (!bp && P->prec == NBODY_SPLIT_COMPENSATED)
        return fail(NBODY_EUNSUPPORTED, "the compensated split form runs in the each-pair-once "
                                        "pass, which takes ensembles of systems of at most "
                                        "%d bodies", 256 * kBatchSlots);
    if (!bp) {
        t = heuristic_tile(2, P->prec, 0);   // one-way, always planned
        bp = batch_plan(offsets_host, ns, t);
    }
    const int64_t n = offsets_host[ns];
    BatchUnit* units = at<BatchUnit>(ws, L.units);
    int8_t* bchunks = at<int8_t>(ws, L.bchunks);
    // the unit list's room in the workspace (the layout's bound covers every
    // plan: per system at most 16 (n_k/64 + 1) units, and each pair once
    // needs R(R+1)/2 <= 64 (R - 1) + 16 of them for R <= 40 ranges)
    if (bp->units.size() > (L.bchunks - L.units) / sizeof(BatchUnit))
        return fail(NBODY_EUNSUPPORTED, "ensemble work list exceeds the workspace");
    NB_HIP(hipMemcpyAsync(units, bp->units.data(), bp->units.size() * sizeof(BatchUnit),
                          hipMemcpyHostToDevice, s));
    NB_HIP(hipMemcpyAsync(bchunks, bp->bchunks.data(), n, hipMemcpyHostToDevice, s));
    int cus = 0;
    NB_TRY(device_cus(&cus));
    P->tile = t;
    P->units = units;
    P->num_units = (int64_t)bp->units.size();
    P->grid = (int)std::min<int64_t>(P->num_units, (int64_t)cus * (16 / t.waves));
    P->bchunks = bchunks;
    return NBODY_OK;
}

// Class order of the ensemble (split form): partition, gathers and G m.
int batched_split_prepare(const double* pos, const double* vel, const double* mass,
                          const int64_t* offsets_host, int32_t ns, double G, double small_mass,
                          void* ws, const Layout& L, hipStream_t s, StepPlan* P)
{
    const int64_t n = offsets_host[ns];
    int64_t* offs = at<int64_t>(ws, L.offs);
    NB_HIP(hipMemcpyAsync(offs, offsets_host, (ns + 1) * sizeof(int64_t), hipMemcpyHostToDevice, s));
    NB_HIP(hipStreamSynchronize(s));   // offsets_host may be released by the caller on return
    int64_t n_max = 0;
    for (int32_t k = 0; k < ns; ++k) n_max = std::max(n_max, offsets_host[k + 1] - offsets_host[k]);
    P->mass = at<double>(ws, L.mass_c);
    P->gm = at<double>(ws, L.gm);
    P->vel = at<double>(ws, L.vel_c);
    P->buf[0] = at<double>(ws, L.pos_c);
    P->buf[1] = at<double>(ws, L.alt_c);
    NB_HIP(launch_class_order(pos, vel, mass, offs, ns, n, n_max, small_mass, G,
                              at<int32_t>(ws, L.perm), at<int64_t>(ws, L.nmaj), P->buf[0], P->vel,
                              at<double>(ws, L.mass_c), at<double>(ws, L.gm), s));
    P->nmaj = at<int64_t>(ws, L.nmaj);
    return NBODY_OK;
}

// Largest system of an ensemble that runs in the group kernel.
constexpr int64_t kGroupBatchMax = 2048;

// How the workgroups that fit on the chip at once (`slots`) are dealt to the systems
// of an ensemble: so that the longest share is as short as it can be.  By
// size, at most kGroupBatchMax of them however many systems: systems and
// workgroups of each.  A workgroup that takes r virtual groups of tw targets of a
// system of n bodies needs about r (n + 64); systems of one workgroup take turns
// in a slot, a step's latency, about kTurn of these units, at least.
struct GroupShares {
    int64_t n_max = 0, tw = 0;
    std::vector<int32_t> count, wgs;
    double time = 0.0;   // of the longest share, or of a slot's turns together

    int64_t groups(int64_t n) const { return (n + tw - 1) / tw; }
    static double cost(int64_t n) { return (double)(n + 64); }
};

GroupShares group_shares(const int64_t* offs, int32_t ns, int64_t tw, int slots)
{
    constexpr double kTurn = 512.0;
    GroupShares S;
    S.tw = tw;
    S.count.resize(kGroupBatchMax + 1);
    S.wgs.resize(kGroupBatchMax + 1);
    for (int32_t k = 0; k < ns; ++k) {
        const int64_t n = offs[k + 1] - offs[k];
        ++S.count[n];
        S.n_max = std::max(S.n_max, n);
    }
    std::vector<int64_t> sizes;
    for (int64_t n = 1; n <= S.n_max; ++n)
        if (S.count[n]) sizes.push_back(n);
    // the slots needed when nothing takes longer than `time`
    auto needed = [&](double time) {
        double sum = 0.0;
        for (int64_t n : sizes) {
            const int64_t groups = S.groups(n);
            const double r = std::floor(time / S.cost(n));
            const int64_t share = std::max<int64_t>(1, r < (double)groups ? (int64_t)r : groups);
            S.wgs[n] = (int32_t)((groups + share - 1) / share);
            const double turn = std::max(S.cost(n) * (double)groups, kTurn);
            sum += S.count[n] * (S.wgs[n] > 1 ? (double)S.wgs[n]
                                              : std::min(1.0, turn / std::max(time, 1.0)));
        }
        return sum;
    };
    double lo = 0.0, hi = 0.0;   // hi: every system has one workgroup
    double turns = 0.0;
    for (int64_t n : sizes) {
        const double whole = S.cost(n) * (double)S.groups(n);
        hi = std::max(hi, whole);
        turns += S.count[n] * std::max(whole, kTurn);
    }
    hi = std::max(hi, turns / slots);
    for (int step = 0; step < 60 && hi - lo > 1.0; ++step) {
        const double mid = 0.5 * (lo + hi);
        (needed(mid) <= slots ? hi : lo) = mid;
    }
    (void)needed(hi);
    S.time = hi;
    return S;
}

// Whether a large ensemble is left to the pass by launches, which when the chip is
// full has the leaner pair loop but ends each pass with a partly filled round:
// by an estimate of both, us per step, from fits to 720 ensembles of 1e8 to
// 3e8 pairs in both forms (5 to 95 %: 0.80 to 1.15 and 0.83 to 1.14 of the measured
// time).  With the factor none of them is more than 3 % slower than by
// launches (without a choice 58 were, the worst 1.49 times: 280 systems of 998
// bodies 389 against 261), 430 stay, at 0.47 to 1.03 of the time by launches.
bool group_shares_lose(const GroupShares& S, double pairs)
{
    // by launches: units of 128 targets and at most kBatchChunkLen sources, the longest
    // first, in turn over the 1,024 SIMDs; the first SIMD's load and rounds
    int64_t units = 0, first = 0;   // first: unit of the SIMD's next one
    double load = 0.0;
    double wgs = 0.0, total = 0.0;
    for (int64_t n = S.n_max; n > 0; --n) {
        if (!S.count[n]) continue;
        const int64_t chunks = (n + kBatchChunkLen - 1) / kBatchChunkLen;
        units += S.count[n] * chunks * ((n + 127) / 128);
        for (; first < units; first += 1024) load += (double)((n + chunks - 1) / chunks);
        wgs += (double)S.count[n] * S.wgs[n];
        total += (double)S.count[n] * (double)S.groups(n) * S.cost(n);
    }
    const double by_launches =
        23.0 + 0.054 * load + 5.2 * (double)((units + 1023) / 1024) + 0.267e-6 * pairs;
    const double rounds = wgs / 256.0;   // workgroups per CU
    const double here =
        0.0045 * total / 256.0 + 0.0035 * S.time + 11.2 * (std::ceil(rounds) - rounds);
    return here > 0.8 * by_launches;
}

// Whether an ensemble runs in the group kernel (and in which shape, with how
// many workgroups at once): systems of up to kGroupBatchMax bodies too small
// on average for each pair once, and not so many that the pass by launches is
// faster (us per step against it: 128 systems of 40 to 400 bodies 9.3 / 53, 8 of
// 300 to 2,000 28 / 109; of 1,230 ensembles of 1.5e7 to 1e8 pairs none takes more
// than 1.01 times as long; above, by group_shares_lose, up to 3e8).
constexpr double kGroupBatchPairs = 3e8;
constexpr double kGroupBatchAlways = 1e8;
// (a launch takes at most 2^32 threads: 16.7 million systems of one workgroup)
constexpr int32_t kGroupBatchSystems = 1 << 22;

bool batch_group_route(int prec, const int64_t* offs, int32_t ns, GroupShape* shape, int* slots)
{
    if (prec == NBODY_SPLIT_COMPENSATED || ns > kGroupBatchSystems) return false;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        auto it = g_tiles.find(std::make_tuple(2, prec, size_class(0)));
        if (it != g_tiles.end() && it->second.forced) return false;
    }
    int64_t n_max = 0;
    double pairs = 0.0;
    for (int32_t k = 0; k < ns; ++k) {
        const int64_t nk = offs[k + 1] - offs[k];
        n_max = std::max(n_max, nk);
        pairs += (double)nk * (double)nk;
    }
    const int64_t n = offs[ns];
    if (n_max > kGroupBatchMax || pairs > kGroupBatchPairs ||
        pairs >= (double)kBatchMutualMin * (double)n)
        return false;
    // targets per workgroup: as many as leave every CU a few workgroups; four
    // waves each, so that one workgroup's exchange hides behind the others' pairs
    int per_cu = 2;
    if (n <= 1024) *shape = {1, 4, 512};
    else if (n <= 4096) *shape = {2, 4, 512};
    else if (n <= 12288) *shape = {2, 8, 256}, per_cu = 4;
    else if (n_max <= 640) *shape = {2, 16, 256}, per_cu = 4;
    else *shape = {4, 8, 256};
    const size_t lds = group_lds_bytes(n_max, *shape) + 512;
    per_cu = (int)std::min<size_t>(per_cu, ((size_t)160 << 10) / lds);
    *slots = 256 * std::max(per_cu, 1);
    return pairs <= kGroupBatchAlways ||
           !group_shares_lose(group_shares(offs, ns, shape->tpl * shape->lanes, *slots), pairs);
}

// The group kernel's work list: a system's workgroups go to one XCD (workgroups
// go to the XCDs in turn), whose L2 then carries its exchange.  Only workgroups
// of the same system wait for each other: systems of one workgroup take turns in
// a slot, so many small ones leave the others theirs (us per step, one system of
// 2,000 bodies and 2,000 of 5: 12, by launches 108; 1,012 where each of the small
// ones had a slot and the large one a single workgroup).
std::shared_ptr<BatchPlan> batch_group_plan(const int64_t* offs, int32_t ns, const GroupShape& g,
                                            int slots)
{
    std::vector<int64_t> key(offs, offs + ns + 1);
    for (int64_t x : {-2, g.tpl, g.lanes, g.threads, slots}) key.push_back(x);
    std::lock_guard<std::mutex> lk(g_mu);
    g_batch_used[key] = ++g_batch_tick;
    auto it = g_batch.find(key);
    if (it != g_batch.end()) return it->second;
    evict_batch_plan_locked();
    auto bp = std::make_shared<BatchPlan>();
    const GroupShares S = group_shares(offs, ns, (int64_t)g.tpl * g.lanes, slots);
    bp->n_max = S.n_max;
    auto size = [&](int32_t k) { return offs[k + 1] - offs[k]; };
    std::vector<int32_t> order(ns), place(kGroupBatchMax + 1);   // largest first, stable
    for (int64_t n = bp->n_max; n > 0; --n) place[n - 1] = place[n] + S.count[n];
    for (int32_t k = 0; k < ns; ++k) order[place[size(k)]++] = k;
    // one list per XCD; a system that no list has room for is spread over all
    constexpr int kXcds = 8;
    std::vector<GroupUnit> lists[kXcds];
    size_t length[kXcds] = {};
    auto shortest = [&] {
        int m = 0;
        for (int l = 1; l < kXcds; ++l)
            if (length[l] < length[m]) m = l;
        return m;
    };
    for (int32_t k : order) {
        const int32_t nk = (int32_t)size(k), w = S.wgs[nk];
        const int l = shortest();
        const bool whole = (int64_t)length[l] + w <= slots / kXcds;
        for (int32_t r = 0; r < w; ++r) {
            const int m = whole || r == 0 ? l : shortest();
            lists[m].push_back(GroupUnit{offs[k], nk, k, w, r});
            ++length[m];
        }
    }
    // in turn, short lists padded (n = 0); unpadded, and so without regard to
    // XCDs, where the padding would outgrow the workspace's room for units
    const size_t len = *std::max_element(length, length + kXcds);
    const bool pad = (int64_t)(kXcds * len) <= offs[ns] / 4 + ns;
    bp->group_units.reserve(kXcds * len);
    for (size_t i = 0; i < len; ++i)
        for (const auto& l : lists)
            if (i < l.size()) bp->group_units.push_back(l[i]);
            else if (pad) bp->group_units.push_back(GroupUnit{0, 0, 0, 1, 0});
    g_batch[key] = bp;
    return bp;
}

// ---------------------------------------------------------------------------
// a share of the targets (one GPU's force pass when the targets are split)

// The one-way tile of the full pass over n bodies, with its source chunks
// chosen for the share's target blocks: about 8192 / waves units, as the
// full pass has, capped by the chunk limit and at 64 * waves sources each.
Tile shard_tile(int64_t n, int64_t t0, int64_t nt)
{
    Tile t = force_only_tile(NBODY_FP64, n);
    const int64_t tpb = targets_per_block(t);
    const int64_t tb = (t0 + nt - 1) / tpb - t0 / tpb + 1;
    int64_t c = std::max<int64_t>(1, 8192 / (tb * t.waves));
    c = std::min<int64_t>(c, std::max<int64_t>(1, n / (64 * t.waves)));
    t.chunks = (int)std::min<int64_t>(c, kMaxChunks);
    return t;
}

// Work list of a share: the target blocks holding t0 .. t0 + nt - 1 times the
// tile's chunks (a single system at body 0), cached with the ensembles' lists.
std::shared_ptr<BatchPlan> shard_plan(int64_t n, int64_t t0, int64_t nt, const Tile& t)
{
    std::vector<int64_t> key = {-1, n, t0, nt, t.tpl, t.waves, t.chunks, t.variant};
    std::lock_guard<std::mutex> lk(g_mu);
    g_batch_used[key] = ++g_batch_tick;
    auto it = g_batch.find(key);
    if (it != g_batch.end()) return it->second;
    evict_batch_plan_locked();
    auto bp = std::make_shared<BatchPlan>();
    const int64_t tpb = targets_per_block(t);
    const int eff = effective_chunks(n, t);
    for (int64_t b = t0 / tpb; b <= (t0 + nt - 1) / tpb; ++b)
        for (int c = 0; c < eff; ++c) {
            BatchUnit u;
            u.body0 = 0;
            u.n = (int32_t)n;
            u.sys = 0;
            u.tblock = (int32_t)b;
            u.chunk = c;
            u.chunks = t.chunks;
            u.pad = 0;
            bp->units.push_back(u);
        }
    g_batch[key] = bp;
    return bp;
}

}  // namespace

extern "C" {

int32_t nbody_accel_shard(const double* pos, const double* mass, int64_t n, double G, int64_t t0,
                          int64_t nt, double* acc_out, void* workspace, size_t workspace_bytes,
                          void* stream)
{
    g_err.clear();
    NB_TRY(check_common(pos, mass, n, G));
    if (!acc_out) return fail(NBODY_EINVAL, "acc_out is NULL");
    if (t0 < 0 || nt < 1 || t0 > n - nt)
        return fail(NBODY_EINVAL, "targets [%lld, %lld) are not a non-empty part of [0, %lld)",
                    (long long)t0, (long long)(t0 + nt), (long long)n);
    const Layout L = layout(NBODY_OP_ACCEL_SHARD, n, 1, 0, 1, NBODY_FP64);
    NB_TRY(check_ws(workspace, workspace_bytes, L.total));
    hipStream_t s = static_cast<hipStream_t>(stream);
    const Tile t = shard_tile(n, t0, nt);
    auto bp = shard_plan(n, t0, nt, t);
    const int64_t nu = (int64_t)bp->units.size();
    if ((size_t)nu * sizeof(BatchUnit) > L.total - L.units)   // (the layout's bound covers it)
        return fail(NBODY_EUNSUPPORTED, "work list exceeds the workspace");
    BatchUnit* units = at<BatchUnit>(workspace, L.units);
    double* part = at<double>(workspace, L.part);
    double* gm = at<double>(workspace, L.gm);
    NB_HIP(hipMemcpyAsync(units, bp->units.data(), nu * sizeof(BatchUnit), hipMemcpyHostToDevice,
                          s));
    NB_HIP(launch_scale(mass, G, n, gm, s));
    int cus = 0;
    NB_TRY(device_cus(&cus));
    const int grid = (int)std::min<int64_t>(nu, (int64_t)cus * (16 / t.waves));
    NB_HIP(launch_force_batched(NBODY_FP64, t, pos, mass, gm, n, G, units, nu, nullptr, grid, part,
                                s));
    NB_HIP(launch_shard_sum(part, effective_chunks(n, t), n, t0, nt, acc_out, s));
    return NBODY_OK;
}

int32_t nbody_verlet_run_batched(double* pos, double* vel, const double* mass,
                                 const int64_t* offsets_host, int32_t num_systems, double G,
                                 double dt, int64_t steps, int32_t precision, double small_mass,
                                 void* workspace, size_t workspace_bytes, void* stream)
{
    g_err.clear();
    NB_TRY(check_offsets(offsets_host, num_systems));
    const int64_t n = offsets_host[num_systems];
    NB_TRY(check_common(pos, mass, n, G));
    NB_TRY(check_prec(precision, small_mass));
    if (!vel) return fail(NBODY_EINVAL, "vel is NULL");
    if (steps < 0) return fail(NBODY_EINVAL, "steps must be >= 0");
    if (!std::isfinite(dt)) return fail(NBODY_EINVAL, "dt is not finite");
    const Layout L = layout(NBODY_OP_BATCHED, n, num_systems, steps, 1, precision);
    NB_TRY(check_ws(workspace, workspace_bytes, L.total));
    if (steps == 0) return NBODY_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);

    StepPlan P;
    P.prec = precision;
    P.chunks = 0;
    P.n = n;
    P.G = G;
    P.dt = dt;
    P.part = at<double>(workspace, L.part);
    P.flags = at<uint32_t>(workspace, L.flags);
    GroupShape gshape;
    int gslots = 0;
    if (batch_group_route(precision, offsets_host, num_systems, &gshape, &gslots)) {
        GroupArgs A{};
        A.pos_in = pos;
        A.pos_out = pos;
        A.vel = vel;
        A.mass = mass;
        if (precision != NBODY_FP64) {
            NB_TRY(batched_split_prepare(pos, vel, mass, offsets_host, num_systems, G, small_mass,
                                         workspace, L, s, &P));
            A.pos_in = P.buf[0];
            A.pos_out = P.buf[0];
            A.vel = P.vel;
            A.mass = P.mass;
            A.nmaj = P.nmaj;
        }
        auto bp = batch_group_plan(offsets_host, num_systems, gshape, gslots);
        GroupUnit* units = at<GroupUnit>(workspace, L.units);
        // (the layout's bound covers it: at most n / 4 + ns units)
        if (bp->group_units.size() * sizeof(GroupUnit) > L.bchunks - L.units)
            return fail(NBODY_EUNSUPPORTED, "ensemble work list exceeds the workspace");
        NB_HIP(hipMemcpyAsync(units, bp->group_units.data(),
                              bp->group_units.size() * sizeof(GroupUnit), hipMemcpyHostToDevice,
                              s));
        A.units = units;
        A.xbuf = P.part;
        A.reg = reinterpret_cast<uint32_t*>(P.part + 12 * n);
        A.flags = P.flags;
        A.n = n;
        A.stride = n;
        A.G = G;
        A.dt = dt;
        A.steps = steps;
        A.spread = 1;
        NB_TRY(group_launches(precision, gshape, A, (int)bp->group_units.size(), bp->n_max,
                              num_systems, steps, s));
        if (precision != NBODY_FP64) {
            const int32_t* perm = at<int32_t>(workspace, L.perm);
            NB_HIP(launch_scatter(perm, n, P.buf[0], pos, P.vel, vel, s));
        }
        return NBODY_OK;
    }
    NB_TRY(batched_plan_upload(offsets_host, num_systems,
                               batch_tile(precision, offsets_host, num_systems), workspace, L, s,
                               &P));
    if (precision == NBODY_FP64) {
        double* alt = at<double>(workspace, L.alt);
        double* gm = at<double>(workspace, L.gm);
        P.mass = mass;
        P.gm = gm;
        P.vel = vel;
        NB_HIP(launch_scale(mass, G, n, gm, s));
        // fixed buffer roles (see verlet_run_on); an odd run is copied back
        P.buf[0] = pos;
        P.buf[1] = alt;
        NB_TRY(run_steps(P, steps, s, true));
        if (steps & 1) NB_HIP(launch_scale(alt, 1.0, 3 * n, pos, s));
        return NBODY_OK;
    }
    NB_TRY(batched_split_prepare(pos, vel, mass, offsets_host, num_systems, G, small_mass,
                                 workspace, L, s, &P));
    const int32_t* perm = at<int32_t>(workspace, L.perm);
    NB_TRY(run_steps(P, steps, s, true));
    NB_HIP(launch_scatter(perm, n, P.buf[steps & 1], pos, P.vel, vel, s));
    return NBODY_OK;
}

int32_t nbody_autotune_batched(int32_t precision, const double* pos, const double* mass,
                               const int64_t* offsets_host, int32_t num_systems, double G,
                               double small_mass, void* workspace, size_t workspace_bytes,
                               void* stream, nbody_tile* best_host, double* best_ms_host)
{
    g_err.clear();
    NB_TRY(check_offsets(offsets_host, num_systems));
    const int64_t n = offsets_host[num_systems];
    NB_TRY(check_common(pos, mass, n, G));
    NB_TRY(check_prec(precision, small_mass));
    const Layout L = layout(NBODY_OP_BATCHED, n, num_systems, 1, 1, precision);
    NB_TRY(check_ws(workspace, workspace_bytes, L.total));
    hipStream_t s = static_cast<hipStream_t>(stream);
    StepPlan P;
    P.prec = precision;
    P.n = n;
    P.G = G;
    P.part = at<double>(workspace, L.part);
    const double* pos_w = pos;
    if (precision == NBODY_FP64) {
        double* gm = at<double>(workspace, L.gm);
        P.mass = mass;
        P.gm = gm;
        NB_HIP(launch_scale(mass, G, n, gm, s));
    } else {
        NB_TRY(batched_split_prepare(pos, nullptr, mass, offsets_host, num_systems, G, small_mass,
                                     workspace, L, s, &P));
        pos_w = P.buf[0];
    }
    std::vector<Tile> cands;
    if (precision != NBODY_SPLIT_COMPENSATED)   // (that form runs each pair once only)
        for (int tpl : {1, 2, 4})
            for (int w : {1, 2, 4})
                for (int v = 0; v < 3; ++v) cands.push_back(Tile{tpl, w, kBatchChunkMax, v});
    bool fits = true;   // each pair once, if every system's ranges fit the slots
    for (int32_t k = 0; k < num_systems; ++k)
        fits = fits && mutual_ranges(offsets_host[k + 1] - offsets_host[k]) <= kBatchSlots;
    if (fits)
        for (const Tile& t : {Tile{2, 4, 1, 5}, Tile{4, 4, 1, 5}}) cands.push_back(t);
    if (cands.empty())
        return fail(NBODY_EUNSUPPORTED, "the compensated split form runs in the each-pair-once "
                                        "pass, which takes ensembles of systems of at most "
                                        "%d bodies", 256 * kBatchSlots);
    double* acc_w = at<double>(workspace, L.alt);
    // a candidate is timed as force pass and epilogue (the partial counts differ)
    auto pass = [&]() -> int {
        NB_TRY(force(P, pos_w, s));
        NB_HIP(launch_step(P.part, 0, P.bchunks, n, nullptr, nullptr, nullptr, acc_w, 0.0,
                           kStoreAcc, nullptr, s));
        return NBODY_OK;
    };
    hipEvent_t e0 = nullptr, e1 = nullptr;
    NB_HIP(hipEventCreate(&e0));
    NB_HIP(hipEventCreate(&e1));
    // two passes over the candidates, each keeping its faster time (the first
    // pass also brings the shader clock up from idle)
    Tile best = cands.front();
    float best_ms = 1e30f;
    int status = NBODY_OK;
    for (int round = 0; round < 2 && status == NBODY_OK; ++round)
    for (const Tile& t : cands) {
        if ((status = batched_plan_upload(offsets_host, num_systems, t, workspace, L, s, &P)) != NBODY_OK)
            break;
        const int reps = 3;
        if ((status = pass()) != NBODY_OK) break;
        if (hipEventRecord(e0, s) != hipSuccess) { status = fail(NBODY_EHIP, "event record"); break; }
        for (int r = 0; r < reps && status == NBODY_OK; ++r) status = pass();
        if (status != NBODY_OK) break;
        if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess) {
            status = fail(NBODY_EHIP, "event sync");
            break;
        }
        float ms = 0.f;
        (void)hipEventElapsedTime(&ms, e0, e1);
        ms /= reps;
        if (ms < best_ms) {
            best_ms = ms;
            best = t;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (status != NBODY_OK) return status;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        g_tiles[std::make_tuple(2, (int)precision, size_class(0))] = TunedTile{best, false};
    }
    if (best_host) {
        best_host->targets_per_lane = best.tpl;
        best_host->waves = best.waves;
        best_host->chunks = best.chunks;
        best_host->variant = best.variant;
    }
    if (best_ms_host) *best_ms_host = best_ms;
    return NBODY_OK;
}

}  // extern "C"

namespace {

// Working data of a timed force pass (class order for the split form).
struct Bench {
    const double* pos = nullptr;
    const double* mass = nullptr;
    const double* gm = nullptr;
    const int64_t* nmaj = nullptr;
    double* part = nullptr;
    double* scratch = nullptr;
};

int bench_prepare(int32_t kind, int32_t precision, const double* pos, const double* mass,
                  int64_t n, double G, double small_mass, void* workspace,
                  size_t workspace_bytes, hipStream_t s, Bench* b)
{
    NB_TRY(check_common(pos, mass, n, G));
    NB_TRY(check_prec(precision, small_mass));
    NB_TRY(check_comp_size(precision, n));
    if (kind != 0 && kind != 1) return fail(NBODY_EINVAL, "kind must be 0 or 1");
    if (kind == 1 && precision != NBODY_FP64) return fail(NBODY_EINVAL, "the adjoint pass is FP64");
    const int op = kind == 0 ? NBODY_OP_ACCEL : NBODY_OP_ADJOINT;
    const Layout L = layout(op, n, 1, 1, 1, precision);
    NB_TRY(check_ws(workspace, workspace_bytes, L.total));
    b->part = at<double>(workspace, L.part);
    b->scratch = at<double>(workspace, L.alt);
    b->pos = pos;
    b->mass = mass;
    if (precision != NBODY_FP64) {
        ClassOrdered c;
        NB_TRY(split_prepare(workspace, L, pos, nullptr, mass, n, G, small_mass, s, &c));
        b->pos = c.pos;
        b->mass = c.mass;
        b->nmaj = c.nmaj;
    }
    if (kind == 1) NB_HIP(launch_fill(b->scratch, 1e-3, 3 * n, s));   // cotangent for timing
    double* gm = at<double>(workspace, L.gm);
    NB_HIP(launch_scale(b->mass, G, n, gm, s));
    b->gm = gm;
    return NBODY_OK;
}

}  // namespace

extern "C" {

int32_t nbody_time_force(int32_t kind, int32_t precision, const double* pos, const double* mass,
                         int64_t n, double G, double small_mass, int32_t reps, void* workspace,
                         size_t workspace_bytes, void* stream, double* ms_per_pass_host)
{
    g_err.clear();
    if (reps < 1 || !ms_per_pass_host) return fail(NBODY_EINVAL, "reps < 1 or null output");
    hipStream_t s = static_cast<hipStream_t>(stream);
    Bench b;
    NB_TRY(bench_prepare(kind, precision, pos, mass, n, G, small_mass, workspace, workspace_bytes,
                         s, &b));
    const Tile t = pick_tile(kind, precision, n);
    auto once = [&]() -> int {
        if (kind == 0 && t.variant == 3)
            NB_HIP(launch_run_small(precision, t, b.pos, nullptr, nullptr, b.mass, n, b.nmaj, G, 0.0,
                                    0, 0, 0, b.scratch, nullptr, nullptr, s));
        else if (kind == 0 && t.variant == 4)
            NB_HIP(launch_step_fused(precision, t, b.pos, nullptr, nullptr, b.gm, n, b.nmaj, 0.0,
                                     kStoreAcc, b.scratch, nullptr, s));
        else if (kind == 0)
            NB_HIP(launch_force(precision, t, b.pos, b.mass, b.gm, n, b.nmaj, G, b.part, s));
        else           NB_HIP(launch_vjp(t, b.pos, b.mass, b.scratch, 1.0, n, G, b.part, s));
        return NBODY_OK;
    };
    NB_TRY(once());
    hipEvent_t e0 = nullptr, e1 = nullptr;
    NB_HIP(hipEventCreate(&e0));
    NB_HIP(hipEventCreate(&e1));
    int st = NBODY_OK;
    if (hipEventRecord(e0, s) != hipSuccess) st = fail(NBODY_EHIP, "hipEventRecord failed");
    for (int r = 0; r < reps && st == NBODY_OK; ++r) st = once();
    if (st == NBODY_OK && (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess))
        st = fail(NBODY_EHIP, "event timing failed");
    float ms = 0.f;
    if (st == NBODY_OK) (void)hipEventElapsedTime(&ms, e0, e1);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (st != NBODY_OK) return st;
    *ms_per_pass_host = (double)ms / reps;
    return NBODY_OK;
}

int32_t nbody_autotune(int32_t kind, int32_t precision, const double* pos, const double* mass,
                       int64_t n, double G, double small_mass, void* workspace,
                       size_t workspace_bytes, void* stream, nbody_tile* best_host,
                       double* best_ms_host)
{
    g_err.clear();
    hipStream_t s = static_cast<hipStream_t>(stream);
    Bench b;
    NB_TRY(bench_prepare(kind, precision, pos, mass, n, G, small_mass, workspace, workspace_bytes,
                         s, &b));
    double* part = b.part;
    double* scratch = b.scratch;
    const double* pos_w = b.pos;
    const double* mass_w = b.mass;
    const int64_t* nmaj = b.nmaj;

    // candidates
    std::vector<Tile> cands;
    const int tpls[3] = {1, 2, 4};
    const int waves[4] = {1, 2, 4, 8};
    for (int it = 0; it < 3; ++it)
        for (int iw = 0; iw < 4; ++iw) {
            for (int variant = 0; variant < (kind == 0 ? 3 : 2); ++variant) {
                Tile t{tpls[it], waves[iw], 1, variant};
                if (kind == 1 && (t.tpl > 2 || t.waves > 4)) continue;
                if (variant != 0 && t.tpl == 4 && t.waves == 8) continue;   // register spills
                const int64_t tpb = targets_per_block(t);
                const int64_t tb = (n + tpb - 1) / tpb;
                std::vector<int> cs = {1};
                for (int64_t target : {512, 1024, 2048, 3072, 4096, 6144, 8192}) {
                    const int64_t waves_per_chunk = tb * t.waves;
                    int64_t c = target / std::max<int64_t>(waves_per_chunk, 1);
                    c = std::min<int64_t>(c, chunk_cap(n));
                    c = std::min<int64_t>(c, std::max<int64_t>(1, n / (64 * t.waves)));
                    if (c >= 1) cs.push_back((int)c);
                }
                std::sort(cs.begin(), cs.end());
                cs.erase(std::unique(cs.begin(), cs.end()), cs.end());
                for (int c : cs) cands.push_back(Tile{t.tpl, t.waves, c, variant});
            }
        }

    if (precision == NBODY_SPLIT_COMPENSATED) cands.clear();   // each pair once only
    if (mutual_fits(kind, precision, n))   // each pair once
        for (const Tile& t : {Tile{1, 4, 1, 5}, Tile{2, 2, 1, 5}, Tile{2, 4, 1, 5}, Tile{4, 4, 1, 5}})
            cands.push_back(t);
    if (kind == 0 && n <= kFusedMax && precision != NBODY_SPLIT_COMPENSATED) {
        // force pass and step in one kernel, waves of a group splitting the sources
        for (int tpl : {1, 2})
            for (int w : {2, 4, 8}) cands.push_back(Tile{tpl, w, 1, 4});
    }
    if (kind == 0 && n <= kSmallMax && precision != NBODY_SPLIT_COMPENSATED) {
        // single workgroup: force pass, reduction and store in one launch
        for (int S : {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 16, 24, 32, 48, 64}) {
            const Tile t{1, 16, S, 3};
            if (small_slices(n, t) == S) cands.push_back(t);
        }
    }

    hipEvent_t e0 = nullptr, e1 = nullptr;
    NB_HIP(hipEventCreate(&e0));
    NB_HIP(hipEventCreate(&e1));
    // The single-workgroup variant is timed as it runs: kSmallPasses launch
    // indices (force pass, reduction, kicks and drift, with dt = 0 so the
    // state stays put) in one launch, on a copy of the state in `part`.
    constexpr int kSmallPasses = 16;
    double* r_small = part;
    double* v_small = part + 3 * n;
    auto once = [&](const Tile& t) -> int {
        if (kind == 0 && t.variant == 3) {
            NB_HIP(launch_run_small(precision, t, r_small, r_small, v_small, mass_w, n, nmaj, G,
                                    0.0, 0, kSmallPasses - 1, kSmallPasses, nullptr, nullptr,
                                    nullptr, s));
        } else if (kind == 0 && t.variant == 4) {
            NB_HIP(launch_step_fused(precision, t, pos_w, nullptr, nullptr, b.gm, n, nmaj, 0.0,
                                     kStoreAcc, scratch, nullptr, s));
        } else if (kind == 0) {
            NB_HIP(launch_force(precision, t, pos_w, mass_w, b.gm, n, nmaj, G, part, s));
            NB_HIP(launch_step(part, force_slots(precision, n, t), nullptr, n, nullptr, nullptr,
                               nullptr, scratch, 0.0, kStoreAcc, nullptr, s));
        } else {
            NB_HIP(launch_vjp(t, pos_w, mass_w, scratch, 1.0, n, G, part, s));
        }
        return NBODY_OK;
    };
    // repetitions so that each measurement covers at least ~2 ms of work
    const double pairs = (double)n * (double)n;
    const int reps = (int)std::max(3.0, std::min(200.0, 2e9 / std::max(pairs, 1.0)));
    // Two passes over the candidates, each keeping its faster time: the first
    // pass also brings the shader clock up from idle (it climbs over the first
    // tens of milliseconds of load), which would otherwise favour the
    // candidates timed last.
    Tile best = cands.front();
    float best_ms = 1e30f;
    int status = NBODY_OK;
    for (int pass = 0; pass < 2 && status == NBODY_OK; ++pass)
    for (const Tile& t : cands) {
        if (t.variant == 3 &&
            (hipMemcpyAsync(r_small, pos_w, 3 * n * sizeof(double), hipMemcpyDeviceToDevice, s) !=
                 hipSuccess ||
             launch_fill(v_small, 0.0, 3 * n, s) != hipSuccess)) {
            status = fail(NBODY_EHIP, "copying the state for the single-workgroup variant failed");
            break;
        }
        if ((status = once(t)) != NBODY_OK) break;
        if (hipEventRecord(e0, s) != hipSuccess) { status = fail(NBODY_EHIP, "event record"); break; }
        for (int r = 0; r < reps && status == NBODY_OK; ++r) status = once(t);
        if (status != NBODY_OK) break;
        if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess) {
            status = fail(NBODY_EHIP, "event sync");
            break;
        }
        float ms = 0;
        (void)hipEventElapsedTime(&ms, e0, e1);
        ms /= reps;
        if (t.variant == 3) ms /= kSmallPasses;
        if (ms < best_ms) {
            best_ms = ms;
            best = t;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (status != NBODY_OK) return status;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        g_tiles[std::make_tuple(kind, precision, size_class(n))] = TunedTile{best, false};
    }
    if (best_host) {
        best_host->targets_per_lane = best.tpl;
        best_host->waves = best.waves;
        best_host->chunks = best.chunks;
        best_host->variant = best.variant;
    }
    if (best_ms_host) *best_ms_host = best_ms;
    return NBODY_OK;
}

}  // extern "C"
