// Whole runs of the kick-drift-kick loop of Eqs. (3)-(4) in one launch, for
// systems too large for one workgroup and too small to fill the chip
// (80 to 4,095 bodies), and for ensembles of such systems.
//
// Below a few thousand bodies a force pass is a microsecond or two of
// arithmetic; a step made of a force kernel and an epilogue is bound by two
// kernel boundaries and the latency of the partials' round trip (about 10 us
// from 500 to 2,100 bodies).  Here the workgroups of one launch stay on the
// chip for all steps.  A workgroup keeps all n sources in LDS and owns a few
// targets ("virtual group" v: targets v * Tw .. v * Tw + Tw - 1); after each
// step it publishes its targets' new positions and picks up everybody
// else's.
//
// The exchange has no barrier and no fence.  Positions are published by
// relaxed agent-scope atomic stores (8 bytes each, written through to where
// every XCD sees them) into one of three exchange buffers; each word of a
// buffer holds a sentinel until its value arrives, so a reader polls the
// data itself: one trip through memory per step where a flag and the data
// behind it would take two, and no cache write-back.  The sentinel is a
// signalling NaN, which arithmetic never produces (and publish() keeps
// out).  Buffer b holds r_i for i = b mod 3.  At launch index i a workgroup
// that has read all of r_i knows that everybody has finished reading
// r_{i-1}, so it resets its own words of that buffer to the sentinel, and it
// waits for those stores before it publishes r_{i+1}: whoever sees r_{i+1}
// complete finds the buffer of r_{i+2} reset.
//
// No workgroup waits for one that may not be on the chip.  The workgroups of
// a system register at entry; the first to arrive starts the run when all have
// come, or after kRegisterTicks (other work may hold part of the chip), and
// those that registered share the virtual groups among themselves.  A workgroup
// that comes later joins at the next even launch index: the exchange buffers
// hold all it needs but the state that only owners keep (velocities; gradients
// in the sweep), which while workgroups are missing is stored past the caches
// ahead of the position, and read behind an acquire.  So every wait is on a
// workgroup that is resident, a run that began on a corner of the chip has all
// of it soon after other work ends, and results do not depend on how many
// share the work: a virtual group's arithmetic is the same whoever runs it.
// (Two runs at once, 1,000 bodies and 1,000 steps each: 7.8 ms, one alone 3.4,
// and 82 where late workgroups left for the rest of the launch; 4,000 bodies, 500
// steps: 17, 7.7 and 243.  Eight at once, us per step of all: 27 at 1,000 bodies,
// 40 by launches; 42 and 47 at 2,000; 89 and 68 at 3,000, where one workgroup fills
// a CU's LDS and the runs take turns.)
//
// The pair arithmetic and the two forms are those of the multi-kernel passes:
// FP64, or (SPLIT, class order) heavy sources with one Newton step and light
// ones in FP32, summed in blocks of at most 16 that are added in FP64.
#include <atomic>
#include <type_traits>

#include "common.hpp"
#include "pair_math.hpp"

namespace nb {
namespace {

using namespace pm;

constexpr uint64_t kSentinel = 0xFFF4B0D1E5A11CEDull;   // a signalling NaN
constexpr uint64_t kRunEnded = ~(uint64_t)0;
#ifndef NB_GROUP_REGISTER_TICKS   // (a test instrument sets it, and what follows)
#define NB_GROUP_REGISTER_TICKS 200000
#define NB_GROUP_ENTRY(reg)
#endif
// How long the first workgroup waits for the others, in ticks of the 100 MHz
// counter: 0.2 ms, if fewer than a quarter of them have come then 2 ms (a run on
// a corner of the chip would hold up those that come when it is freed).
constexpr uint64_t kRegisterTicks = NB_GROUP_REGISTER_TICKS;
constexpr uint64_t kEnoughTicks = kRegisterTicks / 10;
constexpr int kPollBudget = 1 << 26;          // polls of a thread, a last resort
constexpr int kMaxLds = 160 * 1024 - 256;     // beside the kernel's static LDS
constexpr int kBlkG = 16;                     // FP32 block length of the light sums

// A store past the caches that other XCDs' loads do not reach.
__device__ __forceinline__ void agent_store(double* p, double v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Two words at word `off` of `base`, with the cache policy of an agent-scope
// load (sc1: past the caches that other XCDs' stores do not reach).
__device__ __forceinline__ double2 poll_load2(const double* base, int off)
{
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<double*>(base), 0, 0x7FFFFFFF, 0x00020000);
    const u4 v = __builtin_amdgcn_raw_buffer_load_b128(r, 8 * off, 0, 16);
    double2 d;
    d.x = __builtin_bit_cast(double, ((uint64_t)v.y << 32) | v.x);
    d.y = __builtin_bit_cast(double, ((uint64_t)v.w << 32) | v.z);
    return d;
}

__device__ __forceinline__ void publish(double* p, double v)
{
    if (__builtin_bit_cast(uint64_t, v) == kSentinel) v = __builtin_nan("");
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ bool pending(double v)
{
    return __builtin_bit_cast(uint64_t, v) == kSentinel;
}

// Rotation within each row of 16 lanes by N lanes (DPP row_ror).
template <int N>
__device__ __forceinline__ double row_ror(double x)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)u, 0x120 + N, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), 0x120 + N, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// Sum over the slices of a row: lanes t, t + TT, ... of its first TT * (16 / TT),
// complete in the lanes t < TT (in all lanes where TT divides 16).
template <int TT>
__device__ __forceinline__ double row_sum(double x)
{
    static_assert(16 % TT == 0 || TT == 3 || TT == 5, "lanes side by side");
    if (TT == 5) return x + row_ror<16 - 5>(x) + row_ror<16 - 10>(x);
    if (TT == 3) {
        const double y = x + row_ror<16 - 6>(x);
        return y + row_ror<16 - 3>(y) + row_ror<16 - 12>(x);
    }
    if (TT <= 8) x += row_ror<8>(x);
    if (TT <= 4) x += row_ror<4>(x);
    if (TT <= 2) x += row_ror<2>(x);
    if (TT <= 1) x += row_ror<1>(x);
    return x;
}

__device__ __forceinline__ float light_gm(double slot)
{
    return __builtin_bit_cast(float, (uint32_t)__builtin_bit_cast(uint64_t, slot));
}

// A workgroup's place among the `planned` ones of its system.  reg: how many have
// come, how many the run began with, and a word of 64 bits that says how many
// share the work and from which launch index on (counted from the launch's first).
struct Crew {
    int rank, present;
    int first;     // the launch index this workgroup begins at
    int moving;    // the run began without all of them: state changes hands
};

__device__ __forceinline__ uint64_t* crew_word(uint32_t* reg)
{
    return reinterpret_cast<uint64_t*>(reg + 2);
}

__device__ __forceinline__ uint64_t load_word(const uint64_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Registers the workgroup.  False: it came too late and must leave.  Every wait
// here is on the first workgroup, which is on the chip, starts the run in bounded
// time and, while some are missing, says every second launch index how many
// share the work from the next on, and at last that the run has ended.  A
// workgroup that it counts in finds that index here in time: it cannot be
// overtaken, as the others wait for its positions.
__device__ __forceinline__ bool register_workgroup(uint32_t* reg, int planned, Crew& crew)
{
    __shared__ uint32_t s_crew[3];
    NB_GROUP_ENTRY(reg)
    if (threadIdx.x == 0) {
        const uint32_t r = __hip_atomic_fetch_add(&reg[0], 1u, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
        uint64_t word = 0;
        if (r == 0) {   // the first: start the run
            const uint64_t t0 = wall_clock64();
            uint32_t count;
            for (;;) {
                count = __hip_atomic_load(&reg[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const uint64_t t = wall_clock64() - t0;
                if (count >= (uint32_t)planned || t >= kRegisterTicks ||
                    (t >= kEnoughTicks && 4 * count >= (uint32_t)planned))
                    break;
            }
            word = count;
            reg[1] = count;
            __hip_atomic_store(crew_word(reg), word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            while ((uint32_t)(word = load_word(crew_word(reg))) <= r) {
            }
        }
        s_crew[0] = r;
        s_crew[1] = (uint32_t)word;
        s_crew[2] = (uint32_t)(word >> 32);
    }
    __syncthreads();
    crew.rank = __builtin_amdgcn_readfirstlane((int)s_crew[0]);
    crew.present = __builtin_amdgcn_readfirstlane((int)s_crew[1]);
    crew.first = __builtin_amdgcn_readfirstlane((int)s_crew[2]);
    crew.moving =
        __builtin_amdgcn_readfirstlane(crew.first > 0 || crew.present < planned ? 1 : 0);
    return crew.present != (int)(uint32_t)kRunEnded;
}

// At launch index k of 0 .. last, ahead of its work and with all of r_k read,
// while workgroups are missing: at even indices, how many share the work from
// here on; at odd ones the first workgroup announces that for the next, and the
// announcement arrives before its positions do.  (None for the last index, whose
// positions nobody waits for.)
__device__ __forceinline__ void share_work(uint32_t* reg, Crew& crew, int planned, int k, int last)
{
    if (crew.present >= planned && k != crew.first) return;
    if (k > 0 && (k & 1) == 0 && k < last) {
        // (every wave reads the same word: the next is written after this index)
        const int now =
            __builtin_amdgcn_readfirstlane((int)(uint32_t)load_word(crew_word(reg)));
        // where work changes hands, state that others stored is read from here on
        if (now != crew.present || k == crew.first)
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        crew.present = now;
    }
    if (crew.rank == 0 && (k & 1) == 1 && k + 1 < last && threadIdx.x == 0) {
        const uint64_t count =
            __hip_atomic_load(&reg[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(crew_word(reg), (uint64_t)(k + 1) << 32 | count, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
}

// After the last index: those that were never counted in need not wait longer.
__device__ __forceinline__ void end_run(uint32_t* reg, const Crew& crew, int planned)
{
    if (crew.rank == 0 && crew.present < planned && threadIdx.x == 0)
        __hip_atomic_store(crew_word(reg), kRunEnded, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// x + y with x rounded first (no fused multiply-add).
__device__ __forceinline__ double add_rounded(double x, double y)
{
#pragma clang fp contract(off)
    return x + y;
}

// What a finishing lane knows of its word of a virtual group: component (3:
// G m, which travels along unchanged) of body ep of the system.
struct Word {
    bool mine;
    int comp, ep;
    int64_t e;      // of the system's planes
    double* slot;   // in exchange buffer 0; buffers are `words` apart
};

// Where a launch index k of 0 .. last (the run's index i0 + k) stands: which thirds
// of the exchange hold r_k, r_{k-1} and r_{k+1}, and whether the step from r_{k-1}
// closes there and the one to r_{k+1} opens.  (32 bits and launch-relative: the
// scalar unit compares no signed 64-bit numbers.)
struct Index {
    int k, last, cur;   // cur: k mod 3
    bool closes, opens;
    __device__ __forceinline__ int before() const { return cur == 0 ? 2 : cur - 1; }
    __device__ __forceinline__ int after() const { return cur == 2 ? 0 : cur + 1; }
};

// Ahead of the sweep at index x: the word of r_{k-1} is reset; returns the
// velocity.
__device__ __forceinline__ double word_begin(const GroupArgs& A, const Word& w, int words,
                                             const Index& x)
{
    if (!w.mine) return 0.0;
    if (x.k > 1 && x.k < x.last)
        __hip_atomic_store(w.slot + x.before() * words, __builtin_bit_cast(double, kSentinel),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return (x.closes || x.opens) && w.comp < 3 ? A.vel[w.e] : 0.0;
}

// With the acceleration a: kicks and drift, r_{k+1} published.  r0: the word at
// r_k.  Returns whether all of it is finite.
__device__ __forceinline__ bool word_finish(const GroupArgs& A, const Word& w, int words,
                                            const Index& x, double a, double v, double r0,
                                            double hdt, bool moving)
{
    double r = r0;
    if (w.comp < 3) {
        // (rounded as the step epilogue rounds it)
        if (x.closes) v = __builtin_fma(hdt, a, v);
        if (x.opens) {
            v = add_rounded(hdt * a, v);
            r = __builtin_fma(A.dt, v, r0);
        }
    }
    if (x.k < x.last) {
        if (__builtin_expect(moving, 0) && w.comp < 3) agent_store(A.vel + w.e, v);
        // the reset above (and the velocity) has arrived before this word does
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        publish(w.slot + x.after() * words, r);
    }
    if (w.comp == 3) return true;
    if (A.acc) A.acc[A.acc_perm ? w.e - w.ep + A.acc_perm[w.ep] : w.e] = a;
    if (A.traj) A.traj[x.k * (3 * A.n) + w.e] = r;
    if (x.k == x.last && A.pos_out) A.pos_out[w.e] = r;
    if ((x.closes || x.opens) && !(moving && x.k < x.last)) A.vel[w.e] = v;
    return __builtin_isfinite(a) && __builtin_isfinite(r) && __builtin_isfinite(v);
}

// Word pairs x0, x0 + NT, ... (kB of them, below `pairs`) of the exchange buffer
// src to LDS.  All loads go out together; then, two at a time, they are
// repeated until their words have arrived.  (A 16-byte load is two words, each
// whole and each tested.)
template <int kB, int NT>
__device__ __forceinline__ void gather_words(const double* src, int x0, int pairs, double2* to,
                                             int& budget)
{
    double2 v[kB];
#pragma unroll
    for (int u = 0; u < kB; ++u) {
        v[u] = double2{0.0, 0.0};
        if (x0 + u * NT < pairs) v[u] = poll_load2(src, 2 * (x0 + u * NT));
    }
#pragma unroll
    for (int h = 0; h < kB; h += 2) {
        while ((pending(v[h].x) || pending(v[h].y) || pending(v[h + 1].x) ||
                pending(v[h + 1].y)) &&
               --budget > 0) {
            asm volatile("" ::: "memory");
#pragma unroll
            for (int u = h; u < h + 2; ++u)
                if (x0 + u * NT < pairs) v[u] = poll_load2(src, 2 * (x0 + u * NT));
        }
    }
#pragma unroll
    for (int u = 0; u < kB; ++u)
        if (x0 + u * NT < pairs) to[x0 + u * NT] = v[u];
}

// One source against the T targets of a lane, FP64 terms.
template <int T, bool MASK, bool NEWTON1>
__device__ __forceinline__ void pair64(double jx, double jy, double jz, double jg, int j,
                                       const double (&tx)[T], const double (&ty)[T],
                                       const double (&tz)[T], int p0, int TT, double (&ax)[T],
                                       double (&ay)[T], double (&az)[T], const PolyConst& c)
{
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const double dx = jx - tx[t];
        const double dy = jy - ty[t];
        const double dz = jz - tz[t];
        const double r2 = __builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx));
        double f = NEWTON1 ? gm_rinv3_newton1(r2, jg) : gm_rinv3_f64(r2, jg, c);
        if (MASK) f = (j == p0 + t * TT) ? 0.0 : f;
        ax[t] = __builtin_fma(f, dx, ax[t]);
        ay[t] = __builtin_fma(f, dy, ay[t]);
        az[t] = __builtin_fma(f, dz, az[t]);
    }
}

template <int T, bool MASK>
__device__ __forceinline__ void pair32(double jx, double jy, double jz, float gm, int j,
                                       const double (&tx)[T], const double (&ty)[T],
                                       const double (&tz)[T], int p0, int TT, float (&bx)[T],
                                       float (&by)[T], float (&bz)[T])
{
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const float dx = (float)(jx - tx[t]);
        const float dy = (float)(jy - ty[t]);
        const float dz = (float)(jz - tz[t]);
        const float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
        const float y = __builtin_amdgcn_rsqf(r2);
        float w = gm * (y * y * y);
        if (MASK) w = (j == p0 + t * TT) ? 0.f : w;
        bx[t] = __builtin_fmaf(w, dx, bx[t]);
        by[t] = __builtin_fmaf(w, dy, by[t]);
        bz[t] = __builtin_fmaf(w, dz, bz[t]);
    }
}

// The sources [j0, j1) of a class in an order that leaves the group's own
// targets [own0, own1) for the end: the bodies after them, wrapping to j0,
// then the targets.  Lane s of S takes every S-th of that order, so all
// rounds but the last one or two need no test for the self pair.  fast(j) and
// masked(j) are called with the source's index; flush() after every 16 rounds.
template <int S, int UNROLL, class Fast, class Masked, class Flush>
__device__ __forceinline__ void each_source(int j0, int j1, int s, int own0, int own1, Fast&& fast,
                                            Masked&& masked, Flush&& flush)
{
    const int len = j1 - j0;
    if (len <= 0) return;
    const int o0 = own0 > j0 ? own0 : j0;
    const int o1 = own1 < j1 ? own1 : j1;
    const int own = o1 > o0 ? o1 - o0 : 0;
    const int full = (len - own) / S;   // rounds in which every lane meets another body
    int rel = (own > 0 ? o1 - j0 : 0) + s;   // before wrapping at len
    auto at = [&](int x) {   // unsigned minimum of x and x - len: x < 2 len wrapped
        const unsigned a = (unsigned)x, b = (unsigned)(x - len);
        return j0 + (int)(a < b ? a : b);
    };
    int q = s;
    for (int k0 = 0; k0 < full; k0 += kBlkG) {
        const int k1 = k0 + kBlkG < full ? k0 + kBlkG : full;
#pragma unroll UNROLL
        for (int k = k0; k < k1; ++k) {
            fast(at(rel));
            rel += S;
        }
        flush();
    }
    q += full * S;
    for (; q < len; q += S) {
        masked(at(rel));
        rel += S;
    }
    flush();
}

// T targets per lane, TT lanes side by side on different targets (Tw = T TT
// targets per virtual group), NT threads, S source slices, 16 / TT in every row
// of 16 lanes.  (TT = 3 or 5 leaves the row's last lane without work of its
// own: it repeats the last slice.)  A body
// is four words (x, y, z, G m) in LDS and in the exchange buffers alike, so
// the exchange is a linear copy, and a virtual group of four targets has a
// cache line of its own, which then changes hands once per step.
template <int T, int TT, int NT>
struct GroupDims {
    static constexpr int Tw = T * TT;
    static constexpr int E = 4 * Tw;                    // words of a virtual group
    static constexpr int NR = NT / 16;                  // rows of 16 lanes
    static constexpr int S = NR * (16 / TT);
    static constexpr int LPE = E <= 16 ? 4 : (E <= 32 ? 2 : 1);   // finishing lanes per word
    static constexpr int RS = NR + 1;                   // LDS stride of a sum's row parts
    static constexpr int kB = T < 4 ? 4 * T : 16;       // 16-byte loads per thread in flight
    static_assert(E * LPE <= NT && NR % LPE == 0, "lanes finish a virtual group");
};

template <int T, int TT, int NT, bool SPLIT>
__global__ __launch_bounds__(NT) void k_group(GroupArgs A)
{
    using D = GroupDims<T, TT, NT>;
    constexpr int S = D::S;
    constexpr int Tw = D::Tw;
    constexpr int kUnroll = T == 1 ? 4 : (T == 2 ? 2 : 1);
    extern __shared__ double4 body[];   // [n], then the row parts [3 Tw][RS]
    const int tid = threadIdx.x;
    if (A.spread > 1 && blockIdx.x % A.spread != 0) return;
    int sys = 0, planned = (int)gridDim.x / A.spread;
    int64_t body0 = 0, n64 = A.n, xoff = 0;
    if (A.units) {
        const GroupUnit u = A.units[blockIdx.x];
        sys = u.sys;
        planned = u.workgroups;
        body0 = u.body0;
        xoff = 12 * u.body0;
        n64 = u.n;
        if (u.n == 0) return;   // (padding of the list)
    }
    const int n = (int)n64;
    const int groups = (n + Tw - 1) / Tw;
    uint32_t* reg = A.reg + kGroupRegWords * sys;
    Crew crew = {0, planned, 0, 0};
    if (A.i1 == A.i0) {   // one launch index: no exchange, nobody waits
        crew.rank = A.units ? A.units[blockIdx.x].rank : (int)blockIdx.x / A.spread;
    } else if (planned > 1 && !register_workgroup(reg, planned, crew)) {
        return;
    }

    double* red = reinterpret_cast<double*>(body + n);
    const double* lds = reinterpret_cast<const double*>(body);
    const int64_t stride = A.stride;
    const double* pos_in = A.pos_in + body0;
    const int nm = SPLIT ? (int)A.nmaj[sys] : n;
    // (a workgroup that joins later reads all four words in the exchange)
    for (int q = crew.first > 0 ? n : tid; q < n; q += NT) {
        const double g = A.G * A.mass[body0 + q];
        body[q] = double4{pos_in[q], pos_in[stride + q], pos_in[2 * stride + q],
                          q < nm ? g
                                 : __builtin_bit_cast(double, (uint64_t)__builtin_bit_cast(
                                                                  uint32_t, (float)g))};
    }
    __syncthreads();

    const int col = tid & 15;
    const int row = tid >> 4;
    const int t0 = col % TT;
    const int s = row * (16 / TT) + (col / TT < 16 / TT ? col / TT : 16 / TT - 1);
    const int xwords = 4 * n;
    double* xb = A.xbuf + xoff;   // three buffers of xwords words
    const double hdt = 0.5 * A.dt;
    const PolyConst c = {vreg_const(1.875), vreg_const(1.5)};
    // the word of a virtual group that this lane finishes (component 3: G m,
    // which travels along unchanged)
    const int el = tid / D::LPE;
    const int etgt = el >> 2;
    const int ecomp = el & 3;
    const bool finisher = tid < D::E * D::LPE && tid % D::LPE == 0;
    int budget = kPollBudget;
    bool bad = false;

    // One virtual group's part of launch index x.
    auto step_group = [&](int vg, const Index& x) {
        const int base = vg * Tw;
        Word w;
        w.ep = base + etgt;
        w.comp = ecomp;
        w.mine = finisher && w.ep < n;
        w.e = body0 + ecomp * stride + w.ep;
        w.slot = xb + 4 * base + el;
        const double v = word_begin(A, w, xwords, x);
        double tx[T], ty[T], tz[T], ax[T], ay[T], az[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            // (a lane past the last body repeats it; what it sums is not used)
            const int p = base + t0 + t * TT;
            const double4 b = body[p < n ? p : n - 1];
            tx[t] = b.x;
            ty[t] = b.y;
            tz[t] = b.z;
            ax[t] = 0.0;
            ay[t] = 0.0;
            az[t] = 0.0;
        }
        const int p0 = base + t0;
        each_source<S, kUnroll>(
            0, nm, s, base, base + Tw,
            [&](int j) {
                const double4 b = body[j];
                pair64<T, false, SPLIT>(b.x, b.y, b.z, b.w, j, tx, ty, tz, p0, TT, ax, ay, az, c);
            },
            [&](int j) {
                const double4 b = body[j];
                pair64<T, true, SPLIT>(b.x, b.y, b.z, b.w, j, tx, ty, tz, p0, TT, ax, ay, az, c);
            },
            [] {});
        if (SPLIT) {
            float bx[T], by[T], bz[T];
#pragma unroll
            for (int t = 0; t < T; ++t) { bx[t] = 0.f; by[t] = 0.f; bz[t] = 0.f; }
            each_source<S, kUnroll>(
                nm, n, s, base, base + Tw,
                [&](int j) {
                    const double4 b = body[j];
                    pair32<T, false>(b.x, b.y, b.z, light_gm(b.w), j, tx, ty, tz, p0, TT, bx, by,
                                     bz);
                },
                [&](int j) {
                    const double4 b = body[j];
                    pair32<T, true>(b.x, b.y, b.z, light_gm(b.w), j, tx, ty, tz, p0, TT, bx, by,
                                    bz);
                },
                [&] {
#pragma unroll
                    for (int t = 0; t < T; ++t) {
                        ax[t] += (double)bx[t];
                        ay[t] += (double)by[t];
                        az[t] += (double)bz[t];
                        bx[t] = 0.f;
                        by[t] = 0.f;
                        bz[t] = 0.f;
                    }
                });
        }
        // slices of a row by DPP, rows through LDS, finished by the first lanes
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const double sx = row_sum<TT>(ax[t]);
            const double sy = row_sum<TT>(ay[t]);
            const double sz = row_sum<TT>(az[t]);
            if (col < TT) {
                const int q = t0 + t * TT;
                red[q * D::RS + row] = sx;
                red[(Tw + q) * D::RS + row] = sy;
                red[(2 * Tw + q) * D::RS + row] = sz;
            }
        }
        __syncthreads();
        if (tid < D::E * D::LPE) {
            // LPE lanes per word, each every LPE-th row, in four chains
            const int comp = ecomp < 3 ? ecomp : 0;
            const double* rs = red + (comp * Tw + etgt) * D::RS + tid % D::LPE;
            constexpr int M = D::NR / D::LPE;
            double a4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int m = 0; m < M; ++m) a4[m & 3] += rs[m * D::LPE];
            double a = (a4[0] + a4[1]) + (a4[2] + a4[3]);
            if (D::LPE >= 4) a += row_ror<14>(a);   // lane l: l + 2 of its row
            if (D::LPE >= 2) a += row_ror<15>(a);   // lane l: l + 1
            if (w.mine)
                bad = !word_finish(A, w, xwords, x, a, v, lds[4 * w.ep + ecomp], hdt,
                                   crew.moving) || bad;
        }
    };

    const int last = (int)(A.i1 - A.i0);
    const int64_t left = A.steps - A.i0;   // steps still to open
    const int open_end = left > last ? last + 1 : (int)left;
    const bool begun = A.i0 > 0;
    int cur = crew.first % 3;
    for (int k = crew.first; k <= last; ++k) {
        if (k > 0) {
            const double* src = xb + cur * xwords;
            for (int x0 = tid; x0 < 2 * n; x0 += D::kB * NT)
                gather_words<D::kB, NT>(src, x0, 2 * n, reinterpret_cast<double2*>(body), budget);
            __syncthreads();
        }
        // (rare: kept out of the way of the loop)
        if (__builtin_expect(crew.moving, 0)) share_work(reg, crew, planned, k, last);
        const Index x = {k, last, cur, begun || k > 0, k < open_end};
        if (groups <= crew.present) {
            if (crew.rank < groups) step_group(crew.rank, x);
        } else {
            for (int vg = crew.rank; vg < groups; vg += crew.present) {
                step_group(vg, x);
                __syncthreads();   // red is written again
            }
        }
        cur = x.after();
    }
    if (crew.moving) end_run(reg, crew, planned);
    if (bad && A.flags) atomicOr(A.flags, 1u);
}

// Reverse sweep of one checkpoint segment in one launch: at each of its
// positions, last to first, lam_r += c J^T lam_v and g_m += c M^T lam_v, then
// (but at the run's first) lam_v += dt lam_r.  A product and its reduction per
// position are bound by two kernel boundaries and the partials' round trip:
// 9.6, 12.9 and 16.2 us a step at 131, 1,000 and 2,079 bodies, with the recompute
// beside them; here 2.5, 6.5 and 15.2, with a run kernel's recompute on the
// same CUs, of which the arithmetic of both is 0.1, 1.8 and 9.  The
// exchange is the one above with lam_v (and the mass) in the place of the
// position (and G m); the positions are known beforehand, so they are staged
// ahead of the exchange: into LDS (HELD), or by each lane into registers, P
// rounds at a time, where LDS does not hold both.  MW: wavefronts per SIMD whose
// registers the kernel may not exceed, so that a run kernel's fit beside it.
template <int T, int TT, int NT, bool HELD, int MW>
__global__ __launch_bounds__(NT, MW) void k_group_vjp(GroupVjpArgs A)
{
    using D = GroupDims<T, TT, NT>;
    constexpr int S = D::S;
    constexpr int Tw = D::Tw;
    constexpr int P = T == 1 ? 4 : 2;   // rounds whose loads go out together
    extern __shared__ double4 body[];   // u, m [n], (HELD) x, y, z [3][n], row parts [4 Tw][RS]
    const int tid = threadIdx.x;
    if (A.spread > 1 && blockIdx.x % A.spread != 0) return;
    const int n = (int)A.n;
    const int planned = (int)gridDim.x / A.spread;
    const int groups = (n + Tw - 1) / Tw;
    Crew crew = {0, planned, 0, 0};
    if (planned > 1 && !register_workgroup(A.reg, planned, crew)) return;

    double* held = reinterpret_cast<double*>(body + n);
    double* red = held + (HELD ? 3 * n : 0);
    const double* lds = reinterpret_cast<const double*>(body);
    for (int q = crew.first > 0 ? n : tid; q < n; q += NT)
        body[q] = double4{A.lam_v[q], A.lam_v[n + q], A.lam_v[2 * n + q], A.mass[q]};
    __syncthreads();

    const int col = tid & 15;
    const int row = tid >> 4;
    const int t0 = col % TT;
    const int s = row * (16 / TT) + (col / TT < 16 / TT ? col / TT : 16 / TT - 1);
    const int xwords = 4 * n;
    const int el = tid / D::LPE;   // the word that this lane finishes (3: of g_m)
    const int etgt = el >> 2;
    const int ecomp = el & 3;
    const bool finisher = tid < D::E * D::LPE && tid % D::LPE == 0;
    int budget = kPollBudget;
    const int last = (int)A.count - 1;
    int cur = crew.first % 3;   // i mod 3
    for (int i = crew.first; i <= last; ++i) {
        const bool closing = A.last && i == 0;
        const int64_t k = A.k1 - (i - (A.last ? 1 : 0));   // slot of the position
        const bool start = !closing && A.first && k == 0;
        const double* rp = closing ? A.last : A.seg + k * 3 * A.n;
        for (int vg = crew.rank; vg < groups; vg += crew.present) {
            const int base = vg * Tw;
            const int ep = base + etgt;
            const bool mine = finisher && ep < n;
            double* slot = A.xbuf + 4 * base + el;
            double* acc = ecomp < 3 ? A.lam_r + (int64_t)ecomp * n + ep : A.g_m + ep;
            double old = mine ? *acc : 0.0;
            // positions: held in LDS, or the first rounds' in registers.  The
            // order is that of each_source: the bodies after the group's own targets,
            // wrapping, then the targets.
            const int own1 = base + Tw < n ? base + Tw : n;
            const int full = (n - (own1 - base)) / S;
            auto at = [&](int x) {
                const unsigned a = (unsigned)x, b = (unsigned)(x - n);
                return (int)(a < b ? a : b);
            };
            double nx[P], ny[P], nz[P];
            int nj[P];
            auto fetch = [&](int k0) {
#pragma unroll
                for (int u = 0; u < P; ++u) {
                    const int j = k0 + u < full ? at(own1 + s + (k0 + u) * S) : 0;
                    nj[u] = j;
                    nx[u] = rp[j];
                    ny[u] = rp[n + j];
                    nz[u] = rp[2 * n + j];
                }
            };
            if (!HELD)
                fetch(0);
            else if (vg == crew.rank)
                for (int q = tid; q < 3 * n; q += NT) held[q] = rp[q];
            if (vg == crew.rank && i > 0) {
                const double* src = A.xbuf + cur * xwords;
                for (int x0 = tid; x0 < 2 * n; x0 += D::kB * NT)
                    gather_words<D::kB, NT>(src, x0, 2 * n, reinterpret_cast<double2*>(body),
                                            budget);
            }
            if (vg == crew.rank) __syncthreads();
            if (crew.moving) {
                if (vg == crew.rank) share_work(A.reg, crew, planned, i, last);
                if (mine) old = *acc;   // (its owner may have changed)
            }
            if (mine && i > 1 && i < last)
                __hip_atomic_store(slot + (cur == 0 ? 2 : cur - 1) * xwords,
                                   __builtin_bit_cast(double, kSentinel), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            double tx[T], ty[T], tz[T], qm[T], ux[T], uy[T], uz[T], ox[T], oy[T], oz[T], og[T];
            int64_t qid[T];
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int p = base + t0 + t * TT;
                const int q = p < n ? p : n - 1;
                const double4 b = body[q];
                const double* ps = HELD ? held : rp;
                tx[t] = ps[q];
                ty[t] = ps[n + q];
                tz[t] = ps[2 * n + q];
                qid[t] = p;
                ux[t] = b.x;
                uy[t] = b.y;
                uz[t] = b.z;
                qm[t] = b.w;
                ox[t] = 0.0;
                oy[t] = 0.0;
                oz[t] = 0.0;
                og[t] = 0.0;
            }
            const double* ps = HELD ? held : rp;
            auto term = [&](auto mask, int j, double x, double y, double z) {
                const double4 b = body[j];
                vjp_pair<T, decltype(mask)::value>(x, y, z, b.w, b.x, b.y, b.z, j, tx, ty, tz, qm,
                                                   ux, uy, uz, qid, ox, oy, oz, og);
            };
            if (HELD) {
#pragma unroll P
                for (int k0 = 0; k0 < full; ++k0) {
                    const int j = at(own1 + s + k0 * S);
                    term(std::false_type{}, j, ps[j], ps[n + j], ps[2 * n + j]);
                }
            } else {
                for (int k0 = 0; k0 < full; k0 += P) {
                    double bx[P], by[P], bz[P];
                    int bj[P];
#pragma unroll
                    for (int u = 0; u < P; ++u) {
                        bx[u] = nx[u];
                        by[u] = ny[u];
                        bz[u] = nz[u];
                        bj[u] = nj[u];
                    }
                    fetch(k0 + P);
#pragma unroll
                    for (int u = 0; u < P; ++u)
                        if (k0 + u < full) term(std::false_type{}, bj[u], bx[u], by[u], bz[u]);
                }
            }
            for (int q = s + full * S; q < n; q += S) {
                const int j = at(own1 + q);
                term(std::true_type{}, j, ps[j], ps[n + j], ps[2 * n + j]);
            }
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const double sx = row_sum<TT>(ox[t]);
                const double sy = row_sum<TT>(oy[t]);
                const double sz = row_sum<TT>(oz[t]);
                const double sg = row_sum<TT>(og[t]);
                if (col < TT) {
                    const int x = t0 + t * TT;
                    red[x * D::RS + row] = sx;
                    red[(Tw + x) * D::RS + row] = sy;
                    red[(2 * Tw + x) * D::RS + row] = sz;
                    red[(3 * Tw + x) * D::RS + row] = sg;
                }
            }
            __syncthreads();
            if (tid < D::E * D::LPE) {
                const double* rs = red + (ecomp * Tw + etgt) * D::RS + tid % D::LPE;
                constexpr int M = D::NR / D::LPE;
                double a4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int m = 0; m < M; ++m) a4[m & 3] += rs[m * D::LPE];
                double a = (a4[0] + a4[1]) + (a4[2] + a4[3]);
                if (D::LPE >= 4) a += row_ror<14>(a);
                if (D::LPE >= 2) a += row_ror<15>(a);
                if (mine) {
                    const double gc = A.G * (closing || start ? 0.5 * A.dt : A.dt);
                    const double r = old + (ecomp < 3 ? gc : -gc) * a;
                    double w = lds[4 * ep + ecomp];
                    if (crew.moving) agent_store(acc, r);
                    else             *acc = r;
                    if (ecomp < 3 && !start) w = __builtin_fma(A.dt, r, w);
                    if (i < last) {
                        // the reset above has arrived before this word does
                        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                        publish(slot + (cur == 2 ? 0 : cur + 1) * xwords, w);
                    } else if (ecomp < 3) {
                        A.lam_v[(int64_t)ecomp * n + ep] = w;
                    }
                }
            }
            if (groups > crew.present) __syncthreads();   // red is written again
        }
        cur = cur == 2 ? 0 : cur + 1;
    }
    if (crew.moving) end_run(A.reg, crew, planned);
}

__global__ __launch_bounds__(256) void k_group_init(double* __restrict__ xbuf, int64_t words,
                                                    uint32_t* __restrict__ reg, int nreg)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < words) xbuf[i] = __builtin_bit_cast(double, kSentinel);
    if (i < nreg) reg[i] = 0;
}

// Allows a kernel more than the default limit of dynamic LDS, once per device.
hipError_t allow_lds(const void* kernel, std::atomic<uint64_t>& allowed)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = (uint64_t)1 << (dev & 63);
    if (dev <= 63 && (allowed.load(std::memory_order_relaxed) & bit)) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
    if (e == hipSuccess) allowed.fetch_or(bit, std::memory_order_relaxed);
    return e;
}

template <int T, int TT, int NT, bool SPLIT>
hipError_t launch_shape(const GroupArgs& A, int blocks, size_t lds, hipStream_t s)
{
    static std::atomic<uint64_t> allowed{0};
    const hipError_t e =
        allow_lds(reinterpret_cast<const void*>(&k_group<T, TT, NT, SPLIT>), allowed);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_group<T, TT, NT, SPLIT>), dim3((unsigned)(blocks * A.spread)), dim3(NT),
                       lds, s, A);
    return hipGetLastError();
}

template <int T, int TT, int NT, bool HELD, int MW>
hipError_t launch_vjp_shape(const GroupVjpArgs& A, int blocks, size_t lds, hipStream_t s)
{
    static std::atomic<uint64_t> allowed{0};
    const hipError_t e =
        allow_lds(reinterpret_cast<const void*>(&k_group_vjp<T, TT, NT, HELD, MW>), allowed);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_group_vjp<T, TT, NT, HELD, MW>), dim3((unsigned)(blocks * A.spread)),
                       dim3(NT), lds, s, A);
    return hipGetLastError();
}

hipError_t init_exchange(double* xbuf, int64_t words, uint32_t* reg, int nsys, hipStream_t s)
{
    const int nreg = kGroupRegWords * nsys;
    const int64_t m = words > nreg ? words : nreg;
    hipLaunchKernelGGL(k_group_init, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, s, xbuf,
                       words, reg, nreg);
    return hipGetLastError();
}

}  // namespace

size_t group_lds_bytes(int64_t n, const GroupShape& g)
{
    const int64_t tw = (int64_t)g.tpl * g.lanes;
    return (size_t)(4 * n + 3 * tw * (g.threads / 16 + 1)) * sizeof(double);
}

hipError_t launch_group(int precision, const GroupShape& g, const GroupArgs& A, int blocks,
                        int64_t n_max, int64_t words, int nsys, hipStream_t s)
{
    if (blocks < 1 || A.i1 < A.i0 || (precision == 1 && !A.nmaj)) return hipErrorInvalidValue;
    const size_t lds = group_lds_bytes(n_max, g);
    if (lds > (size_t)kMaxLds) return hipErrorInvalidValue;
    if (A.i1 > A.i0) {
        const hipError_t e = init_exchange(A.xbuf, words, A.reg, nsys, s);
        if (e != hipSuccess) return e;
    }
#define NB_CASE(TT_, LL, NN)                                                                 \
    if (g.tpl == TT_ && g.lanes == LL && g.threads == NN)                                    \
        return precision == 0 ? launch_shape<TT_, LL, NN, false>(A, blocks, lds, s)          \
                              : launch_shape<TT_, LL, NN, true>(A, blocks, lds, s);
    NB_GROUP_SHAPES(NB_CASE)
#undef NB_CASE
    return hipErrorInvalidValue;
}

size_t group_vjp_lds_bytes(int64_t n, const GroupVjpShape& g)
{
    const int64_t tw = (int64_t)g.tpl * g.lanes;
    return (size_t)((g.held ? 7 : 4) * n + 4 * tw * (g.threads / 16 + 1)) * sizeof(double);
}

hipError_t launch_group_vjp(const GroupVjpShape& g, const GroupVjpArgs& A, hipStream_t s)
{
    if (A.count < 2 || A.n < 1) return hipErrorInvalidValue;
    const size_t lds = group_vjp_lds_bytes(A.n, g);
    if (lds > (size_t)kMaxLds) return hipErrorInvalidValue;
    const hipError_t e = init_exchange(A.xbuf, 12 * A.n, A.reg, 1, s);
    if (e != hipSuccess) return e;
    const int64_t tw = (int64_t)g.tpl * g.lanes;
    const int blocks = (int)((A.n + tw - 1) / tw);
#define NB_CASE(TT_, LL, NN, HH, MW)                                              \
    if (g.tpl == TT_ && g.lanes == LL && g.threads == NN && g.held == HH)        \
        return launch_vjp_shape<TT_, LL, NN, HH, MW>(A, blocks, lds, s);
    NB_GROUP_VJP_SHAPES(NB_CASE)
#undef NB_CASE
    return hipErrorInvalidValue;
}

}  // namespace nb
