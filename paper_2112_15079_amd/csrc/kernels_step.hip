// O(N) kernels around the force pass: the kick-drift-kick step epilogue that
// realises Eqs. (3)-(4), the class-order gather/scatter of the split form,
// and the diagnostics of Sec. 2 (energy, momenta).
#include "common.hpp"
#include "pair_math.hpp"
#include "reduce.hpp"

namespace nb {
namespace {

using namespace pm;

constexpr int kBlock = 256;

// Sum the chunk partials of a_p in a fixed order (below), then apply the
// half kicks and the drift:
//   kClose: v += dt/2 a                         (v_{i+1}, end of step i)
//   kOpen:  v += dt/2 a;  r_out = r_in + dt v   (v_{i+3/2}, r_{i+2})
// Eqs. (3)-(4) follow: r_{i+1} = r_i + dt (v_i + dt/2 a_i) and
// v_{i+1} = v_i + dt/2 a_i + dt/2 a_{i+1}.
// GS threads per (body, component) sum the partials (chunk_sum); the state
// the epilogue reads is loaded before the partials, so its latency overlaps
// theirs.
// PER_BODY: an ensemble's per-body partial counts (body_chunks) instead of
// one count for every body.  PERM: accelerations are stored at perm[p] (a
// variant of its own: a step of 10,425 bodies took 0.24 us longer with the test).
template <int GS, bool PER_BODY, bool PERM = false>
__global__ __launch_bounds__(kBlock) void k_step(const double* __restrict__ part, int chunks,
                                                 const int8_t* __restrict__ body_chunks,
                                                 int64_t n, double* __restrict__ vel,
                                                 const double* __restrict__ pos_in,
                                                 double* __restrict__ pos_out,
                                                 double* __restrict__ acc,
                                                 const int32_t* __restrict__ perm, double hdt,
                                                 double dt, int mode,
                                                 uint32_t* __restrict__ flags)
{
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t i = t / GS;   // k * n + p
    const int sub = (int)(t % GS);
    const bool live = i < 3 * n;
    const int64_t ii = live ? i : 0;
    const int64_t p = ii % n;
    const int C = PER_BODY ? (int)body_chunks[p] : chunks;
    const bool head = live && sub == 0;
    const double v0 = (head && (mode & (kClose | kOpen))) ? vel[i] : 0.0;
    const double r0 = (head && (mode & kOpen)) ? pos_in[i] : 0.0;
    const double a = chunk_sum<GS>(part, C, 3 * n, ii, sub, live);
    if (!head) return;
    bool finite = __builtin_isfinite(a);
    if (mode & kStoreAcc) acc[PERM ? i - p + perm[p] : i] = a;
    if (mode & (kClose | kOpen)) {
        double v = v0;
        if (mode & kClose) v = v + hdt * a;
        if (mode & kOpen) {
            v = v + hdt * a;
            const double r = r0 + dt * v;
            finite = finite && __builtin_isfinite(r);
            pos_out[i] = r;
        }
        finite = finite && __builtin_isfinite(v);
        vel[i] = v;
    }
    if (!finite && flags) atomicOr(flags, 1u);
}

// The accelerations of targets t0 .. t0 + nt - 1 from the chunk partials of
// a pass over those targets (GS threads per (component, target) element,
// summed by chunk_sum), into planes of stride nt.
template <int GS>
__global__ __launch_bounds__(kBlock) void k_shard_sum(const double* __restrict__ part,
                                                      int chunks, int64_t n, int64_t t0,
                                                      int64_t nt, double* __restrict__ out)
{
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t e = t / GS;   // k * nt + q
    const int sub = (int)(t % GS);
    const bool live = e < 3 * nt;
    const int64_t ee = live ? e : 0;
    const int64_t k = ee / nt;
    const int64_t q = ee - k * nt;
    const double a = chunk_sum<GS>(part, chunks, 3 * n, k * n + t0 + q, sub, live);
    if (live && sub == 0) out[e] = a;
}

// Classical fourth-order Runge-Kutta (r' = v, v' = a(r)): stage s's
// acceleration a (the chunk partials of the force pass at the stage position,
// summed in ascending chunk order) and the stage velocity give the slopes
// (kr, kv); sr, sv accumulate kr1 + 2 kr2 + 2 kr3 and kv1 + 2 kv2 + 2 kv3;
//   s = 1: kr = v,  next stage at (r + dt/2 kr, v + dt/2 kv)
//   s = 2: kr = vs, next stage at (r + dt/2 kr, v + dt/2 kv)
//   s = 3: kr = vs, next stage at (r + dt kr,   v + dt kv)
//   s = 4: kr = vs, r += dt/6 (sr + kr), v += dt/6 (sv + kv).
template <int GS>
__global__ __launch_bounds__(kBlock) void k_rk4_stage(const double* __restrict__ part, int chunks,
                                                      int64_t n, int stage, double dt,
                                                      double* __restrict__ pos,
                                                      double* __restrict__ vel,
                                                      double* __restrict__ rs,
                                                      double* __restrict__ vs,
                                                      double* __restrict__ sr,
                                                      double* __restrict__ sv,
                                                      uint32_t* __restrict__ flags)
{
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t i = t / GS;
    const int sub = (int)(t % GS);
    const bool live = i < 3 * n;
    const int64_t ii = live ? i : 0;
    const bool head = live && sub == 0;
    double p0 = 0.0, v0 = 0.0, vs0 = 0.0, sr0 = 0.0, sv0 = 0.0;
    if (head) {
        p0 = pos[i];
        v0 = vel[i];
        if (stage > 1) {
            vs0 = vs[i];
            sr0 = sr[i];
            sv0 = sv[i];
        }
    }
    const double a = chunk_sum<GS>(part, chunks, 3 * n, ii, sub, live);
    if (!head) return;
    bool finite = __builtin_isfinite(a);
    const double kr = (stage == 1) ? v0 : vs0;
    if (stage < 4) {
        if (stage == 1) {
            sr[i] = kr;
            sv[i] = a;
        } else {
            sr[i] = sr0 + 2.0 * kr;
            sv[i] = sv0 + 2.0 * a;
        }
        const double h = (stage == 3) ? dt : 0.5 * dt;
        const double r = p0 + h * kr;
        const double v = v0 + h * a;
        finite = finite && __builtin_isfinite(r) && __builtin_isfinite(v);
        rs[i] = r;
        vs[i] = v;
    } else {
        const double h6 = dt / 6.0;
        const double r = p0 + h6 * (sr0 + kr);
        const double v = v0 + h6 * (sv0 + a);
        finite = finite && __builtin_isfinite(r) && __builtin_isfinite(v);
        pos[i] = r;
        vel[i] = v;
    }
    if (!finite && flags) atomicOr(flags, 1u);
}

// Back from class order: planes 0 .. 2 of a (and, from grid.y = 3 on, of b).
__global__ __launch_bounds__(kBlock) void k_scatter(const int32_t* __restrict__ perm, int64_t n,
                                                    const double* __restrict__ a_c,
                                                    double* __restrict__ a,
                                                    const double* __restrict__ b_c,
                                                    double* __restrict__ b)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const int k = blockIdx.y;
    if (k < 3) a[(int64_t)k * n + perm[i]] = a_c[(int64_t)k * n + i];
    else       b[(int64_t)(k - 3) * n + perm[i]] = b_c[(int64_t)(k - 3) * n + i];
}

// Class order (split form), one launch: workgroup (x, y) places slice y of
// system x.  It counts the system's heavy bodies itself, before its slice
// and in all, instead of waiting for the other slices' counts (8 n bytes read
// from L2 per workgroup: 2 us at 10,425 bodies, where one workgroup that scans
// slice after slice took 23 us and three gathers and a scale followed it);
// within the slice, ranks come from wave ballots.
constexpr int kPart = 1024;

struct ClassOrder {
    const double* pos;
    const double* vel;
    const double* mass;
    const int64_t* offsets;
    int64_t n;          // plane stride (all systems' bodies)
    double threshold, G;
    int32_t* perm;
    int64_t* nmaj;
    double *pos_c, *vel_c, *mass_c, *gm_c;
};

__global__ __launch_bounds__(kPart) void k_class_order(ClassOrder P)
{
    constexpr int NW = kPart / 64;
    __shared__ int s_before[NW], s_all[NW], s_wave[2][NW];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = tid >> 6;
    const int64_t b0 = P.offsets ? P.offsets[blockIdx.x] : 0;
    const int64_t b1 = P.offsets ? P.offsets[blockIdx.x + 1] : P.n;
    const int64_t per = ((b1 - b0 + gridDim.y - 1) / gridDim.y + kPart - 1) / kPart * kPart;
    const int64_t s0 = b0 + blockIdx.y * per;
    const int64_t s1 = s0 + per < b1 ? s0 + per : b1;
    if (s0 >= b1) return;

    int before = 0, all = 0;
    for (int64_t i = b0 + tid; i < b1; i += kPart) {
        const int f = P.mass[i] >= P.threshold ? 1 : 0;
        all += f;
        before += i < s0 ? f : 0;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        before += __shfl_xor(before, o, 64);
        all += __shfl_xor(all, o, 64);
    }
    if (lane == 0) {
        s_before[w] = before;
        s_all[w] = all;
    }
    __syncthreads();
    int64_t major = 0, total = 0;
    for (int k = 0; k < NW; ++k) {
        major += s_before[k];
        total += s_all[k];
    }
    if (blockIdx.y == 0 && tid == 0) P.nmaj[blockIdx.x] = total;
    int64_t small = total + (s0 - b0) - major;   // next place of each class

    int buf = 0;
    for (int64_t c0 = s0; c0 < s1; c0 += kPart, buf ^= 1) {
        const int64_t i = c0 + tid;
        const bool valid = i < s1;
        const double m = valid ? P.mass[i] : 0.0;
        const bool f = valid && m >= P.threshold;
        const uint64_t mask = __ballot(f);
        if (lane == 0) s_wave[buf][w] = __popcll(mask);
        __syncthreads();   // (the next round writes the other buffer)
        int rank = __popcll(mask & (((uint64_t)1 << lane) - 1)), sum = 0;
        for (int k = 0; k < NW; ++k) {
            const int c = s_wave[buf][k];
            rank += k < w ? c : 0;
            sum += c;
        }
        if (valid) {
            const int64_t o = b0 + (f ? major + rank : small + (tid - rank));
            P.perm[o] = (int32_t)i;
            P.mass_c[o] = m;
            P.gm_c[o] = P.G * m;
            for (int k = 0; k < 3; ++k) P.pos_c[k * P.n + o] = P.pos[k * P.n + i];
            if (P.vel)
                for (int k = 0; k < 3; ++k) P.vel_c[k * P.n + o] = P.vel[k * P.n + i];
        }
        major += sum;
        small += (s1 - c0 < kPart ? s1 - c0 : kPart) - sum;
    }
}

// ---------------------------------------------------------------------------
// Diagnostics.  Neumaier-compensated sums; fixed summation order.
struct CSum {
    double s, c;
};

__device__ __forceinline__ void cadd(CSum& a, double x)
{
    const double t = a.s + x;
    if (fabs(a.s) >= fabs(x)) a.c += (a.s - t) + x;
    else                      a.c += (x - t) + a.s;
    a.s = t;
}

__device__ __forceinline__ void cmerge(CSum& a, const CSum& b)
{
    cadd(a, b.s);
    cadd(a, b.c);
}

// The compensated sum of s and x without a branch (Knuth's two-sum: the error is
// exact, as in cadd, in 7 additions).
__device__ __forceinline__ void cadd7(CSum& a, double x)
{
    const double t = a.s + x;
    const double z = t - a.s;
    a.c += (a.s - (t - z)) + (x - z);
    a.s = t;
}

// m times a compensated sum, compensated.
__device__ __forceinline__ CSum cscale(double m, const CSum& a)
{
    const double p = m * a.s;
    return CSum{p, __builtin_fma(m, a.s, -p) + m * a.c};
}

// The sums of V values over a workgroup of NT threads, in a fixed order: wave v
// takes value v, each lane every 64th thread's, then the lanes pairwise.  The
// sum of value v is complete in lane 0 of wave v.  sh: V * NT values.
template <int V, int NT>
__device__ __forceinline__ CSum block_sums(CSum* sh, const CSum (&x)[V])
{
    static_assert(V <= NT / 64, "a wave per value");
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
#pragma unroll
    for (int v = 0; v < V; ++v) sh[v * NT + threadIdx.x] = x[v];
    __syncthreads();
    CSum a = {0.0, 0.0};
    if (w < V) {
        const CSum* row = sh + w * NT;
        a = row[lane];
#pragma unroll
        for (int k = 1; k < NT / 64; ++k) cmerge(a, row[64 * k + lane]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
            cmerge(a, CSum{__shfl_down(a.s, o, 64), __shfl_down(a.c, o, 64)});
    }
    return a;
}

constexpr int kRowTile = 256;
constexpr int kSrcTile = 128;

// The pair potential of Sec. 2, each unordered pair once, and the kinetic
// energy: workgroup (x, y) sums m_p m_j / |r_j - r_p| over its 256 rows p and
// the sources j > p of chunk y (compensated per row, then over the rows) and,
// if y = 0, its rows' m v^2 / 2, into part[4 (y gridDim.x + x) ..] as two
// (s, c).  Bound by the vector ALU: 23 issue slots a pair, 7 of them the
// compensation (the branch-free two-sum, for 10 slots with compares and
// selects); the diagonal's tiles select instead of branching, which keeps their
// pairs in flight together.  Both energies of 10,425 bodies: 57 us (102 with
// rows merged through memory and one workgroup's tree), 1,000 bodies 16 (47),
// 131,072 7.1 ms (11.8).  Two rows per lane: 63 us, 22 us and 6.4 ms.
__global__ __launch_bounds__(kRowTile) void k_energy_tiles(const double* __restrict__ pos,
                                                           const double* __restrict__ vel,
                                                           const double* __restrict__ mass,
                                                           int64_t n, int64_t chunk_len,
                                                           double* __restrict__ part)
{
    __shared__ double4 src[kSrcTile];
    __shared__ CSum sh[2 * kRowTile];
    const int tid = threadIdx.x;
    const int64_t row0 = (int64_t)blockIdx.x * kRowTile;
    const int64_t c0 = (int64_t)blockIdx.y * chunk_len;
    const int64_t c1 = c0 + chunk_len < n ? c0 + chunk_len : n;
    CSum x[2] = {{0.0, 0.0}, {0.0, 0.0}};
    if (blockIdx.y == 0 || c1 > row0) {   // (a chunk wholly before the rows: zeros)
        const int64_t p = row0 + tid;
        const int64_t q = p < n ? p : n - 1;
        const double px = pos[q], py = pos[n + q], pz = pos[2 * n + q];
        const double m = p < n ? mass[q] : 0.0;
        CSum acc = {0.0, 0.0};
        // sources j > p only: from the tile that holds the first row on
        for (int64_t j0 = c0 > row0 ? c0 : row0; j0 < c1; j0 += kSrcTile) {
            __syncthreads();
            const int64_t j = j0 + tid;
            const int cnt = c1 - j0 < kSrcTile ? (int)(c1 - j0) : kSrcTile;
            if (tid < cnt) src[tid] = double4{pos[j], pos[n + j], pos[2 * n + j], mass[j]};
            __syncthreads();
            auto term = [&](const double4& b) {
                const double dx = b.x - px, dy = b.y - py, dz = b.z - pz;
                const double r2 = __builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx));
                return b.w * rinv_f64(r2);
            };
            if (j0 >= row0 + kRowTile && cnt == kSrcTile) {   // all past every row
#pragma unroll 4
                for (int k = 0; k < kSrcTile; ++k) cadd7(acc, term(src[k]));
            } else {
#pragma unroll 4
                for (int k = 0; k < cnt; ++k) {
                    const double e = term(src[k]);
                    cadd7(acc, j0 + k > q ? e : 0.0);
                }
            }
        }
        x[0] = cscale(m, acc);
        if (blockIdx.y == 0 && p < n) {
            const double vx = vel[p], vy = vel[n + p], vz = vel[2 * n + p];
            x[1].s = 0.5 * m * (vx * vx + vy * vy + vz * vz);
        }
    }
    const CSum a = block_sums<2, kRowTile>(sh, x);
    if ((tid & 63) == 0 && tid < 128) {
        double* o = part + 4 * ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) + 2 * (tid >> 6);
        o[0] = a.s;
        o[1] = a.c;
    }
}

constexpr int kRed = 1024;

// out = kinetic, potential, total from the tiles' sums, in tile order per lane.
__global__ __launch_bounds__(kRed) void k_energy_finish(const double* __restrict__ part,
                                                        int64_t tiles, double G,
                                                        double* __restrict__ out)
{
    __shared__ CSum sh[2 * kRed];
    const int tid = threadIdx.x;
    CSum x[2] = {{0.0, 0.0}, {0.0, 0.0}};
    for (int64_t i = tid; i < tiles; i += kRed) {
        const double4 t = reinterpret_cast<const double4*>(part)[i];
        cmerge(x[0], CSum{t.x, t.y});
        cmerge(x[1], CSum{t.z, t.w});
    }
    CSum a = block_sums<2, kRed>(sh, x);
    __syncthreads();
    if ((tid & 63) == 0 && tid < 128) sh[tid >> 6] = a;
    __syncthreads();
    if (tid == 0) {
        const CSum U = cscale(-G, sh[0]);
        const double k = sh[1].s + sh[1].c, u = U.s + U.c;
        CSum e = {0.0, 0.0};
        cadd(e, k);
        cadd(e, u);
        out[0] = k;
        out[1] = u;
        out[2] = e.s + e.c;
    }
}

// One workgroup (the call has no scratch memory): 6 waves finish a component
// each (11 us at 10,425 bodies; 18 with a tree over all threads per component).
__global__ __launch_bounds__(kRed) void k_momenta(const double* __restrict__ pos,
                                                  const double* __restrict__ vel,
                                                  const double* __restrict__ mass, int64_t n,
                                                  double* __restrict__ out)
{
    __shared__ CSum sh[6 * kRed];
    const int tid = threadIdx.x;
    CSum c[6];
    for (int k = 0; k < 6; ++k) c[k] = {0.0, 0.0};
#pragma unroll 2
    for (int64_t i = tid; i < n; i += kRed) {
        const double rx = pos[i], ry = pos[n + i], rz = pos[2 * n + i];
        const double vx = vel[i], vy = vel[n + i], vz = vel[2 * n + i];
        const double m = mass[i];
        cadd7(c[0], m * vx);
        cadd7(c[1], m * vy);
        cadd7(c[2], m * vz);
        cadd7(c[3], m * (ry * vz - rz * vy));
        cadd7(c[4], m * (rz * vx - rx * vz));
        cadd7(c[5], m * (rx * vy - ry * vx));
    }
    const CSum a = block_sums<6, kRed>(sh, c);
    if ((tid & 63) == 0 && tid < 6 * 64) out[tid >> 6] = a.s + a.c;
}

}  // namespace

static inline unsigned blocks_for(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

hipError_t launch_step(const double* part, int chunks, const int8_t* body_chunks, int64_t n,
                       double* vel, const double* pos_in, double* pos_out, double* acc,
                       double dt, int mode, uint32_t* flags, hipStream_t s, const int32_t* perm)
{
    // four threads per element for 16 to 95 partials of a single system; one
    // below that, from 96 partials (the each-pair-once pass on large systems)
    // and for an ensemble's per-body counts, where each load of a wavefront
    // then reads 512 contiguous bytes of one partial plane (measured faster)
    const double hdt = 0.5 * dt;
#define NB_STEP(GS, PER_BODY, PERM)                                                         \
    hipLaunchKernelGGL((k_step<GS, PER_BODY, PERM>), dim3(blocks_for(3 * GS * n, kBlock)),  \
                       dim3(kBlock), 0, s, part, chunks, body_chunks, n, vel, pos_in, pos_out, \
                       acc, perm, hdt, dt, mode, flags)
    const bool four = chunks >= 16 && chunks < 96;
    if (body_chunks) NB_STEP(1, true, false);
    else if (perm && four) NB_STEP(4, false, true);
    else if (perm) NB_STEP(1, false, true);
    else if (four) NB_STEP(4, false, false);
    else NB_STEP(1, false, false);
#undef NB_STEP
    return hipGetLastError();
}

hipError_t launch_shard_sum(const double* part, int chunks, int64_t n, int64_t t0, int64_t nt,
                            double* out, hipStream_t s)
{
    if (chunks >= 16 && chunks < 96)
        hipLaunchKernelGGL(k_shard_sum<4>, dim3(blocks_for(12 * nt, kBlock)), dim3(kBlock), 0, s,
                           part, chunks, n, t0, nt, out);
    else
        hipLaunchKernelGGL(k_shard_sum<1>, dim3(blocks_for(3 * nt, kBlock)), dim3(kBlock), 0, s,
                           part, chunks, n, t0, nt, out);
    return hipGetLastError();
}

hipError_t launch_rk4_stage(const double* part, int chunks, int64_t n, int stage, double dt,
                            double* pos, double* vel, double* rs, double* vs, double* sr,
                            double* sv, uint32_t* flags, hipStream_t s)
{
    if (stage < 1 || stage > 4) return hipErrorInvalidValue;
    if (chunks >= 16)
        hipLaunchKernelGGL(k_rk4_stage<4>, dim3(blocks_for(12 * n, kBlock)), dim3(kBlock), 0, s,
                           part, chunks, n, stage, dt, pos, vel, rs, vs, sr, sv, flags);
    else
        hipLaunchKernelGGL(k_rk4_stage<1>, dim3(blocks_for(3 * n, kBlock)), dim3(kBlock), 0, s,
                           part, chunks, n, stage, dt, pos, vel, rs, vs, sr, sv, flags);
    return hipGetLastError();
}

hipError_t launch_class_order(const double* pos, const double* vel, const double* mass,
                              const int64_t* offsets, int num_systems, int64_t n, int64_t n_max,
                              double threshold, double G, int32_t* perm, int64_t* nmaj,
                              double* pos_c, double* vel_c, double* mass_c, double* gm_c,
                              hipStream_t s)
{
    // slices of 1,024 bodies, fewer and longer ones for large systems and for many
    // (every system has as many as the largest); the systems along x, which
    // alone takes more than 65,535
    const int64_t most = num_systems < 64 ? 1024 : num_systems < 65536 ? 65536 / num_systems : 1;
    const int64_t slices = (n_max + kPart - 1) / kPart;
    const dim3 grid((unsigned)num_systems, (unsigned)(slices < most ? slices : most));
    const ClassOrder P{pos, vel, mass, offsets, n, threshold, G, perm, nmaj,
                       pos_c, vel_c, mass_c, gm_c};
    hipLaunchKernelGGL(k_class_order, grid, dim3(kPart), 0, s, P);
    return hipGetLastError();
}

hipError_t launch_scatter(const int32_t* perm, int64_t n, const double* a_c, double* a,
                          const double* b_c, double* b, hipStream_t s)
{
    hipLaunchKernelGGL(k_scatter, dim3(blocks_for(n, kBlock), b ? 6 : 3), dim3(kBlock), 0, s,
                       perm, n, a_c, a, b_c, b);
    return hipGetLastError();
}

hipError_t launch_energy(const double* pos, const double* vel, const double* mass, int64_t n,
                         double G, double* part, int64_t part_doubles, double* out, hipStream_t s)
{
    // source chunks of whole tiles until about 2,048 workgroups have work (half
    // of the (row block, chunk) grid lies below the diagonal; 10,425 bodies:
    // about 7 per CU), as far as the tiles' sums (4 doubles each) have room
    const int64_t row_blocks = blocks_for(n, kRowTile);
    int64_t c = (4096 + row_blocks - 1) / row_blocks;
    const int64_t room = part_doubles / (4 * row_blocks);
    c = c < 1 ? 1 : c > room ? room : c;
    if (c < 1) return hipErrorInvalidValue;
    const int64_t per = (n + c - 1) / c;
    const int64_t chunk_len = (per + kSrcTile - 1) / kSrcTile * kSrcTile;
    const int chunks = (int)((n + chunk_len - 1) / chunk_len);
    hipLaunchKernelGGL(k_energy_tiles, dim3((unsigned)row_blocks, (unsigned)chunks),
                       dim3(kRowTile), 0, s, pos, vel, mass, n, chunk_len, part);
    hipLaunchKernelGGL(k_energy_finish, dim3(1), dim3(kRed), 0, s, part, row_blocks * chunks, G,
                       out);
    return hipGetLastError();
}

hipError_t launch_momenta(const double* pos, const double* vel, const double* mass, int64_t n,
                          double* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_momenta, dim3(1), dim3(kRed), 0, s, pos, vel, mass, n, out);
    return hipGetLastError();
}

}  // namespace nb
