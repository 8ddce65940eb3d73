// Test instrument: the kernels of runs that stay on the chip with workgroups
// that come late.  This file includes the library's own source; the first
// workgroup to register starts the run at once, and workgroups from block
// `late_from` on register only when the run has begun and its announced launch
// index has reached late_step times 1 to 5 (block mod 5), or the run has ended.
// Every wait ends: blocks below late_from do not wait, so the run begins and
// ends without the others.  Built into tests/host/libgroupprobe.so by the
// package build; used by the GPU tests only, never by the library.
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nb {
namespace {
__device__ int probe_late_from, probe_late_step;

__device__ void probe_entry(uint32_t* reg)
{
    if (threadIdx.x != 0 || (int)blockIdx.x < probe_late_from) return;
    const uint32_t want = (uint32_t)probe_late_step * (1 + blockIdx.x % 5);
    uint64_t word;
    do {
        word = __hip_atomic_load(reinterpret_cast<uint64_t*>(reg + 2), __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
    } while (word == 0 || (uint32_t)(word >> 32) < want);
}
}  // namespace
}  // namespace nb

#define NB_GROUP_REGISTER_TICKS 0
#define NB_GROUP_ENTRY(reg) probe_entry(reg);
#include "kernels_group.hip"

namespace {

int hold(int late_from, int late_step, hipStream_t s)
{
    if (late_from < 1 || late_step < 0) return 1;
    if (hipMemcpyToSymbolAsync(HIP_SYMBOL(nb::probe_late_from), &late_from, sizeof late_from, 0,
                               hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemcpyToSymbolAsync(HIP_SYMBOL(nb::probe_late_step), &late_step, sizeof late_step, 0,
                               hipMemcpyHostToDevice, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return 2;
    return 0;
}

}  // namespace

#define EXPORT extern "C" __attribute__((visibility("default")))

// One launch of launch indices 0 .. steps: state in pos, vel; traj (or NULL)
// takes the positions after each drift.  nmaj: NULL for FP64.
EXPORT int group_probe_run(int tpl, int lanes, int threads, int spread, int late_from,
                           int late_step, double* pos, double* vel, const double* mass, int64_t n,
                           const int64_t* nmaj, double G, double dt, int64_t steps, double* traj,
                           double* xbuf, uint32_t* reg, uint32_t* flags, void* stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (n < 1 || steps < 1 || tpl < 1 || lanes < 1 || spread < 1) return 1;
    if (const int rc = hold(late_from, late_step, s)) return rc;
    nb::GroupArgs A{};
    A.pos_in = pos;
    A.pos_out = pos;
    A.vel = vel;
    A.mass = mass;
    A.xbuf = xbuf;
    A.reg = reg;
    A.nmaj = nmaj;
    A.traj = traj;
    A.flags = flags;
    A.n = n;
    A.stride = n;
    A.G = G;
    A.dt = dt;
    A.i1 = steps;
    A.steps = steps;
    A.spread = spread;
    const int tw = tpl * lanes;
    return nb::launch_group(nmaj ? 1 : 0, {tpl, lanes, threads}, A, (int)((n + tw - 1) / tw), n,
                            12 * n, 1, s) == hipSuccess ? 0 : 3;
}

// One launch of the reverse sweep: `last` and slots count - 2 .. 0 of seg, slot 0
// the run's first position.
EXPORT int group_probe_sweep(int tpl, int lanes, int threads, int held, int spread, int late_from,
                             int late_step, const double* seg, const double* last,
                             const double* mass, double* lam_r, double* lam_v, double* g_m,
                             int64_t n, double G, double dt, int64_t count, double* xbuf,
                             uint32_t* reg, void* stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (n < 1 || count < 2 || spread < 1) return 1;
    if (const int rc = hold(late_from, late_step, s)) return rc;
    nb::GroupVjpArgs A{};
    A.seg = seg;
    A.last = last;
    A.mass = mass;
    A.lam_r = lam_r;
    A.lam_v = lam_v;
    A.g_m = g_m;
    A.xbuf = xbuf;
    A.reg = reg;
    A.n = n;
    A.G = G;
    A.dt = dt;
    A.k1 = count - 2;
    A.count = count;
    A.first = 1;
    A.spread = spread;
    return nb::launch_group_vjp({tpl, lanes, threads, held != 0}, A, s) == hipSuccess ? 0 : 3;
}
