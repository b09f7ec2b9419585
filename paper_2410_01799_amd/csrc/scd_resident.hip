// Probes of workgroup-to-workgroup exchange latency inside one persistent launch (measurement only).
#include "scd_resident_kernel.h"

namespace scd {

__device__ __forceinline__ uint64_t tagged(float v, uint32_t tag)
{
    return ((uint64_t)tag << 32) | (uint64_t)__float_as_uint(v);
}

// Every workgroup publishes 256 tagged values per round and reads those of the `group` workgroups
// it shares a group with; value and tag travel in one 8-byte store, so the data is its own flag.
__global__ void __launch_bounds__(256) exchange_probe_kernel(uint64_t* buf, int rounds, int group, int max_spin,
                                                            unsigned* err, float* out)
{
    const int g = blockIdx.x, tid = threadIdx.x;
    const int nvals = (group >> 16) ? (group >> 16) : 256;  // values each workgroup publishes per round
    group &= 0xFFFF;
    const int g0 = (g / group) * group;
    float carry = 0.f;
    if (tid >= nvals) return;
    for (int r = 1; r <= rounds; ++r) {
        uint64_t* mine = buf + ((size_t)(r & 1) * gridDim.x + g) * 256;
        __hip_atomic_store(mine + tid, tagged(carry + (float)tid, (uint32_t)r), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        float s = 0.f;
        for (int q0 = 0; q0 < group; q0 += 16) {
            // all loads of a batch of 16 members are in flight together; stale ones are retried
            uint64_t w[16];
            const int nq = group - q0 < 16 ? group - q0 : 16;
            unsigned pending = (nq == 16) ? 0xFFFFu : ((1u << nq) - 1u);
            int spin = 0;
            while (pending) {
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const uint64_t* theirs = buf + ((size_t)(r & 1) * gridDim.x + g0 + q0 + (q < nq ? q : 0)) * 256;
                    if ((pending >> q) & 1u)
                        w[q] = __hip_atomic_load(theirs + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
                for (int q = 0; q < 16; ++q)
                    if (((pending >> q) & 1u) && (uint32_t)(w[q] >> 32) == (uint32_t)r) pending &= ~(1u << q);
                if (pending && ++spin > max_spin) {
                    atomicExch(err, 1u);
                    return;
                }
            }
#pragma unroll
            for (int q = 0; q < 16; ++q)
                if (q < nq) s += __uint_as_float((uint32_t)w[q]);
        }
        carry = s * 1e-3f;
    }
    if (tid == 0) out[g] = carry;
}

// Classic counter barrier over the whole grid, for comparison.
__global__ void __launch_bounds__(256) barrier_probe_kernel(unsigned* counter, int rounds, int max_spin, unsigned* err,
                                                           float* out)
{
    unsigned target = 0;
    for (int r = 1; r <= rounds; ++r) {
        __syncthreads();
        if (threadIdx.x == 0) {
            __threadfence();
            __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            target += gridDim.x;
            int spin = 0;
            while (__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
                if (++spin > max_spin) {
                    atomicExch(err, 1u);
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            __threadfence();
        }
        __syncthreads();
        if (*(volatile unsigned*)err) return;
    }
    if (threadIdx.x == 0) out[blockIdx.x] = (float)target;
}

hipError_t launch_exchange_probe(int which, int grid, uint64_t* buf, unsigned* counter, int rounds, int group,
                                 int max_spin, unsigned* err, float* out, hipStream_t st)
{
    if (which == 0)
        hipLaunchKernelGGL(exchange_probe_kernel, dim3(grid), dim3(256), 0, st, buf, rounds, group, max_spin, err, out);
    else
        hipLaunchKernelGGL(barrier_probe_kernel, dim3(grid), dim3(256), 0, st, counter, rounds, max_spin, err, out);
    return hipGetLastError();
}

bool resident_supported(scd_dtype dt, int order, const int64_t* dims)
{
    int p, tr, tc;
    return order == 2 && resident_shape(dt, dims[0], dims[1], &p, &tr, &tc);
}

int resident_workgroups(scd_dtype dt, const int64_t* dims)
{
    int p = 0, tr, tc;
    return resident_shape(dt, dims[0], dims[1], &p, &tr, &tc) ? p * p : 0;
}

// Sleep units between publishing and the first read, per exchange, from the option's value (default 16).  A read
// that comes before the last partner's words costs another trip to memory (0.4 us and its traffic), one that comes
// late costs what it waits, so the optimum is just behind the arrival, which moves with the words of an exchange.
// Measured in us per alternation: grids of up to 8 x 8 at 10 units 2.87 (256^2) and 3.41 (1024^2), at 16 3.17 and
// 3.70; 16 x 16 with slots of 256 columns at 18 / 14 units (rows / columns) 5.38 (4096^2), at 16 / 16 5.44, at
// 12 / 8 5.84; with shorter slots at 16 / 8 4.55 (2048^2) and 4.95 (4096x1024), at 16 / 16 4.69 and 5.14.
// f64 has twice the words: up to 8 x 8 at 10 / 10 3.40 (256^2), 4.55 (600x400) and 4.78 (1024^2), at 18 / 14 3.66, 4.71
// and 4.81; 16 x 16 at 22 / 18 6.78 (1501x999) and 6.93 (2048^2), at 18 / 14 7.03 and 7.24, at 26 / 22 6.95 and 7.09; with
// column slots of 256 values at 26 / 22 7.68 (2048x4096), at 22 / 18 8.56.  f64 sums inside a workgroup make the slots of
// tall blocks later: three units more, 5.50 instead of 5.99 (3000x1999) and 6.77 instead of 7.40 (4095x4093).
void resident_poll_delays(scd_dtype dt, const int64_t* dims, double fro, int delay, int32_t* rows, int32_t* cols)
{
    int p = 16, tr = 8, tc = 16;
    (void)resident_shape(dt, dims[0], dims[1], &p, &tr, &tc);
    int u = delay - 6, v = delay - 6;
    const ResSums sums = resident_sums(dt, dims[0], dims[1], fro);
    const bool wide = sums == ResSums::wide;  // twice the words
    if (sums == ResSums::wide_inside && p > 8 && tr > 2) delay = delay ? delay + 3 : 0;
    if (p > 8 && !wide) u = delay + 2, v = tc == 16 ? delay - 2 : delay - 8;
    if (p > 8 && wide) u = tc == 16 ? delay + 10 : delay + 6, v = tc == 16 ? delay + 6 : delay + 2;
    *rows = delay == 0 || u < 0 ? 0 : u;
    *cols = delay == 0 || v < 0 ? 0 : v;
}

template <typename TE, typename TA, typename TX, int TR, int TC, int P, bool PAD>
static hipError_t launch_resident_k(const ResidentArgs& a, hipStream_t st)
{
    // All P x P workgroups must be resident at once.  One workgroup of 512 threads fits every compute
    // unit (checked here against the occupancy the runtime reports); an ordinary launch on an idle
    // device then places them all, and every wait in the kernel is bounded in case it does not.
    int dev = 0, per_cu = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, resident_kernel<TE, TA, TX, TR, TC, P, PAD>, kResThreads, 0);
    if (e != hipSuccess) return e;
    if ((int64_t)per_cu * cus < P * P) return hipErrorCooperativeLaunchTooLarge;
    hipLaunchKernelGGL((resident_kernel<TE, TA, TX, TR, TC, P, PAD>), dim3(P * P), dim3(kResThreads), 0, st, a);
    return hipGetLastError();
}

template <typename TE, typename Tile>
static hipError_t launch_resident_t(const ResidentArgs& a, hipStream_t st)
{
    constexpr scd_dtype dt = sizeof(TE) == 4 ? SCD_F32 : SCD_F64;
    constexpr int P = Tile::P, TR = Tile::TR, TC = Tile::TC;
    // one workgroup: f32 sums inside a thread (columns: a wave), f64 beyond; in f32 rows that are no 16-byte steps f64 from
    // the first addition
    using TA = std::conditional_t<P == 1, double, TE>;
    const int form = resident_form(dt, a.m, a.n, a.fro, P, TR, TC);
    if constexpr (Tile::taken(dt, kResExact)) {
        if (form == kResExact) return launch_resident_k<TE, TA, TE, TR, TC, P, false>(a, st);
    }
    if constexpr (Tile::taken(dt, (int)ResSums::plain)) {
        if (form == (int)ResSums::plain) return launch_resident_k<TE, TA, TE, TR, TC, P, true>(a, st);
    }
    if constexpr (Tile::taken(dt, (int)ResSums::wide_inside)) {
        if (form == (int)ResSums::wide_inside) return launch_resident_k<TE, double, TE, TR, TC, P, true>(a, st);
    }
    if constexpr (Tile::taken(dt, (int)ResSums::wide)) {
        if (form == (int)ResSums::wide) return launch_resident_k<TE, double, double, TR, TC, P, true>(a, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_resident(const ResidentArgs& a, scd_dtype dt, hipStream_t st)
{
    int p = 0, tr = 0, tc = 0;
    if (!resident_shape(dt, a.m, a.n, &p, &tr, &tc)) return hipErrorInvalidValue;
    return res_with_tile(p, tr, tc, [&](auto tile) {
        return dt == SCD_F32 ? launch_resident_t<float, decltype(tile)>(a, st) : launch_resident_t<double, decltype(tile)>(a, st);
    });
}

}  // namespace scd
