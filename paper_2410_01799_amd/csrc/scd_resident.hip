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

// The same with the words and reads of the register-resident engine, in groups of as many as it has: 256 f32 sums a workgroup, P
// neighbours.
template <int P>
__global__ void __launch_bounds__(kResThreads) resident_exchange_probe_kernel(uint64_t* buf, int rounds, int max_spin, unsigned* err, float* out)
{
    constexpr int N = 256;
    using Read = ResRead<float, N, P>;
    __shared__ float sum[N];
    __shared__ int fail;
    const int g = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(buf, 0, (int)((size_t)2 * gridDim.x * kResSlotWords * 8), 0x00027000);
    const uint32_t off = (uint32_t)(tid % Read::L * Read::H * kResSlotWords) * 8u + (uint32_t)(tid / Read::L) * 16u;
    if (tid < N) sum[tid] = 0.f;
    if (tid == 0) fail = 0;
    __syncthreads();
    for (uint32_t r = 1; r <= (uint32_t)rounds; ++r) {
        const uint32_t half = (r & 1u) * gridDim.x;
        if (tid < N / 2) res_publish(buf + (size_t)(half + g) * kResSlotWords + tid, sum[2 * tid] * 0.01f, sum[2 * tid + 1] * 0.01f + 1e-3f, exchange_tag(r));
        for (int d = 0; d < 16; ++d) __builtin_amdgcn_s_sleep(1);
        double s[Read::Q] = {}, x0, x1;
        int spin = 0;
        if (tid < Read::waves * 64) {
            if (!res_gather<float, Read::H, false, false>(buf, rs, (half + (uint32_t)(g / P * P)) * kResSlotWords * 8u, off, kResSlotWords * 8, true, 0, r, max_spin, s, x0,
                                               x1, spin))
                fail = 1;
            const double v = res_join<Read::L, Read::Q>(s, lane);
            if (tid % Read::L < Read::Q) sum[tid / Read::L * Read::Q + tid % Read::L] = (float)v;
        }
        __syncthreads();
        if (fail) {
            if (tid == 0) atomicExch(err, 1u);
            return;
        }
    }
    if (tid == 0) out[g] = sum[0];
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
    void (*resident)(uint64_t*, int, int, unsigned*, float*) = group == 4    ? resident_exchange_probe_kernel<4>
                                                               : group == 8  ? resident_exchange_probe_kernel<8>
                                                               : group == 16 ? resident_exchange_probe_kernel<16>
                                                                             : nullptr;
    if (which == 0 && resident)
        hipLaunchKernelGGL(resident, dim3(grid), dim3(kResThreads), 0, st, buf, rounds, max_spin, err, out);
    else if (which == 0)
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

// Exponent e such that a workgroup's sums, which are at most 16 ||R||_F, stay below 2^e, with `slack` more: what is
// exchanged is scaled by 2^-e.  No scaling up: a sum then keeps all its bits down to 2^-126 or 2^-1022 of that scale.
int resident_exponent(double fro, int slack)
{
    int e = 0;
    (void)frexp(16.0 * fro, &e);
    e += slack;
    return e > 0 ? e : 0;
}

int resident_sum_bytes(scd_dtype dt, const int64_t* dims, double fro)
{
    return resident_sums(dt, dims[0], dims[1], fro) == ResSums::wide ? 8 : 4;
}

// Sleep units between publishing and the first read, per exchange, from the option's value (default 16).  A read
// that comes before the last partner's words costs another trip to memory (0.4 us and its traffic), one that comes
// late costs what it waits, so the optimum is just behind the arrival, which moves with the words of an exchange and with
// what the slowest partner does before it publishes.  Rows (partners on all dies) need more than columns (one die).
// Measured in us per alternation at (rows / columns): up to 8 x 8 workgroups at 17 / 8 2.87 (512^2), 3.10 (1024^2), f64 3.23
// (600x400), 3.44 (1024^2), at 10 / 10 2.93, 3.18, f64 half a tenth more; 16 x 16 with at most 16 values a thread at 16 / 8 3.32
// (1501x999), at 20 / 8 3.42, f64 at 17 / 8 3.61, at 16 / 8 3.69; f32 beyond at 19 / 8 3.45 (2048^2), at 18 / 14 3.56, with 256
// columns a block at 19 / 11 4.34 (4096^2), 3.93 (1024x4096), at 18 / 8 4.62, 4.08; f64 at 23 / 8 4.03 (2048^2), at 16 / 8 4.21, with
// eight rows a thread at 23 / 9 4.89 (4096x2048), at 23 / 8 5.07, with 256 columns a block at 23 / 13 5.16 (2048x4096), at 22 / 8
// 5.41, and at 16 / 13 4.72 with two rows a thread (1024x4096), at 24 / 12 4.89.
void resident_poll_delays(scd_dtype dt, const int64_t* dims, double fro, int delay, int32_t* rows, int32_t* cols)
{
    int p = 16, tr = 8, tc = 16;
    (void)resident_shape(dt, dims[0], dims[1], &p, &tr, &tc);
    const ResSums sums = resident_sums(dt, dims[0], dims[1], fro);
    int u = delay + 1, v = delay - 8;
    if (p > 8 && sums == ResSums::wide) {
        u = tr * tc <= 16 ? delay + 1 : tr == 2 ? delay : delay + 7;
        if (tc == 16) v = delay - 3;
        if (tr == 8) v = delay - 7;
    } else if (p > 8) {
        u = tr * tc <= 16 ? delay : delay + 3;
        if (tc == 16 && sums == ResSums::plain) v = delay - 5;
    }
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
