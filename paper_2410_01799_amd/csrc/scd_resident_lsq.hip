// The register-resident engine for least squares decompositions (Algorithm 6, Section 3.3 of arXiv 2410.01799): one launch
// finds one greedy cut of the remainder R = A - sum_j c_j s_j t_j^T.  The refit changes every coefficient with every
// term, so the remainder is formed anew at the start of a launch, in f64 and in the registers: a thread loads its tile of A
// and subtracts the terms from their sign bits (one multiply-add per entry and term), after which an alternation costs
// what it does for a greedy decomposition in f64, two exchanges, whatever the number of terms.
#include "scd_resident_kernel.h"

namespace scd {

// What the dispatch does with the kernel of a shape: launch it (st), or ask how many of its workgroups the device holds.
// All P x P must be resident at once (see launch_resident_k): the caller asks once, ahead of a call's launches.
struct LsqDo {
    const ResidentArgs* a;
    hipStream_t st;
    int room;
};

template <int TR, int TC, int P>
static hipError_t lsq_k(LsqDo& d)
{
    if (d.a) {
        hipLaunchKernelGGL((resident_kernel<double, double, double, TR, TC, P, true, true>), dim3(P * P), dim3(kResThreads), 0, d.st, *d.a);
        return hipGetLastError();
    }
    int dev = 0, per_cu = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, resident_kernel<double, double, double, TR, TC, P, true, true>,
                                                         kResThreads, 0);
    if (e == hipSuccess) d.room = per_cu > 0 ? cus : 0;  // (leases count one workgroup per compute unit)
    return e;
}

static hipError_t lsq_do(LsqDo& d, int64_t m, int64_t n)
{
    int p = 0, tr = 0, tc = 0;
    if (!resident_shape(SCD_F64, m, n, &p, &tr, &tc)) return hipErrorInvalidValue;
    return res_with_tile(p, tr, tc, [&](auto tile) {
        using Tile = decltype(tile);
        if constexpr (Tile::taken(SCD_F64, kResExact) || Tile::taken(SCD_F64, (int)ResSums::wide)) return lsq_k<Tile::TR, Tile::TC, Tile::P>(d);
        else return hipErrorInvalidValue;
    });
}

int resident_lsq_room(const int64_t* dims)
{
    LsqDo d = {nullptr, nullptr, 0};
    if (lsq_do(d, dims[0], dims[1]) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return d.room;
}

hipError_t launch_resident_lsq(const ResidentArgs& a, hipStream_t st)
{
    LsqDo d = {&a, st, 0};
    return lsq_do(d, a.m, a.n);
}

}  // namespace scd
