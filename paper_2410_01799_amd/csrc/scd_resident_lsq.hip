// The register-resident engine for least squares decompositions (Algorithm 6, Section 3.3 of arXiv 2410.01799): one launch
// finds one greedy cut of the remainder R = A - sum_j c_j s_j t_j^T.  The refit changes every coefficient with every
// term, so the remainder is formed anew at the start of a launch, in f64 and in the registers: a thread loads its tile of A
// and subtracts the terms from their sign bits (one add and one xor per entry and term), after which an alternation costs
// what it does for a greedy decomposition in f64, two exchanges, whatever the number of terms.
#include "scd_resident_kernel.h"

namespace scd {

template <int TR, int TC, int P>
static hipError_t launch_lsq_k(const ResidentArgs& a, hipStream_t st)
{
    // all P x P workgroups at once, as in launch_resident_k
    int dev = 0, per_cu = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, resident_kernel<double, double, double, TR, TC, P, true, true>,
                                                         kResThreads, 0);
    if (e != hipSuccess) return e;
    if ((int64_t)per_cu * cus < P * P) return hipErrorCooperativeLaunchTooLarge;
    hipLaunchKernelGGL((resident_kernel<double, double, double, TR, TC, P, true, true>), dim3(P * P), dim3(kResThreads), 0, st, a);
    return hipGetLastError();
}

template <int P>
static hipError_t launch_lsq_p(const ResidentArgs& a, int tr, int tc, hipStream_t st)
{
    const int key = tr * 100 + tc;
    switch (key) {
        case 204: return launch_lsq_k<2, 4, P>(a, st);
        case 208: return launch_lsq_k<2, 8, P>(a, st);
        case 404: return launch_lsq_k<4, 4, P>(a, st);
        case 408: return launch_lsq_k<4, 8, P>(a, st);
        default: break;
    }
    if constexpr (P >= 8 || P == 1) {
        switch (key) {
            case 216: return launch_lsq_k<2, 16, P>(a, st);
            case 416: return launch_lsq_k<4, 16, P>(a, st);
            case 804: return launch_lsq_k<8, 4, P>(a, st);
            case 808: return launch_lsq_k<8, 8, P>(a, st);
            default: break;
        }
    }
    return hipErrorInvalidValue;
}

hipError_t launch_resident_lsq(const ResidentArgs& a, hipStream_t st)
{
    int p = 0, tr = 0, tc = 0;
    if (!resident_shape(SCD_F64, a.m, a.n, &p, &tr, &tc)) return hipErrorInvalidValue;
    if (p == 16) return launch_lsq_p<16>(a, tr, tc, st);
    if (p == 8) return launch_lsq_p<8>(a, tr, tc, st);
    if (p == 1) return launch_lsq_p<1>(a, tr, tc, st);
    return launch_lsq_p<4>(a, tr, tc, st);
}

}  // namespace scd
