// Every size the register-resident engine takes has a form that is built, and every form that is built is some size's.
#include <cstdio>
#include <memory>

#include "scd_resident_shape.h"

using namespace scd;

int main()
{
    auto seen = std::make_unique<ResForms>();
    long taken = 0;
    for (int dt = 0; dt < 2; ++dt)
        for (int64_t m = 1; m <= 4100; ++m)
            for (int64_t n = 1; n <= 4100; ++n) {
                int p = 0, tr = 0, tc = 0;
                if (!resident_shape((scd_dtype)dt, m, n, &p, &tr, &tc)) continue;
                ++taken;
                if (dt == SCD_F64 && resident_sums(SCD_F64, m, n, 0.0) != ResSums::wide) {
                    std::printf("f64 %ld x %ld: two words a value\n", (long)m, (long)n);
                    return 1;
                }
                const bool grid = (p == 1 || p == 4 || p == 8 || p == 16) && (tr == 2 || tr == 4 || tr == 8) && (tc == 4 || tc == 8 || tc == 16);
                if (!grid || (int64_t)p * 32 * tr < m || (int64_t)p * 16 * tc < n || tr * tc > (dt == SCD_F32 ? 128 : 64)) {
                    std::printf("type %d %ld x %ld: grid %d tile %d x %d\n", dt, (long)m, (long)n, p, tr, tc);
                    return 1;
                }
                for (double fro : {0.0, 1e37}) {
                    const int f = resident_form((scd_dtype)dt, m, n, fro, p, tr, tc);
                    if (!kResForms.taken((scd_dtype)dt, f, p, tr, tc)) {
                        std::printf("type %d %ld x %ld: form %d of grid %d tile %d x %d is not built\n", dt, (long)m, (long)n, f, p, tr, tc);
                        return 1;
                    }
                    seen->at[dt][f][res_log2(p)][res_log2(tr)][res_log2(tc)] = true;
                }
            }
    int built = 0;
    for (int i = 0; i < (int)sizeof(ResForms); ++i) {
        built += ((const bool*)&kResForms)[i];
        if (((const bool*)&kResForms)[i] != ((const bool*)seen.get())[i]) {
            std::printf("form at %d is built and never taken\n", i);
            return 1;
        }
    }
    std::printf("%ld sizes, %d forms\n", taken, built);
    return 0;
}
