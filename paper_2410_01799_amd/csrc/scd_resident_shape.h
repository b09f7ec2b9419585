// Which form of the register-resident engine takes a matrix (host arithmetic only).
#pragma once
#include <cstdint>
#include <initializer_list>

#include "scd.h"

namespace scd {

// Grid side P and thread tile TR x TC for an m x n matrix: the P x P workgroups of 32 x 16 threads cover
// P * 32 * TR rows and P * 16 * TC columns, at least the matrix (the overhang is kept as zeros).  Fewer
// workgroups mean fewer partners per exchange, more workgroups less arithmetic each; one workgroup exchanges nothing and
// takes what it can hold.  Beyond it, measured on the square sizes: 512 fastest with 8 values per thread on 8 x 8 workgroups,
// 1024 with 32 values on 8 x 8, 2048 with 32 values on 16 x 16, which gives the order of preference: the smallest grid of at
// most 8 x 8 with at most 8 values per thread, else the smallest grid with at most 32, else the grid that fits with
// the smallest tile.  Rows that are no multiple of 16 bytes are loaded and written back element by element, once per
// launch (1501x999, 16 terms: 2.4 ms a call; two launches per alternation on the unaligned rows took 8.7 ms).
constexpr bool resident_shape(scd_dtype dt, int64_t m, int64_t n, int* p, int* tr, int* tc)
{
    if (m < 1 || n < 4) return false;
    const int most = dt == SCD_F32 ? 128 : 64;  // values a thread can hold
    constexpr int grids[3] = {4, 8, 16};
    constexpr int trs[3] = {2, 4, 8}, tcs[3] = {4, 8, 16};
    // One workgroup, whatever a thread can hold (odd f32 rows: 64 values, which are widened in every phase): three barriers
    // an alternation instead of two exchanges.  Us per alternation, 4 x 4 workgroups / one: f32 64x64 3.15 / 1.07, 128x128
    // 3.01 / 1.31, 256x128 3.02 / 1.60, 192x192 2.97 / 2.40, 256x256 2.91 / 2.17; 61x67 3.69 / 1.43, 130x101 3.62 / 2.37,
    // 127x255 3.64 / 2.74; f64 128x128 3.56 / 1.47, 256x128 3.55 / 1.84, 127x255 3.59 / 2.28.
    {
        int r = 0, c = 0;
        for (int t : trs)
            if (!r && 32 * t >= m) r = t;
        for (int t : tcs)
            if (!c && 16 * t >= n) c = t;
        if (r && c && r * c <= (dt == SCD_F32 && n % 4 == 0 ? 128 : 64)) {
            *p = 1, *tr = r, *tc = c;
            return true;
        }
    }
    int best = -1, bp = 0, btr = 0, btc = 0;
    for (int pass = 0; pass < 2; ++pass) {
        for (int P : grids) {
            int r = 0, c = 0;
            for (int t : trs)
                if (!r && (int64_t)P * 32 * t >= m) r = t;
            for (int t : tcs)
                if (!c && (int64_t)P * 16 * t >= n) c = t;
            if (!r || !c || r * c > most) continue;
            if (P == 4 && (r > 4 || c > 8)) continue;  // (the 4 x 4 grid takes the small tiles only)
            if (pass == 0 ? (P <= 8 && r * c <= 8) : (r * c <= 32)) {
                *p = P, *tr = r, *tc = c;
                return true;
            }
            if (best < 0 || r * c < best) best = r * c, bp = P, btr = r, btc = c;
        }
    }
    if (best < 0) return false;
    *p = bp, *tr = btr, *tc = btc;
    return true;
}

// Types of the sums.  f64 matrices: f64 throughout.  f32 matrices whose rows are 16-byte steps: f32 inside a workgroup.
// The other f32 matrices come here from the launch stream, which adds across lanes, waves and workgroups in f64 after f32
// sums of ceil(n / 64) entries a lane (rows) and ceil(m / 256) rows a workgroup (columns): here f64 inside a workgroup, and
// f32 words where one rounding a workgroup is no more than those f32 sums cost, that is from two of them on each side
// (emulated, rms error of the row and column sums against f64, launch stream / here: 257x255 4.5e-8, 3.0e-8 / 2.6e-8,
// 2.7e-8; 1501x999 7.3e-8, 5.1e-8 / 2.4e-8, 2.5e-8; 4095x4093 1.5e-7, 7.8e-8 / 2.6e-8, 2.5e-8; with f32 sums inside the
// workgroup too the column sums of 1501x999 are off by 7.9e-8).  Smaller ones exchange f64, and so do those of any row
// length whose sums of up to 256 entries a workgroup could pass the largest f32: they are at most 16 ||R||_F.
// plain: the input's type (one workgroup: see the kernel), wide: f64 throughout.
enum class ResSums { plain, wide_inside, wide };
constexpr ResSums resident_sums(scd_dtype dt, int64_t m, int64_t n, double fro)
{
    if (dt == SCD_F64 || fro >= 1e36) return ResSums::wide;
    if (n % 4 == 0) return ResSums::plain;
    return m > 256 && n > 128 ? ResSums::wide_inside : ResSums::wide;
}

// The forms of the kernel that some matrix takes; no others are built.  The rules above change only where a side passes what a
// grid and tile cover and with the remainder of a row by 4 (256 rows and 128 columns are such sides), so the smallest sizes and
// those at and one or four past such a side stand for all.
constexpr int kResExact = 3;  // rows of 16-byte steps and a matrix that the grid covers without overhang (0 .. 2: ResSums, overhang)
constexpr int res_log2(int v) { return v <= 1 ? 0 : 1 + res_log2(v / 2); }
struct ResForms {
    bool at[2][4][5][4][5];  // [type][form][log2 P][log2 TR][log2 TC]
    constexpr bool taken(scd_dtype dt, int form, int p, int tr, int tc) const
    {
        return at[dt][form][res_log2(p)][res_log2(tr)][res_log2(tc)];
    }
};
constexpr int resident_form(scd_dtype dt, int64_t m, int64_t n, double fro, int p, int tr, int tc)
{
    if (p == 1) fro = 0.0;  // (nothing is exchanged)
    const ResSums sums = resident_sums(dt, m, n, fro);
    return m == (int64_t)p * 32 * tr && n == (int64_t)p * 16 * tc && (dt == SCD_F64 || sums == ResSums::plain) ? kResExact : (int)sums;
}
constexpr ResForms res_forms()
{
    constexpr int sides[4] = {1, 4, 8, 16}, tiles[3] = {2, 4, 8};
    ResForms f = {};
    for (int dt = 0; dt < 2; ++dt)
        for (int i = 0; i < 25; ++i)
            for (int k = 0; k < 39; ++k) {
                const int64_t m = i == 24 ? 1 : 32 * tiles[i / 2 % 3] * sides[i / 6] + i % 2;
                const int64_t n = (k >= 36 ? 4 : 32 * tiles[k / 3 % 3] * sides[k / 9]) + (k % 3 == 2 ? 4 : k % 3);
                int p = 0, tr = 0, tc = 0;
                if (!resident_shape((scd_dtype)dt, m, n, &p, &tr, &tc)) continue;
                for (double fro : {0.0, 1e37})
                    f.at[dt][resident_form((scd_dtype)dt, m, n, fro, p, tr, tc)][res_log2(p)][res_log2(tr)][res_log2(tc)] = true;
            }
    return f;
}
inline constexpr ResForms kResForms = res_forms();
static_assert(SCD_F32 == 0 && SCD_F64 == 1, "index of the type");

}  // namespace scd
