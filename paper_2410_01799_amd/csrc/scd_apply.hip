// Product of a signed cut decomposition with a vector, straight from the packed factors
// (Section 6.1 of arXiv 2410.01799, Question A):
//     y = (sum_j c_j s_j t_j^T) x = sum_j z_j s_j,    z_j = c_j <t_j, x>.
// The matrix is never expanded: the kernels read the w (m + n) / 8 bytes of sign bits, once per group of vectors.
//
// f32: both passes are contractions of a +-1 matrix with a vector and run on the matrix cores in block
// fixed point (see the two MFMA kernels).  f64: vector units; a wave owns 64 consecutive entries (one per
// lane), takes a 64-bit word of sign bits that is the same for all its lanes (fetched by one lane,
// broadcast through a scalar register), turns bit `lane` into a multiplier +-1.0 and adds with one fused
// multiply-add in f64 (the product with +-1 is exact, so each step rounds like the sign-flip-and-add of
// Section 3.4).
//   inner pass  <t_j, x> per chunk of 4096 entries
//   outer pass  z_j = c_j * (sum of the chunk parts, in order) is formed on the way in; per split of the
//               terms, y_i = sum_j +-z_j
//   reduce      y = sum of the splits, in order, rounded once to the output type
// Every sum has a fixed order: results are bit-identical from run to run.
#include "scd_bits.h"
#include "scd_device.h"

namespace scd {

namespace {

constexpr int kApChunkWords = 64;   // words of sign bits per lane-resident chunk of x (4096 entries)
constexpr int kApInnerWaves = 4;    // waves per workgroup of the inner pass
constexpr int kApOuterWaves = 8;    // waves per workgroup of the outer pass: 8 adjacent words = one 64-byte line

// Cross-lane steps without LDS traffic (a chain of ds_bpermute costs an LDS round trip per step): the value
// of lane (l ^ D) for D = 1, 2, 4, 8 by the data-parallel lane modes (4 = mirror of half a row then reversed
// quads, 8 = mirror of a row then of half a row); the two partners at distance 16 or 32 by the row-swap
// instructions of gfx950 (swapping the odd rows of one copy with the even rows of another leaves them in the
// two results, in the same order for both partners).
template <int D>
__device__ __forceinline__ uint32_t ap_dpp_xor(uint32_t v)
{
    static_assert(D == 1 || D == 2 || D == 4 || D == 8, "distance within a row of 16 lanes");
    constexpr int c0 = D == 1 ? 0xB1 : D == 2 ? 0x4E : D == 4 ? 0x141 : 0x140;
    constexpr int c1 = D == 4 ? 0x1B : D == 8 ? 0x141 : 0;
    int r = __builtin_amdgcn_update_dpp(0, (int)v, c0, 0xF, 0xF, true);
    if constexpr (c1 != 0) r = __builtin_amdgcn_update_dpp(0, r, c1, 0xF, 0xF, true);
    return (uint32_t)r;
}
template <int D>
__device__ __forceinline__ double ap_dpp_xor_f64(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const uint32_t lo = ap_dpp_xor<D>((uint32_t)b), hi = ap_dpp_xor<D>((uint32_t)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <int D>
__device__ __forceinline__ void ap_swap_pair_f64(double v, double& a, double& b)
{
    const unsigned long long w = (unsigned long long)__double_as_longlong(v);
    uint32_t la, lb, ha, hb;
    swap_pair<D>((uint32_t)w, la, lb);
    swap_pair<D>((uint32_t)(w >> 32), ha, hb);
    a = __longlong_as_double((long long)(((unsigned long long)ha << 32) | la));
    b = __longlong_as_double((long long)(((unsigned long long)hb << 32) | lb));
}

__device__ __forceinline__ double ap_wave_sum(double a)
{
    a += ap_dpp_xor_f64<1>(a);
    a += ap_dpp_xor_f64<2>(a);
    a += ap_dpp_xor_f64<4>(a);
    a += ap_dpp_xor_f64<8>(a);
    double p, q;
    ap_swap_pair_f64<16>(a, p, q);
    a = p + q;
    ap_swap_pair_f64<32>(a, p, q);
    return p + q;
}
__device__ __forceinline__ double ap_wave_max(double a)
{
    a = fmax(a, ap_dpp_xor_f64<1>(a));
    a = fmax(a, ap_dpp_xor_f64<2>(a));
    a = fmax(a, ap_dpp_xor_f64<4>(a));
    a = fmax(a, ap_dpp_xor_f64<8>(a));
    double p, q;
    ap_swap_pair_f64<16>(a, p, q);
    a = fmax(p, q);
    ap_swap_pair_f64<32>(a, p, q);
    return fmax(p, q);
}
__device__ __forceinline__ float ap_wave_max(float a)
{
    a = fmaxf(a, __uint_as_float(ap_dpp_xor<1>(__float_as_uint(a))));
    a = fmaxf(a, __uint_as_float(ap_dpp_xor<2>(__float_as_uint(a))));
    a = fmaxf(a, __uint_as_float(ap_dpp_xor<4>(__float_as_uint(a))));
    a = fmaxf(a, __uint_as_float(ap_dpp_xor<8>(__float_as_uint(a))));
    uint32_t p, q;
    swap_pair<16>(__float_as_uint(a), p, q);
    a = fmaxf(__uint_as_float(p), __uint_as_float(q));
    swap_pair<32>(__float_as_uint(a), p, q);
    return fmaxf(__uint_as_float(p), __uint_as_float(q));
}

// +-1.0 for lane `lane` from bit `lane` of a wave-uniform word (a 1 bit stands for -1)
__device__ __forceinline__ double ap_sign(uint64_t word)
{
    const int hi = __builtin_amdgcn_inverse_ballot_w64(word) ? (int)0xBFF00000 : (int)0x3FF00000;
    return __hiloint2double(hi, 0);
}

// word `p` of a lane-distributed row of sign bits (lane p holds word p), as a wave-uniform value
__device__ __forceinline__ uint64_t ap_word(uint64_t lane_word, int p)
{
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)lane_word, p);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(lane_word >> 32), p);
    return ((uint64_t)hi << 32) | lo;
}

constexpr int kApDepth = 4;  // rows of sign bits in flight per wave

template <typename TE>
__global__ void __launch_bounds__(kApInnerWaves* kWave)
    apply_inner_kernel(const uint64_t* __restrict__ bits, int64_t nw, int64_t w, const TE* __restrict__ x, int64_t n,
                       double* __restrict__ part, int terms_per_wave)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t chunk = blockIdx.y;
    const int64_t p0 = chunk * kApChunkWords;
    const int nwc = (int)(nw - p0 < kApChunkWords ? nw - p0 : kApChunkWords);  // words of this chunk
    double xr[kApChunkWords];
#pragma unroll
    for (int p = 0; p < kApChunkWords; ++p) {
        // unconditional loads (all in flight together); entries past the end count as zero
        const int64_t l = (p0 + p) * 64 + lane;
        const TE v = x[l < n ? l : n - 1];
        xr[p] = l < n ? (double)v : 0.0;
    }
    const int64_t j0 = ((int64_t)blockIdx.x * kApInnerWaves + wv) * terms_per_wave;
    const int64_t j1 = j0 + terms_per_wave < w ? j0 + terms_per_wave : w;
    if (j0 >= j1) return;
    // Lane p fetches word p of a term's row (one coalesced load per term), kApDepth terms ahead.  Loads
    // are unconditional: terms past the end re-read the last one, lanes past the end of the row read its
    // first word (the entries of x there are zero, so any valid word will do).
    const int64_t lw = p0 + (lane < nwc ? lane : 0);
    uint64_t buf[kApDepth];
#pragma unroll
    for (int d = 0; d < kApDepth; ++d) {
        const int64_t jn = j0 + d < j1 ? j0 + d : j1 - 1;
        buf[d] = bits[jn * nw + lw];
    }
    for (int64_t j = j0; j < j1; j += kApDepth) {
#pragma unroll
        for (int d = 0; d < kApDepth; ++d) {
            const uint64_t row = buf[d];
            const int64_t jn = j + kApDepth + d < j1 ? j + kApDepth + d : j1 - 1;
            buf[d] = bits[jn * nw + lw];
            if (j + d < j1) {
                // four independent chains: a dependent f64 add would wait for the one before it
                double a4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int p = 0; p < kApChunkWords; ++p) a4[p & 3] = __builtin_fma(xr[p], ap_sign(ap_word(row, p)), a4[p & 3]);
                double acc = (a4[0] + a4[1]) + (a4[2] + a4[3]);
                acc = ap_wave_sum(acc);
                if (lane == 0) part[chunk * w + j + d] = acc;
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------
// Inner pass on the matrix cores (f32 x).  <t_j, x> for many terms j is a dense contraction of a +-1
// matrix with x, so it belongs on MFMA; what keeps it exact is fixed point.  Per chunk of 4096 entries
// x is scaled by a power of two so that |x| 2^s < 2^30, rounded to integers and cut into four balanced
// base-256 digits (int8).  The only rounding is the fixed point itself: at most max|x| 2^-30 per entry of the
// chunk, below the resolution of the f32 input for all but entries more than 64 times smaller than the largest.
// v_mfma_i32_16x16x64_i8 takes 16 terms x 64 entries of sign bits (as bytes 0 / 1) against the digits of up to four
// vectors (16 columns); <t, x> = sum x - 2 sum over the -1 signs, exact in integers, the digits recombined in f64.
// The order of the contraction index is free as long as both operands share it, and is chosen for the bits: lane
// (term, kq) reads words 2 kq and 2 kq + 1 of eight neighbouring words of its term (64 bytes per term and load), and
// byte b of operand dword q of its instruction k = 0..7 is bit k + 8 b of half word q of the two: a mask, and for odd k a shift.
// (With v_mfma_i32_4x4x4_16B_i8 and a table look-up per nibble the pass used a quarter of the instruction's columns for one
// vector and took them one after the other: 14336x4096 transposed, four vectors, 4 x 30 us.)
typedef int ap_int4 __attribute__((ext_vector_type(4)));

// a barrier for what goes through LDS: loads stay on their way
__device__ __forceinline__ void ap_lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

constexpr int kApMfmaWaves = 8;                      // waves per workgroup of the outer pass: one word of outputs each
constexpr int kApFxRows = 4, kApFxQuarters = 4;      // waves of the inner pass: 16 terms, a quarter of the chunk each
constexpr int kApFxWaves = kApFxRows * kApFxQuarters;
constexpr int kApFxThreads = kApFxWaves * kWave;     // one dword of the fixed point per thread and digit
constexpr int kApFxTile = 16 * kApFxRows;            // terms per workgroup and turn
constexpr int kApInnerGrid = 256;                    // most workgroups of the inner pass
static_assert(kApFxThreads == kApChunkWords * 16, "a thread per four entries of the chunk");

// four integers |q| < 2^30 -> digit jd of each as one dword per digit.  With 128 added to each of the three lower digits they
// are the bytes of q + 128 (1 + 256 + 65536), and flipping the top bit of a byte takes the 128 off again.
__device__ __forceinline__ void ap_digits(const int (&q4)[4], uint32_t (&dig)[4])
{
    uint32_t r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = ((uint32_t)q4[k] + 0x00808080u) ^ 0x00808080u;
    const uint32_t t0 = __builtin_amdgcn_perm(r[1], r[0], 0x05010400u), t1 = __builtin_amdgcn_perm(r[1], r[0], 0x07030602u);
    const uint32_t u0 = __builtin_amdgcn_perm(r[3], r[2], 0x05010400u), u1 = __builtin_amdgcn_perm(r[3], r[2], 0x07030602u);
    dig[0] = __builtin_amdgcn_perm(u0, t0, 0x05040100u);
    dig[1] = __builtin_amdgcn_perm(u0, t0, 0x07060302u);
    dig[2] = __builtin_amdgcn_perm(u1, t1, 0x05040100u);
    dig[3] = __builtin_amdgcn_perm(u1, t1, 0x07060302u);
}

// part[v * pstride + chunk * w + j] = <t_j, x_v> restricted to the chunk, for nv <= NV vectors.
//
// Vector instructions bound the pass, not bits or matrix cores.  Sixteen waves form the fixed point of a workgroup once,
// four entries a thread and vector, and share the contraction: wave (r, k) takes 16 terms and a quarter of the chunk.  The
// quarters' integers are added through LDS (exact, so the split changes no bit), by the four waves of a row for one register
// each.  Half of the sign bytes need no shift: bit 2 c of a byte counts 4^c in an accumulator of its own.  sum x comes from the
// matrix cores too, as a term of 1 bits.  The bits of the next two tiles are on their way meanwhile; with one tile per workgroup
// (ONE) there are none, and asking for it again would cost two microseconds (9.2 and 6.9).  Us a launch, with four waves that
// each took whole rows, a shift and a mask for every four signs, the digits cut one after the other and f64 sums / now:
// 14336x4096 transposed to 25442 terms, four vectors 32.6 / 25.0, 4096x4096 to 16320, one vector 8.5 / 6.9.
template <int NV, bool ONE>
__global__ void __launch_bounds__(kApFxThreads)
    apply_inner_fx_kernel(const uint64_t* __restrict__ bits, int64_t nw, int64_t w, const float* __restrict__ x, int nv, int64_t n,
                          double* __restrict__ part, int64_t pstride, int tiles_per_wg)
{
    constexpr int NC = 4 * NV;  // columns in use
    constexpr int kAhead = 3;   // tiles whose bits are held or requested
    __shared__ __align__(16) uint32_t xd[kApChunkWords * 4 * NC * 4];  // [8 words][bit of a byte][kq][column ^ bit][dword]
    __shared__ int quarter[2][4][kApFxWaves][kWave];                  // [turn][register][wave][lane]
    __shared__ int total_of[kApFxQuarters][kWave];
    __shared__ uint32_t most[NV];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wr = wv & (kApFxRows - 1), wk = wv / kApFxRows;
    const int64_t chunk = blockIdx.y;
    const int64_t p0 = chunk * kApChunkWords;
    const int nwc = (int)(nw - p0 < kApChunkWords ? nw - p0 : kApChunkWords);
    const int ngrp = (nwc + 7) / 8;
    const int row = lane & 15, kq = lane >> 4;
    const int64_t tile0 = (int64_t)blockIdx.x * tiles_per_wg, last0 = w > kApFxTile ? w - kApFxTile : 0;

    // ---- fixed point of this chunk: thread t owns dword t (word, half, d): entries d + 8 b of the half word
    if (tid < NV) most[tid] = 0u;
    float xv[NV][4];
    const int64_t l0 = p0 * 64 + (tid >> 4) * 64 + ((tid >> 3) & 1) * 32 + (tid & 7);
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int64_t l = l0 + 8 * b;
            const float val = x[(int64_t)(v < nv ? v : nv - 1) * n + (l < n ? l : n - 1)];
            xv[v][b] = l < n ? val : 0.f;
        }
    // The sign bits of the first tiles are requested before x is waited for (no barrier here waits for loads): their latency
    // hides behind the fixed point.  A tile that would pass the last term starts 64 terms before it.
    const uint64_t* from[2][2];
    {
        const int local = wr * 16 + row;
        const uint64_t* r = bits + (local < w ? local : w - 1) * nw + p0;
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const int gg = 2 * wk + g;
            const int q = (gg < ngrp ? gg : 0) * 8 + 2 * kq;  // (words past the end meet digits that are zero)
            from[g][0] = r + (q < nwc ? q : nwc - 1);
            from[g][1] = r + (q + 1 < nwc ? q + 1 : nwc - 1);
        }
    }
    auto first_term = [&](int64_t tile) { return tile * kApFxTile < last0 ? tile * kApFxTile : last0; };
    uint64_t wbuf[kAhead][2][2];
    auto fetch = [&](int64_t tile, uint64_t (&to)[2][2]) {
        // (unconditional, else the compiler waits for them where the paths meet)
        const int64_t off = first_term(tile < tile0 + tiles_per_wg ? tile : tile0 + tiles_per_wg - 1) * nw;
#pragma unroll
        for (int g = 0; g < 2; ++g) to[g][0] = from[g][0][off], to[g][1] = from[g][1][off];
    };
#pragma unroll
    for (int a = 0; a < (ONE ? 1 : kAhead - 1); ++a) fetch(tile0 + a, wbuf[a]);
    ap_lds_barrier();
    // the largest |x|, by its bits: those of infinities and NaNs lie above
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        if (v >= nv) continue;
        uint32_t m = 0u;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const uint32_t u = __float_as_uint(xv[v][b]) & 0x7FFFFFFFu;
            m = u > m ? u : m;
        }
        auto join = [&](uint32_t o) { m = o > m ? o : m; };
        join(ap_dpp_xor<1>(m));
        join(ap_dpp_xor<2>(m));
        join(ap_dpp_xor<4>(m));
        join(ap_dpp_xor<8>(m));
        if (row == 0) atomicMax(&most[v], m);
    }
    ap_lds_barrier();
    const uint32_t finite_most = __float_as_uint(3.0e38f);
    const int wd = tid >> 4, hd = tid & 7;
    uint32_t* dst = xd + (((wd >> 3) * 8 + hd) * 4 + ((wd & 7) >> 1)) * NC * 4 + (wd & 1) * 2 + ((tid >> 3) & 1);
    int shift[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        shift[v] = 0;
        if (v >= nv) continue;  // (the columns of vectors past nv hold what they hold and are not stored)
        const uint32_t am = most[v];
        const bool finite = am <= finite_most;
        shift[v] = 30 - __builtin_amdgcn_frexp_expf(__uint_as_float(am));  // |x| < 2^(30 - shift); exponent 0 for zero
        int q4[4];
        uint32_t dig[4];
        // (scaled in f32: exact but for values that are zero once rounded)
#pragma unroll
        for (int b = 0; b < 4; ++b) q4[b] = finite ? (int)rintf(__builtin_amdgcn_ldexpf(xv[v][b], shift[v])) : 0;
        ap_digits(q4, dig);
#pragma unroll
        for (int jd = 0; jd < 4; ++jd) dst[((4 * v + jd) ^ (hd & (NC - 1))) * 4] = dig[jd];
    }
    ap_lds_barrier();
    // this lane's column: digit jd of vector vc
    const int col = row & (NC - 1), jd = lane & 3, vc = col >> 2;
    int sh = 0;
#pragma unroll
    for (int v = 0; v < NV; ++v)
        if (v == vc) sh = shift[v];
    const bool fin = most[vc] <= finite_most;
    // the digits' weight in units of x
    const double weight = fin ? __hiloint2double((1023 + 8 * jd - sh) << 20, 0) : __longlong_as_double(0x7FF8000000000000ll);
    const ap_int4* xb[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) xb[k] = (const ap_int4*)xd + (2 * wk * 8 + k) * 4 * NC + kq * NC + (col ^ (k & (NC - 1)));
    if (wr == 0) {
        ap_int4 acc = {0, 0, 0, 0};
        const ap_int4 ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
#pragma unroll
        for (int g = 0; g < 2; ++g)
            if (2 * wk + g < ngrp)
#pragma unroll
                for (int k = 0; k < 8; ++k) acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(ones, xb[k][g * 8 * 4 * NC], acc, 0, 0, 0);
        total_of[wk][lane] = acc[0];  // (all rows are the same)
    }
    ap_lds_barrier();
    int total = 0;
#pragma unroll
    for (int k = 0; k < kApFxQuarters; ++k) total += total_of[k][lane];
    double* mypart = part + (int64_t)vc * pstride + chunk * w;
    const int local = wr * 16 + 4 * kq + wk;  // register wk of this lane: the term, column lane mod 16
    const bool store = jd == 0 && row < NC && vc < nv && local < w;
    auto turn = [&](int t0, uint64_t (&mine)[2][2], uint64_t (&next)[2][2]) {
        if constexpr (!ONE) fetch(tile0 + t0 + kAhead - 1, next);
        ap_int4 acc[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] = ap_int4{0, 0, 0, 0};
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            if (2 * wk + g < ngrp) {
                const uint32_t d4[4] = {(uint32_t)mine[g][0], (uint32_t)(mine[g][0] >> 32), (uint32_t)mine[g][1], (uint32_t)(mine[g][1] >> 32)};
#pragma unroll
                for (int odd = 0; odd < 2; ++odd)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        ap_int4 A;
#pragma unroll
                        for (int q = 0; q < 4; ++q) A[q] = (int)((d4[q] >> odd) & (0x01010101u << (2 * c)));
                        acc[c] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A, xb[2 * c + odd][g * 8 * 4 * NC], acc[c], 0, 0, 0);
                    }
            }
        }
        int(*mail)[kApFxWaves][kWave] = quarter[t0 & 1];
#pragma unroll
        for (int i = 0; i < 4; ++i) mail[i][wv][lane] = ((acc[0][i] * 4 + acc[1][i]) * 4 + acc[2][i]) * 4 + acc[3][i];
        ap_lds_barrier();
        int sum = 0;
#pragma unroll
        for (int k = 0; k < kApFxQuarters; ++k) sum += mail[wk][k * kApFxRows + wr][lane];
        // recombine the digits: exact in f64
        double v = (double)(total - 2 * (sum >> 6)) * weight;
        v += ap_dpp_xor_f64<1>(v);
        v += ap_dpp_xor_f64<2>(v);
        const int64_t j = first_term(tile0 + t0) + local;
        if (store && j >= (tile0 + t0) * kApFxTile) mypart[j] = v;
    };
    static_assert(kAhead == 3, "the turns below");
    if constexpr (ONE) {
        turn(0, wbuf[0], wbuf[1]);
        return;
    }
    for (int t0 = 0; t0 < tiles_per_wg; t0 += kAhead) {
        if ((tile0 + t0) * kApFxTile >= w) break;
        turn(t0, wbuf[0], wbuf[2]);
        if (t0 + 1 >= tiles_per_wg || (tile0 + t0 + 1) * kApFxTile >= w) break;
        turn(t0 + 1, wbuf[1], wbuf[0]);
        if (t0 + 2 >= tiles_per_wg || (tile0 + t0 + 2) * kApFxTile >= w) break;
        turn(t0 + 2, wbuf[2], wbuf[1]);
    }
}

// sum over the chunks of <t_j, x>, in order; four loads in flight at a time (a loop that adds each part before
// it loads the next would pay a trip to memory per chunk)
__device__ __forceinline__ double ap_sum_parts(const double* __restrict__ part, int64_t w, int64_t jc, int chunks)
{
    double s = 0.0;
    for (int q0 = 0; q0 < chunks; q0 += 4) {
        double v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = q0 + u < chunks ? part[(int64_t)(q0 + u) * w + jc] : 0.0;
#pragma unroll
        for (int u = 0; u < 4; ++u) s += v[u];
    }
    return s;
}

// Outer pass.  Wave (p, split) owns the 64 output entries of word p and the terms of its split; lane q
// fetches word p of term (tile + q) and forms z of that term (the scale step: c times the chunk parts in
// order); z goes through a wave-private strip of LDS so that every lane can read every term's value.
template <typename TE>
__global__ void __launch_bounds__(kApOuterWaves* kWave)
    apply_outer_kernel(const uint64_t* __restrict__ bits, int64_t mw, int64_t w, const double* __restrict__ part, int chunks,
                       const TE* __restrict__ c, int64_t terms_per_split, double* __restrict__ ypart)
{
    __shared__ double zs[kApOuterWaves][2][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t p = (int64_t)blockIdx.x * kApOuterWaves + wv;  // word of the output this wave owns
    if (p >= mw) return;                                           // (no workgroup-wide barrier below)
    const int64_t split = blockIdx.y;
    const int64_t j0 = split * terms_per_split;
    const int64_t j1 = j0 + terms_per_split < w ? j0 + terms_per_split : w;
    auto fetch = [&](int64_t tile, uint64_t& word, double& z) {
        // unconditional loads; terms past the end re-read the last one and count as z = 0
        const int64_t j = tile + lane;
        const int64_t jc = j < j1 ? j : j1 - 1;
        word = bits[jc * mw + p];
        const double s = ap_sum_parts(part, w, jc, chunks);
        z = j < j1 ? (double)c[jc] * s : 0.0;
    };
    double a4[4] = {0.0, 0.0, 0.0, 0.0};
    if (j0 < j1) {
        // two tiles of 64 terms in flight ahead of the one being added
        uint64_t word_a, word_b;
        double z_a, z_b;
        fetch(j0, word_a, z_a);
        fetch(j0 + kWave < j1 ? j0 + kWave : j0, word_b, z_b);
        int b = 0;
        for (int64_t tile = j0; tile < j1; tile += kWave, b ^= 1) {
            const uint64_t word = word_a;
            zs[wv][b][lane] = z_a;
            word_a = word_b;
            z_a = z_b;
            fetch(tile + 2 * kWave < j1 ? tile + 2 * kWave : tile, word_b, z_b);
            // the strip is written and read by this wave only: LDS operations of one wave complete in order
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll 16
            for (int q = 0; q < kWave; ++q) a4[q & 3] = __builtin_fma(zs[wv][b][q], ap_sign(ap_word(word, q)), a4[q & 3]);
        }
    }
    ypart[split * (mw * 64) + p * 64 + lane] = (a4[0] + a4[1]) + (a4[2] + a4[3]);
}

// ------------------------------------------------------------------------------------------------
// Outer pass on the matrix cores (f32).  y_i = sum_j z_j s_j[i] is the same kind of contraction as the
// inner pass with the roles swapped: the terms are the contraction index and z plays the part of x (block
// fixed point per split of the terms: |z| 2^s < 2^30, four balanced base-256 digits, at most
// max|z| 2^-30 per term, exact sums afterwards; up to four vectors in the 16 columns).  The bitset is term-major, so
// the signs an instruction wants per lane (one output entry, 16 terms) sit in 16 different words: a wave loads word p of
// 64 consecutive terms (one per lane) and transposes every 16 x 16 block of bits in place (the four lower stages of the
// butterfly).  Field b (16 bits) of lane (a, i) then holds terms 16 a .. 16 a + 15 at entry 16 b + i, which is what lane
// (row i, quarter a) of the instruction for entries 16 b .. 16 b + 15 takes; byte q' of its operand dword q is term
// 16 a + 4 q' + q, a shift and a mask once the field's nibbles are spread over the bytes.
constexpr int kApFxMaxTerms = 2048;  // terms per split: one dword set (four terms) per thread of the workgroup
constexpr int kApFxMaxTiles = kApFxMaxTerms / kWave;
constexpr int kApFxOctet = 8;        // splits that are added as a tree (see apply_reduce_kernel)

// acc[b] += the 64 terms whose word of the output `mine` holds (one per lane) times their digits B
__device__ __forceinline__ void ap_outer_tile(uint64_t mine, ap_int4 B, int lane, ap_int4 (&acc)[4])
{
    uint32_t half[2] = {(uint32_t)mine, (uint32_t)(mine >> 32)};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        half[h] = bit_butterfly<8>(half[h], lane);
        half[h] = bit_butterfly<4>(half[h], lane);
        half[h] = bit_butterfly<2>(half[h], lane);
        half[h] = bit_butterfly<1>(half[h], lane);
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        // nibbles 0..3 of the field into bytes 0..3
        const uint32_t two = __builtin_amdgcn_perm(0u, half[b >> 1], (b & 1) ? 0x0C030C02u : 0x0C010C00u);
        const uint32_t nib = (two | (two << 4)) & 0x0F0F0F0Fu;
        ap_int4 A;
#pragma unroll
        for (int q = 0; q < 4; ++q) A[q] = (int)((nib >> q) & 0x01010101u);
        acc[b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A, B, acc[b], 0, 0, 0);
    }
}

template <int NV>
__global__ void __launch_bounds__(kApMfmaWaves* kWave)
    apply_outer_fx_kernel(const uint64_t* __restrict__ bits, int64_t mw, int64_t w, const double* __restrict__ part, int64_t pstride,
                          int chunks, const float* __restrict__ c, int nv, int64_t terms_per_split, double* __restrict__ ypart)
{
    constexpr int NC = 4 * NV;
    __shared__ __align__(16) uint32_t zd[kApFxMaxTerms / 4 * NC];  // [tile of 64 terms][quarter][column][dword]
    __shared__ double redmax[NV][kApMfmaWaves], redsum[NV][kApMfmaWaves];
    __shared__ int bad[NV];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int64_t p = (int64_t)blockIdx.x * kApMfmaWaves + wv;  // word of the output this wave owns
    const int64_t pc = p < mw ? p : mw - 1;
    const int64_t split = blockIdx.y;
    const int64_t j0 = split * terms_per_split;
    const int64_t j1 = j0 + terms_per_split < w ? j0 + terms_per_split : w;  // (the plan leaves no split empty)
    // lane q fetches word p of term (tile + q); terms past the end re-read the last one (their z is zero)
    auto fetch = [&](int64_t tile) {
        const int64_t j = j0 + tile * kWave + lane;
        return bits[(j < j1 ? j : j1 - 1) * mw + pc];
    };
    uint64_t next = fetch(0);

    // ---- z of this split in fixed point: thread t owns terms 16 (t / 4) + t mod 4 + 4 b
    if (tid < NV) bad[tid] = 0;
    __syncthreads();
    double zv[NV][4];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        if (v >= nv) continue;  // (as above)
        double amax = 0.0;
        bool finite = true;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int64_t j = j0 + 16 * (tid >> 2) + (tid & 3) + 4 * b;
            const int64_t jc = j < j1 ? j : j1 - 1;
            const double sp = ap_sum_parts(part + (int64_t)v * pstride, w, jc, chunks);
            zv[v][b] = j < j1 ? (double)c[jc] * sp : 0.0;
            finite = finite && (fabs(zv[v][b]) <= 1.7e308);
            amax = fmax(amax, fabs(zv[v][b]));
        }
        amax = ap_wave_max(amax);
        if (lane == 0) redmax[v][wv] = amax;
        if (!finite) bad[v] = 1;
    }
    __syncthreads();
    double inv_scale[NV];
    bool all_finite[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        inv_scale[v] = 1.0;
        all_finite[v] = true;
        if (v >= nv) continue;
        double amax = 0.0;
#pragma unroll
        for (int q = 0; q < kApMfmaWaves; ++q) amax = fmax(amax, redmax[v][q]);
        all_finite[v] = bad[v] == 0;
        int ex = 0;
        if (amax > 0.0) (void)frexp(amax, &ex);  // amax < 2^ex
        int sh = 30 - ex;
        sh = sh > 1000 ? 1000 : sh;              // (2^sh stays a normal number; smaller z round to zero)
        const double scale = ldexp(1.0, sh);
        inv_scale[v] = ldexp(1.0, -sh);
        int q4[4];
        uint32_t dig[4];
        double sum = 0.0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            q4[b] = all_finite[v] ? (int)rint(zv[v][b] * scale) : 0;
            sum += (double)q4[b];
        }
        ap_digits(q4, dig);
        uint32_t* dst = zd + ((tid >> 2) * NC + 4 * v) * 4 + (tid & 3);  // (tile * 4 + quarter = tid / 4)
#pragma unroll
        for (int jd = 0; jd < 4; ++jd) dst[jd * 4] = dig[jd];
        sum = ap_wave_sum(sum);
        if (lane == 0) redsum[v][wv] = sum;
    }
    __syncthreads();
    if (p >= mw) return;  // (no workgroup-wide barrier below)

    const int col = lane & 15, a = lane >> 4;
    const int jd = lane & 3, vc = (col & (NC - 1)) >> 2;
    double total = 0.0, inv = 0.0;
    bool fin = true;
#pragma unroll
    for (int v = 0; v < NV; ++v)
        if (v == vc) {
#pragma unroll
            for (int q = 0; q < kApMfmaWaves; ++q) total += redsum[v][q];
            inv = inv_scale[v];
            fin = all_finite[v];
        }
    const int ntiles = (int)((j1 - j0 + kWave - 1) / kWave);
    const ap_int4* zb = (const ap_int4*)zd + a * NC + (col & (NC - 1));
    ap_int4 acc[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[b] = ap_int4{0, 0, 0, 0};
    for (int t = 0; t < ntiles; ++t) {
        const uint64_t mine = next;
        if (t + 1 < ntiles) next = fetch(t + 1);
        ap_outer_tile(mine, zb[t * 4 * NC], lane, acc);
    }
    // register i of acc[b] = output entry 64 p + 16 b + 4 (lane / 16) + i, column lane mod 16
    const double digit_weight = (double)(1u << (8 * jd));
    double* out = ypart + (split * nv + vc) * (mw * 64) + p * 64 + 4 * a;
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            double v = (double)acc[b][i] * digit_weight;
            v += ap_dpp_xor_f64<1>(v);
            v += ap_dpp_xor_f64<2>(v);
            if (jd == 0 && col < NC && vc < nv) out[16 * b + i] = fin ? (total - 2.0 * v) * inv : __longlong_as_double(0x7FF8000000000000ll);
        }
}

// The same for `group` = 2, 4 or 8 splits in a row per workgroup, added as the tree of apply_reduce_kernel: with several
// vectors the workspace, which is sized for one, has no room for the results of every split.  A split stays what it is
// with one vector, the block of the fixed point, so that a vector keeps its bits in company; as many splits as there are
// threads for (four terms each) are put into fixed point at a time.  With few workgroups, as here, the end of a split
// weighs most: joining the digits in f64 in all four lanes and not one entry a lane took 70 instead of 63 us a call at
// 4096x4096, four vectors (one block of the fixed point for all terms of a workgroup, with fewer bits: 57), and workgroups
// of four or two waves, which form z more often, 75 and 92.
template <int NV>
__global__ void __launch_bounds__(kApMfmaWaves* kWave)
    apply_outer_group_kernel(const uint64_t* __restrict__ bits, int64_t mw, int64_t w, const double* __restrict__ part, int64_t pstride,
                             int chunks, const float* __restrict__ c, int nv, int64_t terms_per_split, int group,
                             double* __restrict__ ypart)
{
    constexpr int NC = 4 * NV;
    __shared__ __align__(16) uint32_t zd[kApFxMaxTerms / 4 * NC];  // [tile of 64 terms][quarter][column][dword]
    __shared__ double redmax[NV][kApFxMaxTiles], redsum[NV][kApFxMaxTiles], unit[NV][kApFxOctet];
    __shared__ int bad[NV];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int64_t p = (int64_t)blockIdx.x * kApMfmaWaves + wv;  // word of the output this wave owns
    const int64_t pc = p < mw ? p : mw - 1;
    const int64_t j0 = blockIdx.y * terms_per_split * group;
    const int64_t j1 = j0 + terms_per_split * group < w ? j0 + terms_per_split * group : w;  // (the plan leaves no split empty)
    const int tps = (int)(terms_per_split / kWave);                        // tiles per split, at most kApFxMaxTiles
    const int ntiles = (int)((j1 - j0 + kWave - 1) / kWave);
    const int fit = kApFxMaxTiles / tps, spr = fit < group ? fit : group;  // splits per round
    // lane q fetches word p of term (tile + q); terms past the end re-read the last one (their z is zero)
    auto fetch = [&](int64_t tile) {
        const int64_t j = j0 + tile * kWave + lane;
        return bits[(j < j1 ? j : j1 - 1) * mw + pc];
    };
    uint64_t next = fetch(0);
    const int col = lane & 15, a = lane >> 4;
    const int jd = lane & 3, vc = (col & (NC - 1)) >> 2;
    const ap_int4* zb = (const ap_int4*)zd + a * NC + (col & (NC - 1));
    // sums of 1, 2 and 4 splits that wait for their partners, and the last result
    double y1[4], y2[4], y4[4], r[4];
    int g = 0;
    if (tid < NV) bad[tid] = 0;
    for (int base = 0; base < ntiles; base += spr * tps) {
        // ---- z in fixed point: thread t owns terms 16 (t / 4) + t mod 4 + 4 b of the round, all of them of tile t / 16
        const int mytile = tid >> 4, mysplit = mytile / tps;
        const int64_t jr = j0 + (int64_t)base * kWave;
        const int64_t je = jr + spr * terms_per_split < j1 ? jr + spr * terms_per_split : j1;
        __syncthreads();  // (what the last round left is read)
        // sums over the chunks in order, a chunk of all vectors and terms at a time (their loads in flight together)
        double zv[NV][4];
        int64_t jc[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int64_t j = jr + 16 * (tid >> 2) + (tid & 3) + 4 * b;
            jc[b] = j < je ? j : je - 1;
#pragma unroll
            for (int v = 0; v < NV; ++v) zv[v][b] = 0.0;
        }
        for (int q = 0; q < chunks; ++q) {
            double x[NV][4];
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int b = 0; b < 4; ++b) x[v][b] = part[(v < nv ? v : 0) * pstride + q * w + jc[b]];
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int b = 0; b < 4; ++b) zv[v][b] += x[v][b];
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            if (v >= nv) continue;  // (as above)
            double amax = 0.0;
            bool finite = true;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                zv[v][b] = jr + 16 * (tid >> 2) + (tid & 3) + 4 * b < je ? (double)c[jc[b]] * zv[v][b] : 0.0;
                finite = finite && (fabs(zv[v][b]) <= 1.7e308);
                amax = fmax(amax, fabs(zv[v][b]));
            }
            amax = fmax(amax, ap_dpp_xor_f64<1>(amax));
            amax = fmax(amax, ap_dpp_xor_f64<2>(amax));
            amax = fmax(amax, ap_dpp_xor_f64<4>(amax));
            amax = fmax(amax, ap_dpp_xor_f64<8>(amax));
            if ((lane & 15) == 0) redmax[v][mytile] = amax;
            if (!finite) bad[v] = 1;
        }
        __syncthreads();
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            if (v >= nv) continue;
            double amax = 0.0;
            for (int q = 0; q < tps; ++q) {
                const int t = mysplit * tps + q;
                amax = fmax(amax, redmax[v][t < kApFxMaxTiles ? t : mytile]);  // (past the round's splits all z are zero)
            }
            const bool all_finite = bad[v] == 0;
            int ex = 0;
            if (amax > 0.0) (void)frexp(amax, &ex);  // amax < 2^ex
            int sh = 30 - ex;
            sh = sh > 1000 ? 1000 : sh;              // (2^sh stays a normal number; smaller z round to zero)
            const double scale = ldexp(1.0, sh);
            if (mysplit < spr && tid == mysplit * tps * 16) unit[v][mysplit] = ldexp(1.0, -sh);
            int q4[4];
            uint32_t dig[4];
            double sum = 0.0;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                q4[b] = all_finite ? (int)rint(zv[v][b] * scale) : 0;
                sum += (double)q4[b];
            }
            ap_digits(q4, dig);
            uint32_t* dst = zd + ((tid >> 2) * NC + 4 * v) * 4 + (tid & 3);  // (tile * 4 + quarter = tid / 4)
#pragma unroll
            for (int d = 0; d < 4; ++d) dst[d * 4] = dig[d];
            sum += ap_dpp_xor_f64<1>(sum);  // (integers below 2^36: exact)
            sum += ap_dpp_xor_f64<2>(sum);
            sum += ap_dpp_xor_f64<4>(sum);
            sum += ap_dpp_xor_f64<8>(sum);
            if ((lane & 15) == 0) redsum[v][mytile] = sum;
        }
        __syncthreads();
        if (p >= mw) continue;
        for (int s = 0; s < spr && base + s * tps < ntiles; ++s, ++g) {
            ap_int4 acc[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[b] = ap_int4{0, 0, 0, 0};
            double total = 0.0;
            const int t1 = (s + 1) * tps < ntiles - base ? (s + 1) * tps : ntiles - base;
            for (int t = s * tps; t < t1; ++t) {
                const uint64_t mine = next;
                if (base + t + 1 < ntiles) next = fetch(base + t + 1);
                total += redsum[vc][t];
                ap_outer_tile(mine, zb[t * 4 * NC], lane, acc);
            }
            const double inv = unit[vc][s];
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                // register i = entry 16 b + 4 a + i of the word, digit jd of it in lane jd of four: lane jd gathers the
                // digits of entry i = jd.  Two of them make an integer below 2^29 (digits up to 128, 2048 terms).
                int x[4], even, odd;
#pragma unroll
                for (int i = 0; i < 4; ++i) x[i] = acc[b][i] << (8 * (jd & 1));
                even = (jd & 1 ? x[1] : x[0]) + (int)ap_dpp_xor<1>((uint32_t)(jd & 1 ? x[0] : x[1]));
                odd = (jd & 1 ? x[3] : x[2]) + (int)ap_dpp_xor<1>((uint32_t)(jd & 1 ? x[2] : x[3]));
                const int keep = jd & 2 ? odd : even, got = (int)ap_dpp_xor<2>((uint32_t)(jd & 2 ? even : odd));
                const double v = __builtin_fma((double)(jd & 2 ? keep : got), 65536.0, (double)(jd & 2 ? got : keep));
                r[b] = (total - 2.0 * v) * inv;
                if (!(g & 1)) {
                    y1[b] = r[b];
                } else {
                    r[b] = y1[b] + r[b];
                    if (!(g & 2)) {
                        y2[b] = r[b];
                    } else {
                        r[b] = y2[b] + r[b];
                        if (!(g & 4)) y4[b] = r[b];
                        else r[b] = y4[b] + r[b];
                    }
                }
            }
        }
    }
    if (p >= mw || col >= NC || vc >= nv) return;
    const bool fin = bad[vc] == 0;  // (last written ahead of two barriers)
    double* out = ypart + ((int64_t)blockIdx.y * nv + vc) * (mw * 64) + p * 64 + 4 * a + jd;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        // a group that is cut short: the sums that wait, the shortest first
        double s = 0.0;
        if (g & 1) s = y1[b];
        if (g & 2) s = y2[b] + s;
        if (g & 4) s = y4[b] + s;
        if (g == 8) s = r[b];
        out[16 * b] = fin ? s : __longlong_as_double(0x7FF8000000000000ll);
    }
}

// y = sum of the splits, rounded once, for vector blockIdx.y of the launch (ypart: [split][vector][mpad]).  64 entries per
// workgroup.  The splits are cut into four runs that are added side by side (their loads in flight together) and joined in
// order.  f32 (TREE): eight splits at a time are added as a tree, ((0 + 1) + (2 + 3)) + ((4 + 5) + (6 + 7)), so that sums
// of 2, 4 or 8 neighbours that the outer pass has formed (then per_octet is 4, 2 or 1) lead to the same bits.
template <typename TE, bool TREE>
__global__ void __launch_bounds__(256)
    apply_reduce_kernel(const double* __restrict__ ypart, int splits, int per_octet, int64_t mpad, int64_t m, TE* __restrict__ y)
{
    __shared__ double run[4][64];
    const int r = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * 64 + r;
    const int64_t len = mpad;
    ypart += (int64_t)blockIdx.y * mpad;
    y += (int64_t)blockIdx.y * m;
    mpad *= gridDim.y;  // from one split to the next
    const int units = TREE ? (splits + per_octet - 1) / per_octet : splits;
    const int per = (units + 3) / 4;
    const int q0 = g * per, q1 = q0 + per < units ? q0 + per : units;
    double s = 0.0;
    if (i < len) {
        int q = q0;
        if constexpr (TREE) {
            for (; q < q1; ++q) {
                double x[kApFxOctet];
#pragma unroll
                for (int e = 0; e < kApFxOctet; ++e) {
                    const int sp = q * per_octet + e;
                    x[e] = e < per_octet && sp < splits ? ypart[(int64_t)sp * mpad + i] : 0.0;
                }
                s += ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
            }
        } else {
            for (; q + 4 <= q1; q += 4) {
                const double a0 = ypart[(int64_t)q * mpad + i], a1 = ypart[(int64_t)(q + 1) * mpad + i];
                const double a2 = ypart[(int64_t)(q + 2) * mpad + i], a3 = ypart[(int64_t)(q + 3) * mpad + i];
                s = (((s + a0) + a1) + a2) + a3;
            }
            for (; q < q1; ++q) s += ypart[(int64_t)q * mpad + i];
        }
    }
    run[g][r] = s;
    __syncthreads();
    if (g == 0 && i < m) y[i] = (TE)(((run[0][r] + run[1][r]) + run[2][r]) + run[3][r]);
}

}  // namespace

void apply_plan(int64_t nin, int64_t nout, int64_t w, ApplyPlan* pl)
{
    const int64_t win = (nin + 63) / 64, wout = (nout + 63) / 64;
    pl->chunks = (int)((win + kApChunkWords - 1) / kApChunkWords);
    if (pl->chunks < 1) pl->chunks = 1;
    // inner pass: enough waves to fill the device, enough terms per wave to pay for loading its chunk of x
    int64_t tpw = (w * pl->chunks + 4095) / 4096;
    if (tpw < 8) tpw = 8;
    if (tpw > 64) tpw = 64;
    pl->terms_per_wave = (int)tpw;
    // outer pass: one wave per word of the output and split of the terms
    int64_t splits = wout > 0 ? (4096 + wout - 1) / wout : 1;
    if (splits > 64) splits = 64;
    while (splits > 1 && (w + splits - 1) / splits < 32) --splits;
    if (splits < 1) splits = 1;
    pl->terms_per_split = (w + splits - 1) / splits;
    if (pl->terms_per_split < 1) pl->terms_per_split = 1;
    pl->splits = (int)((w + pl->terms_per_split - 1) / pl->terms_per_split);
    if (pl->splits < 1) pl->splits = 1;
    // outer pass in fixed point (f32): a workgroup takes 8 words of the output and one split of the terms
    // (whole tiles of 64, at most kApFxMaxTerms); two to four workgroups per compute unit
    {
        const int64_t gx = (wout + kApMfmaWaves - 1) / kApMfmaWaves;
        const int64_t target = gx >= 16 ? 1024 : 512;
        int64_t want = gx > 0 ? (target + gx - 1) / gx : 1;
        const int64_t least = (w + kApFxMaxTerms - 1) / kApFxMaxTerms, most = (w + kWave - 1) / kWave;
        if (want > most) want = most;
        if (want < least) want = least;
        if (want < 1) want = 1;
        int64_t tps = ((w + want - 1) / want + kWave - 1) / kWave * kWave;
        if (tps < kWave) tps = kWave;
        pl->terms_per_split_fx = tps;
        pl->splits_fx = (int)((w + tps - 1) / tps);
        if (pl->splits_fx < 1) pl->splits_fx = 1;
    }
    pl->off_part = 0;
    pl->parts = pl->chunks;  // slices of <t_j, x> the inner pass writes per term
    pl->off_ypart = pl->off_part + (size_t)pl->parts * (size_t)w * 8;
    const int most_splits = pl->splits > pl->splits_fx ? pl->splits : pl->splits_fx;
    pl->bytes = pl->off_ypart + (size_t)most_splits * (size_t)wout * 64 * 8;
    if (pl->bytes < 8) pl->bytes = 8;
}

namespace {

template <int NV>
hipError_t launch_fx(const uint64_t* in_bits, const uint64_t* out_bits, const float* c, int64_t nin, int64_t nout, int64_t w,
                     const float* x, int nv, float* y, const ApplyPlan& pl, int group, void* workspace, hipStream_t st)
{
    const int64_t win = (nin + 63) / 64, wout = (nout + 63) / 64;
    const int64_t pstride = (int64_t)pl.parts * w;
    double* part = (double*)workspace;
    double* ypart = part + nv * pstride;
    // a workgroup per tile of 64 terms; several tiles per workgroup once there are more workgroups than compute units, which
    // hold one each: the fixed point, half of a workgroup's time with seven tiles, is paid for once
    const int64_t tiles = (w + kApFxTile - 1) / kApFxTile;
    int tpw = (int)((tiles * pl.chunks + kApInnerGrid - 1) / kApInnerGrid);
    if (tpw < 1) tpw = 1;
    const int64_t wgs = (tiles + tpw - 1) / tpw;
    const dim3 gi((unsigned)wgs, (unsigned)pl.chunks);
    if (tpw == 1)
        hipLaunchKernelGGL((apply_inner_fx_kernel<NV, true>), gi, dim3(kApFxThreads), 0, st, in_bits, win, w, x, nv, nin, part, pstride, tpw);
    else
        hipLaunchKernelGGL((apply_inner_fx_kernel<NV, false>), gi, dim3(kApFxThreads), 0, st, in_bits, win, w, x, nv, nin, part, pstride, tpw);
    const int splits = (pl.splits_fx + group - 1) / group;
    dim3 go((unsigned)((wout + kApMfmaWaves - 1) / kApMfmaWaves), (unsigned)splits);
    bool one_each = true;
    if constexpr (NV > 1) {
        if (group > 1) {
            hipLaunchKernelGGL((apply_outer_group_kernel<NV>), go, dim3(kApMfmaWaves * kWave), 0, st, out_bits, wout, w, part, pstride,
                               pl.parts, c, nv, pl.terms_per_split_fx, group, ypart);
            one_each = false;
        }
    }
    if (one_each)
        hipLaunchKernelGGL((apply_outer_fx_kernel<NV>), go, dim3(kApMfmaWaves * kWave), 0, st, out_bits, wout, w, part, pstride, pl.parts, c,
                           nv, pl.terms_per_split_fx, ypart);
    hipLaunchKernelGGL((apply_reduce_kernel<float, true>), dim3((unsigned)((nout + 63) / 64), (unsigned)nv), dim3(256), 0, st, ypart, splits,
                       kApFxOctet / group, wout * 64, nout, y);
    return hipGetLastError();
}

}  // namespace

// nvec vectors (rows of x and y).  f32: up to four share a pass over the bits, with the bits of y that each has alone: the
// splits of the terms (the blocks of the fixed point) and the order of their sums do not depend on the number of vectors
// or on the workspace.  The workspace is sized for one vector whatever their number: several take it with the sums of
// groups of splits, and where even those do not fit, in smaller sets, as many at once as fit.
hipError_t launch_apply(const uint64_t* in_bits, const uint64_t* out_bits, const void* c, scd_dtype dt, int64_t nin,
                        int64_t nout, int64_t w, const void* x, int64_t nvec, void* y, void* workspace, size_t workspace_bytes, hipStream_t st)
{
    ApplyPlan pl;
    apply_plan(nin, nout, w, &pl);
    const int64_t win = (nin + 63) / 64, wout = (nout + 63) / 64;
    double* part = (double*)((char*)workspace + pl.off_part);
    double* ypart = (double*)((char*)workspace + pl.off_ypart);
    if (nout == 0) return hipSuccess;
    const unsigned gr = (unsigned)((nout + 63) / 64);
    if (w == 0 || nin == 0) {
        // the empty sum: a reduce over no splits writes zeros
        for (int64_t v = 0; v < nvec; ++v) {
            if (dt == SCD_F32)
                hipLaunchKernelGGL((apply_reduce_kernel<float, true>), dim3(gr), dim3(256), 0, st, ypart, 0, kApFxOctet, wout * 64, nout, (float*)y + v * nout);
            else
                hipLaunchKernelGGL((apply_reduce_kernel<double, false>), dim3(gr), dim3(256), 0, st, ypart, 0, 1, wout * 64, nout, (double*)y + v * nout);
        }
        return hipGetLastError();
    }
    if (dt == SCD_F32) {
        for (int64_t v = 0; v < nvec;) {
            const float* xv = (const float*)x + v * nin;
            float* yv = (float*)y + v * nout;
            int group = 1;
            auto fits = [&](int64_t nv) {  // sets group to the smallest that fits
                if (nv == 1) return group = 1, true;
                const int64_t room = (int64_t)(workspace_bytes / 8) - nv * pl.parts * w;
                const int64_t most = room > 0 ? room / (nv * wout * 64) : 0;
                for (group = 1; group <= kApFxOctet; group *= 2)
                    if ((pl.splits_fx + group - 1) / group <= most) return true;
                return false;
            };
            int64_t nv = nvec - v < 4 ? nvec - v : 4;
            while (!fits(nv)) --nv;
            hipError_t e;
            if (nv > 2) e = launch_fx<4>(in_bits, out_bits, (const float*)c, nin, nout, w, xv, (int)nv, yv, pl, group, workspace, st);
            else if (nv == 2) e = launch_fx<2>(in_bits, out_bits, (const float*)c, nin, nout, w, xv, 2, yv, pl, group, workspace, st);
            else e = launch_fx<1>(in_bits, out_bits, (const float*)c, nin, nout, w, xv, 1, yv, pl, group, workspace, st);
            if (e != hipSuccess) return e;
            v += nv;
        }
        return hipSuccess;
    }
    for (int64_t v = 0; v < nvec; ++v) {
        const int64_t waves = (w + pl.terms_per_wave - 1) / pl.terms_per_wave;
        dim3 gi((unsigned)((waves + kApInnerWaves - 1) / kApInnerWaves), (unsigned)pl.chunks);
        hipLaunchKernelGGL((apply_inner_kernel<double>), gi, dim3(kApInnerWaves * kWave), 0, st, in_bits, win, w,
                           (const double*)x + v * nin, nin, part, pl.terms_per_wave);
        dim3 go((unsigned)((wout + kApOuterWaves - 1) / kApOuterWaves), (unsigned)pl.splits);
        hipLaunchKernelGGL((apply_outer_kernel<double>), go, dim3(kApOuterWaves * kWave), 0, st, out_bits, wout, w, part,
                           pl.parts, (const double*)c, pl.terms_per_split, ypart);
        hipLaunchKernelGGL((apply_reduce_kernel<double, false>), dim3(gr), dim3(256), 0, st, ypart, pl.splits, 1, wout * 64, nout, (double*)y + v * nout);
    }
    return hipGetLastError();
}

}  // namespace scd
